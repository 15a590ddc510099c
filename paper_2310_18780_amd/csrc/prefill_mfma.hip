// Prefill of the distilled modal recurrence on the matrix cores (MFMA).
//
// The recurrence of Proposition "modal_realization" (Sec. 3.4), cut into
// chunks of C = 16 steps (the blocked form of the parallel-scan prefill of
// Sec. 3.4), is three dense contractions per channel c, over 16 columns (the
// MFMA N dimension), each one chunk of one batch row:
//
//   Y    = T U + W X_in            outputs of the chunk          [C x 16]
//   S    = P U                      chunk end state from zero     [2d x 16]
//   X_in of the row's next chunk = lambda^C X_in + S              (scan)
//
//   U[j][n] = input at step j of column n's chunk
//   T[t][j] = h_{t-j} for j <= t, else 0              (Toeplitz of the filter:
//             h_0 = h0, h_m = Re sum_n R_n lambda_n^(m-1), eq. "modal_impulse")
//   P[n][j] = Re / Im of lambda_n^(C-1-j)             (Vandermonde, 2d real rows)
//   W[t][n] = Re(R_n lambda_n^t) on the Re component of mode n and
//             -Im(R_n lambda_n^t) on its Im component, so that
//             W X_in = Re sum_n R_n lambda_n^t x_in,n
//
// so that y_t = Re(R x_t) + h0 u_t at every step and the last entry state is x_T.
//
// Columns.  The 16 columns are 16/S batch rows times S consecutive chunks of
// each.  S = 1, for many rows: a column is a row, its states stay in registers.
// S = 2, 4 or 16 (256 steps of one row at a time), for few: the end states are
// exchanged through LDS (within the wave that owns the channel, no barrier), one
// lane per (channel, mode) walks the columns of a row in order and leaves the entry
// states in their place.  The prompt of one row is thus a single pass at any batch
// size.  Only where (channel group, row) pairs
// are too few to occupy the GPU is the prompt cut into segments as well
// (segmented plan): a pass for the segments' end states from zero, a carry,
// and the pass from the carried entry states.
//
// Arithmetic: v_mfma_f32_16x16x32_bf16 (float32 accumulation).  A float32
// operand is split into bfloat16 terms a = a1 + a2 (+ a3), each the nearest
// bfloat16 of what the previous terms leave.  U has K = 16, half of the
// instruction's K, so two products share one instruction: [a1 | a2] times
// [u; u] is (a1 + a2) u.  Two kernels:
//   three terms of every operand, products of the six pairs with i + j <= 2 (an
//   error of a few float32 ulps of |a b|): every size that the VALU scan would take
//   otherwise, and unaligned u or y;
//   two terms where the outputs allow it: the plans that callers name, or that the
//   automatic call takes at their sizes.  With float32 u and y the entry states
//   have two terms (error of the outputs 2e-6 of their norm at radii U[0.9, 0.9999],
//   2.4e-6 at U[0.999, 0.99999]; 3.1e-6 and 3.6e-6 without the product of the second
//   terms), all else three.  With bfloat16 u (exact in one term) and y (rounded)
//   T, W and the entry states have two (2^-17 of a row's size, lost in the rounding
//   but of outputs that cancel), P three: the end states, and through the scan
//   x_T, are formed at float32 precision in either kernel.
// Small products come before large ones: the sums are then rounded at their full
// size only once or twice (x_T at radii U[0, 0.5]: 6.5e-8 against 8.2e-8).
// The matrices and lambda^C come from float64 powers, rounded
// once; lambda^C keeps the error of its rounding beside it (it would repeat every
// 16 steps with the same sign).  d is padded to a multiple of 16 with
// modes of zero operands.
//
// What bounds it.  No unit is full: a tile (256 (row, step) cells of a workgroup's
// channels) takes 2 to 3 us, of which the matrix units are busy for 0.19 (bfloat16 d =
// 16; float32 d = 32 0.24, d = 64 0.27; 16 cycles per product) and vector
// instructions issue for 0.31 to 0.33 (4 cycles each, by the counters of the three
// prefills); the two waves of a SIMD wait for 0.4 of their time, for operands from LDS
// and for each other at the tile's barrier, S > 1 also for the walk.  Beside it the
// movement of u and y, whose rate depends on how much of it
// is in flight, in the opposite sense of a plain copy: moved without arithmetic
// in 64-byte pieces of lines that lie D elements apart, the [64, 4096, 2048] bfloat16
// prompt takes 0.43 ms (5.0 TB/s; a contiguous copy of these bytes 0.45 ms) with 8 KiB
// of loads in flight per workgroup and CU, 0.60-0.65 ms with 16 KiB, 0.71-0.77 ms with 32
// KiB; 32-byte pieces take 0.54-0.61 ms.  Hence
//   - chunks of 16 steps: the A operands of a channel are 7 KiB (bfloat16, d <= 16,
//     two terms) to 30 KiB (d = 64), half of what chunks of 32 steps need, so that a
//     wave holds up to four channels and moves pieces of up to 64 bytes;
//   - loads a tile ahead in two halves, staged as they arrive;
//   - independent chains of products issued in turn, lambda^C and its correction
//     read from LDS, the tile loop free of any other path.
// Against chunks of 32 steps in 16- to 32-byte pieces (and, for few rows, one pass
// for segment states more; for other d or D the VALU scan): [16, 2048, 768] float32
// d = 16 167 -> 74 us; [4, 65536, 1024] float32 d = 32 938 -> 690 us; [256, 1024, 2048]
// float32 d = 64 2280 -> 2180 us; [64, 4096, 2048] bfloat16 d = 16 601 -> 583 us; [7,
// 1999, 1000] bfloat16 d = 12 (VALU) 112 -> 34 us.  Slower than they were are some
// batches of 50 to 120 rows with bfloat16 u and y, whose wider channel groups fill
// the last round of CUs worse ([59, 256, 2272] d = 32 95 -> 119 us, [117, 512, 256] 39 -> 46
// us).  Also measured: the pairs' loads issued
// half a tile ahead 1.04-1.15x the time, one at a time with a forced wait between
// the halves 1.02-1.5x, outputs stored at the tile's start 1.05-1.16x, scalar-base
// addresses for the stores 1.1-1.2x.
#include "prefill_mfma.hpp"

#include "lh_internal.hpp"

namespace lh {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kC = kMfmaChunk;
constexpr int kSetupThreads = 256;
constexpr int64_t kCus = 256;       // workgroups that run at a time, one per CU
constexpr int64_t kTile = 256;      // (row, step) cells of a tile
constexpr int64_t kMaxOffset = 0x7fffffff;  // bytes a workgroup's rows span

__device__ __forceinline__ void split3(float v, __bf16 (&t)[3])
{
    t[0] = static_cast<__bf16>(v);
    const float r1 = v - static_cast<float>(t[0]);
    t[1] = static_cast<__bf16>(r1);
    const float r2 = r1 - static_cast<float>(t[1]);
    t[2] = static_cast<__bf16>(r2);
}

// One workgroup per channel: float64 powers lambda_n^e (e = 0 .. C) and filter
// taps in LDS, then the A operands (rounded to float32, split into bfloat16
// terms) in lane order at frag[(c F + f) 64 + lane], and lambda^C rounded to
// float32 with what its rounding left, relative to it.  Lane m + 16 g of a fragment
// holds row m, K indices 8 g .. 8 g + 7.  For T and P (K = 16) K index 8 g + i is
// step 8 (g % 2) + i of term a (g < 2) or b of the fragment's pair [a | b]; row m of
// P fragment pair f is the (m % 2 ? Im : Re) of mode 8 f + m / 2.  For W, K index
// 8 g + i is component (i % 2 ? Im : Re) of mode 16 q + 8 (i / 4) + 2 g + (i % 4) / 2,
// the one that the same lane holds in the accumulators of P fragments 2 q + i / 4.
// Latency bound at few channels (two loads, the powers, three barriers): a lane
// forms a power by repeated squaring, and a wave forms all fragments of a matrix
// tile from one evaluation of its values (D = 768, d = 16: 8-10 us before, 5.6-7.6 us
// so; D = 2048, d = 64: 41 and 28 us).
template <bool BF, int DM, bool X3>
__global__ __launch_bounds__(kSetupThreads) void mfma_setup_kernel(const float2* __restrict__ lam,
                                                                   const float2* __restrict__ R,
                                                                   const float* __restrict__ h0,
                                                                   int d, bf16x8* __restrict__ frag,
                                                                   float4* __restrict__ lamc)
{
    using Cf = MfmaTiling<BF, DM, X3>;
    constexpr int dp = 16 * DM, F = Cf::kFrags, NTW = BF && !X3 ? 2 : 3;
    __shared__ double pwr[dp][kC + 1], pwi[dp][kC + 1];
    __shared__ double rre[dp], rim[dp];
    __shared__ double taps[kC];
    const int c = blockIdx.x;
    const int tid = threadIdx.x;
    static_assert(kSetupThreads == 16 * kC, "a lane per power and per tap part");
    const double h0c = tid == 0 ? double(h0[c]) : 0.0;
    float2 ll[DM], rl[DM];
#pragma unroll
    for (int k = 0; k < DM; ++k) {  // modes tid / 16 + 16 k; padded modes are zero throughout
        const int n = tid / 16 + 16 * k;
        const bool in = n < d;
        ll[k] = in ? lam[int64_t(c) * d + n] : make_float2(0.f, 0.f);
        rl[k] = in ? R[int64_t(c) * d + n] : make_float2(0.f, 0.f);
    }
#pragma unroll
    for (int k = 0; k < DM; ++k) {
        const int n = tid / 16 + 16 * k, e = tid % 16;
        double br = ll[k].x, bi = ll[k].y, pr = n < d ? 1.0 : 0.0, pi = 0.0;
#pragma unroll
        for (int bit = 0; bit < 4; ++bit) {  // lambda^e, and the base to lambda^16
            const double t = pr * br - pi * bi, ti = pr * bi + pi * br;
            if (e >> bit & 1) {
                pr = t;
                pi = ti;
            }
            const double sr = br * br - bi * bi;
            bi = 2.0 * br * bi;
            br = sr;
        }
        pwr[n][e] = pr;
        pwi[n][e] = pi;
        if (e == 0) {
            rre[n] = rl[k].x;
            rim[n] = rl[k].y;
            const float hr = float(br), hi = float(bi);
            const double dr = br - hr, di = bi - hi, q = double(hr) * hr + double(hi) * hi;
            // relative rounding error (none for values near underflow, whose states vanish)
            const bool tiny = !(q > 1e-60);
            lamc[int64_t(c) * dp + n] =
                make_float4(hr, hi, tiny ? 0.f : float((dr * hr + di * hi) / q),
                            tiny ? 0.f : float((di * hr - dr * hi) / q));
        }
    }
    __syncthreads();
    {  // h_0 = h0, h_m = Re sum_n R_n lambda_n^(m-1): 16 lanes per tap
        const int m = tid / 16, part = tid % 16;
        double h = 0.0;
        if (m > 0)
            for (int n = part; n < dp; n += 16) h += rre[n] * pwr[n][m - 1] - rim[n] * pwi[n][m - 1];
        for (int o = 8; o > 0; o /= 2) h += __shfl_xor(h, o, 16);
        if (part == 0) taps[m] = m == 0 ? h0c : h;
    }
    __syncthreads();
    const int lane = tid % 64, g = lane / 16, m = lane % 16;
    bf16x8* const out = frag + int64_t(c) * F * 64 + lane;
    // tiles: P (2 DM), W (DM), T
    for (int tile = tid / 64; tile < 3 * DM + 1; tile += kSetupThreads / 64) {
        bf16x8 t[3];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int j = 8 * (g % 2) + i;
            double val;
            if (tile < 2 * DM) {
                const int mode = 8 * tile + m / 2;
                val = m % 2 ? pwi[mode][kC - 1 - j] : pwr[mode][kC - 1 - j];
            } else if (tile < 3 * DM) {
                const int mode = 16 * (tile - 2 * DM) + 8 * (i / 4) + 2 * g + i % 4 / 2;
                val = i % 2 ? -(rre[mode] * pwi[mode][m] + rim[mode] * pwr[mode][m])
                            : rre[mode] * pwr[mode][m] - rim[mode] * pwi[mode][m];
            } else {
                val = j <= m ? taps[m - j] : 0.0;
            }
            __bf16 s[3];
            split3(float(val), s);
            t[0][i] = s[0];
            t[1][i] = s[1];
            t[2][i] = s[2];
        }
        if (tile >= 2 * DM && tile < 3 * DM) {
#pragma unroll
            for (int k = 0; k < NTW; ++k) out[(Cf::kW + (tile - 2 * DM) * NTW + k) * 64] = t[k];
        } else {  // [a1 | a2], then [a1 | a3], or with bfloat16 u [a3 | 0] (if T has it)
            const int f = tile < 2 * DM ? Cf::kP + 2 * tile : 0;
            const bf16x8 none = {};
            out[f * 64] = g < 2 ? t[0] : t[1];
            if (!BF) out[(f + 1) * 64] = g < 2 ? t[0] : t[2];
            if (BF && (X3 || tile < 2 * DM)) out[(f + 1) * 64] = g < 2 ? t[2] : none;
        }
    }
}

int modes16(int64_t d) { return int((d + 15) / 16); }

size_t frag_bytes(bool bf16_io, bool two_terms, int64_t D, int64_t d)
{
    const int dm = modes16(d);
    return size_t(D) * size_t(bf16_io && two_terms ? 1 + 6 * dm : 2 + 7 * dm) * 64 * sizeof(bf16x8);
}

template <bool BF, int DM, bool X3>
hipError_t launch_setup_tiled(const float2* lam, const float2* R, const float* h0, int64_t D,
                              int64_t d, void* workspace, hipStream_t stream)
{
    hipLaunchKernelGGL((mfma_setup_kernel<BF, DM, X3>), dim3(uint32_t(D)), dim3(kSetupThreads), 0,
                       stream, lam, R, h0, int(d), static_cast<bf16x8*>(workspace),
                       reinterpret_cast<float4*>(static_cast<char*>(workspace) +
                                                 frag_bytes(BF, !X3, D, d)));
    return hipGetLastError();
}

template <bool BF>
hipError_t launch_setup(const float2* lam, const float2* R, const float* h0, int64_t D, int64_t d,
                        bool two_terms, void* workspace, hipStream_t stream)
{
    // tables of float32 u and y serve either kernel
    switch (modes16(d)) {
        case 1:
            if (BF && two_terms)
                return launch_setup_tiled<BF, 1, !BF>(lam, R, h0, D, d, workspace, stream);
            return launch_setup_tiled<BF, 1, true>(lam, R, h0, D, d, workspace, stream);
        case 2:
            if (BF && two_terms)
                return launch_setup_tiled<BF, 2, !BF>(lam, R, h0, D, d, workspace, stream);
            return launch_setup_tiled<BF, 2, true>(lam, R, h0, D, d, workspace, stream);
        case 3: return launch_setup_tiled<BF, 3, true>(lam, R, h0, D, d, workspace, stream);
        case 4: return launch_setup_tiled<BF, 4, true>(lam, R, h0, D, d, workspace, stream);
        default: return hipErrorInvalidValue;
    }
}

static_assert(MfmaTiling<true, 1, false>::kFrags == 7 && MfmaTiling<true, 2, false>::kFrags == 13 &&
                  MfmaTiling<true, 1, true>::kFrags == 9 && MfmaTiling<true, 4, true>::kFrags == 30 &&
                  MfmaTiling<false, 1, true>::kFrags == 9 && MfmaTiling<false, 4, false>::kFrags == 30,
              "frag_bytes counts these fragments");

// Time of a pass in tiles of the busiest CU: its workgroups run one at a time,
// each loading its operands (worth about kEntry tiles) and walking its tiles.
constexpr int64_t kEntry = 2;
int64_t pass_tiles(int64_t groups, int64_t rows, int64_t steps, int s)
{
    const int64_t wgs = groups * ((rows + 16 / s - 1) / (16 / s));
    return (wgs + kCus - 1) / kCus * ((steps + 16 * s - 1) / (16 * s) + kEntry);
}

}  // namespace

// Sizes that the explicit matrix-core requests take.
bool mfma_supported(int64_t B, int64_t D, int64_t d, int64_t T, bool bf16_io)
{
    const bool tiles = d == 16 || d == 32 ? D % 8 == 0 : d == 64 && !bf16_io && D % 4 == 0;
    return tiles && T >= 1 && B <= (INT64_C(1) << 30) && D <= (INT64_C(1) << 30);
}

// Sizes that the kernel takes: whole 8-byte pieces of channels, moved back into
// range at the end of a row, so either a whole channel group or whole pieces; a
// tile of one row within the 32-bit offsets.
bool mfma_possible(int64_t B, int64_t D, int64_t d, int64_t T, bool bf16_io)
{
    const int64_t piece = bf16_io ? 4 : 2;
    return d <= kMfmaMaxModes && T >= 1 && D >= piece &&
           (D % piece == 0 || D >= mfma_channels(bf16_io, modes16(d))) &&
           B <= (INT64_C(1) << 30) && (kTile + 1) * D * (bf16_io ? 2 : 4) <= kMaxOffset;
}

// Bytes of the tables.  The named plans keep the size that their callers may
// have stored ((4 d/16 + 2) x 3 fragments and lambda^C), which covers them.
size_t mfma_workspace_bytes(int64_t D, int64_t d)
{
    const int dm = int(d / 16);
    const size_t frag = size_t(D) * (4 * dm + 2) * 3 * 64 * sizeof(bf16x8);
    return (frag + 255) / 256 * 256 + size_t(D) * d * sizeof(float2);
}

size_t mfma_table_bytes(bool bf16_io, bool two_terms, int64_t D, int64_t d)
{
    return frag_bytes(bf16_io, two_terms, D, d) + size_t(D) * 16 * modes16(d) * sizeof(float4);
}

// Segment slots of the segmented plan: the fewest segments (a power of two,
// each a multiple of 32 and at least 256 steps long) whose (batch row, segment)
// columns give at least 1024 workgroups of 8 channels and 16 columns, else the
// most segments allowed; 0 when T does not split so.
int64_t mfma_segments(int64_t B, int64_t D, int64_t d, int64_t T)
{
    constexpr int64_t kSegWorkgroups = 1024, kMinSeg = 256;
    const int64_t cw = d == 64 ? 4 : 8;
    int64_t best = 0;
    for (int64_t s = 2; T % (s * 32) == 0 && T / s >= kMinSeg; s *= 2) {
        best = s;
        if ((B * s + 15) / 16 * ((D + cw - 1) / cw) >= kSegWorkgroups) break;
    }
    return best;
}

// Columns and segments of a call.  Segments (of whole tiles) only where they
// shorten the walk of the busiest CU by more than the extra pass, carry and
// launches cost (about kExtra tiles).
MfmaCut mfma_cut(int64_t B, int64_t D, int64_t d, int64_t T, bool bf16_io, int64_t max_seg)
{
    constexpr int64_t kExtra = 6;
    const int64_t cw = mfma_channels(bf16_io, modes16(d));
    const int64_t groups = (D + cw - 1) / cw;
    MfmaCut best{16, 1, T, pass_tiles(groups, B, T, 16)};
    const int64_t row_bytes = T * D * (bf16_io ? 2 : 4);  // T D 8 does not overflow (checked sizes)
    for (int s : {4, 2, 1}) {
        if (row_bytes > kMaxOffset / (16 / s)) continue;
        const int64_t t = pass_tiles(groups, B, T, s);
        if (t <= best.tiles) best = MfmaCut{s, 1, T, t};
    }
    for (int64_t k = 2; k <= max_seg; k *= 2) {
        const int64_t len = ((T + k - 1) / k + kTile - 1) / kTile * kTile;
        const int64_t nseg = (T + len - 1) / len;
        if (nseg < 2 || len < 2 * kTile || nseg > max_seg || B * nseg > 0x7fffffff) continue;
        const int64_t t = pass_tiles(groups, B * (nseg - 1), len, 16) +
                          pass_tiles(groups, B * nseg, len, 16) + kExtra;
        if (t < best.tiles) best = MfmaCut{16, int(nseg), len, t};
    }
    return best;
}

// Time of the three-term kernels in microseconds: launches, the tables, then the passes
// of the busiest CU, whose workgroups each load their operands and walk their tiles.
double mfma_us(int64_t B, int64_t D, int64_t d, int64_t T, bool bf16_io, const MfmaCut& cut)
{
    constexpr double kTileUs[2][4] = {{1.65, 2.87, 2.0, 2.8}, {2.56, 2.6, 1.35, 2.27}};
    const int dm = modes16(d);
    const int64_t cw = mfma_channels(bf16_io, dm), groups = (D + cw - 1) / cw;
    auto pass = [&](int64_t rows, int64_t steps) {
        const int64_t wgs = groups * ((rows + 16 / cut.s - 1) / (16 / cut.s));
        const double tile = kTileUs[bf16_io][dm - 1] * (cut.s == 1 ? 1.2 : 1.0);
        return double((wgs + kCus - 1) / kCus) *
               (4.5 + tile * double((steps + 16 * cut.s - 1) / (16 * cut.s)));
    };
    const double base = 5.1 + 6.1e-3 * double(D) * dm;
    if (cut.nseg == 1) return base + pass(B, T);
    return base + 5.9 + 0.75 * pass(B * (cut.nseg - 1), cut.seg_len) + pass(B * cut.nseg, cut.seg_len);
}

hipError_t launch_mfma_setup(const float2* lam, const float2* R, const float* h0, int64_t D,
                             int64_t d, bool bf16_io, bool two_terms, void* workspace,
                             hipStream_t stream)
{
    (void)hipGetLastError();
    if (D > 0x7fffffff) return hipErrorInvalidConfiguration;
    return bf16_io ? launch_setup<true>(lam, R, h0, D, d, two_terms, workspace, stream)
                   : launch_setup<false>(lam, R, h0, D, d, two_terms, workspace, stream);
}

hipError_t launch_mfma_pass(bool outputs, const float2* lam, const float2* R, const float* h0,
                            const void* u, bool bf16_io, int64_t B, int64_t D, int64_t d,
                            int64_t T, const MfmaCut& cut, float2* xs, float2* state, void* y,
                            const void* workspace, hipStream_t stream)
{
    (void)hipGetLastError();
    if (cut.nseg > 1 && (cut.s != 16 || cut.seg_len % kTile != 0 ||
                         (T + cut.seg_len - 1) / cut.seg_len != cut.nseg))
        return hipErrorInvalidValue;
    MfmaArgs a{};
    a.lam = lam;
    a.R = R;
    a.h0 = h0;
    a.u = u;
    a.y = y;
    a.state = state;
    a.frag = workspace;
    a.lamc = static_cast<const char*>(workspace) + frag_bytes(bf16_io, cut.two_terms, D, d);
    a.xs = xs;
    a.T = T;
    a.seg_len = cut.seg_len;
    a.B = int(B);
    a.D = int(D);
    a.d = int(d);
    a.nseg = cut.nseg;
    a.two_terms = cut.two_terms;
    return bf16_io ? launch_mfma_kernel_bf16(modes16(d), cut.s, outputs, a, stream)
                   : launch_mfma_kernel_f32(modes16(d), cut.s, outputs, a, stream);
}

}  // namespace lh
