// Prefill of the distilled modal recurrence: all prompt outputs and the
// post-prompt state (Sec. 3.4, "fast pre-filling").
//
// The prompt of each (b, c) row is cut into nchunks chunks of C steps that run
// in parallel (the blocked form of the parallel-scan prefill of Sec. 3.4):
//
//   1. pow    : lambda^C per (c, n), computed in float64 and rounded once;
//   2. state  : each chunk but the last runs x <- lambda x + u from x = 0 and
//               writes its end state s_k (no outputs);
//   3. carry  : per (b, c, n), x_in[0] = 0, x_in[k+1] = lambda^C x_in[k] + s_k,
//               written over s_k (a sequential scan over <= a few dozen chunks);
//   4. output : each chunk restarts from x_in[k] and runs the full step of
//               Proposition "modal_realization" (y_t = Re(R x_t) + h0 u_t, then
//               x_{t+1} = lambda x_t + u_t), writing y; the last chunk writes
//               x_T to the state.
//
// When the plan has one chunk (enough (b, c) rows to fill the GPU), only the
// output pass runs, from x = 0: a single sequential pass per row.
//
// Lane layout of the state/output passes: a wavefront covers CW = 64 / LPR
// consecutive channels of one (b, chunk); lane l handles channel
// cblk * CW + (l % CW) and modes [(l / CW) * MPL, (l / CW + 1) * MPL).  Every
// time step a wave therefore reads (and writes) one contiguous run of CW
// channels of u (y), and the LPR mode groups of a row are combined with a
// butterfly over lanes CW apart.  Inputs are prefetched kPf steps ahead; the
// main loop carries no bounds checks (the channel index is clamped for lanes
// past D, whose results are discarded), a short tail loop finishes the chunk.
#include <algorithm>

#include "lh_internal.hpp"

namespace lh {
namespace {

constexpr int kBlock = 256;
constexpr int kWavesPerBlock = kBlock / 64;
constexpr int kPf = 16;  // prefetch depth (time steps)

// ---------------------------------------------------------------- pow kernel
__global__ __launch_bounds__(kBlock) void pow_kernel(const float2* __restrict__ lam,
                                                     float2* __restrict__ lamC, int64_t n,
                                                     int64_t C)
{
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    if (i >= n) return;
    // binary exponentiation in float64: lambda^C with a relative error of a
    // few float64 ulps, rounded once to complex64
    double br = lam[i].x, bi = lam[i].y;
    double pr = 1.0, pi = 0.0;
    for (int64_t e = C; e > 0; e >>= 1) {
        if (e & 1) {
            const double tr = pr * br - pi * bi;
            pi = pr * bi + pi * br;
            pr = tr;
        }
        const double sr = br * br - bi * bi;
        bi = 2.0 * br * bi;
        br = sr;
    }
    lamC[i] = make_float2(static_cast<float>(pr), static_cast<float>(pi));
}

// ------------------------------------------------------------ carry kernel
// One thread per (b, c, n); xs is [B, nchunks, D, d]: on entry slot k < nchunks-1
// holds s_k, on exit slot k holds x_in[k].
__global__ __launch_bounds__(kBlock) void carry_kernel(const float2* __restrict__ lamC,
                                                       float2* __restrict__ xs, int64_t B,
                                                       int64_t Dd, int64_t nchunks)
{
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    if (i >= B * Dd) return;
    const int64_t b = i / Dd;
    const int64_t e = i - b * Dd;  // c * d + n
    const float2 lc = lamC[e];
    float2* p = xs + b * nchunks * Dd + e;
    float xr = 0.f, xi = 0.f;
    for (int64_t k = 0; k < nchunks; ++k) {
        const float2 s = (k + 1 < nchunks) ? p[k * Dd] : make_float2(0.f, 0.f);
        p[k * Dd] = make_float2(xr, xi);
        const float nr = fmaf(lc.x, xr, fmaf(-lc.y, xi, s.x));
        const float ni = fmaf(lc.x, xi, fmaf(lc.y, xr, s.y));
        xr = nr;
        xi = ni;
    }
}

// ---------------------------------------------------------- zero-fill kernel
__global__ __launch_bounds__(kBlock) void zero_kernel(float2* __restrict__ p, int64_t n)
{
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    if (i < n) p[i] = make_float2(0.f, 0.f);
}

// ------------------------------------------------------- chunk scan kernel
// OUTPUT = false: state pass over chunks 0 .. nk-1 (nk = nchunks - 1), from 0,
//                 end state written to xs slot k.
// OUTPUT = true : output pass over chunks 0 .. nchunks-1, from xs slot k (or 0
//                 when nchunks == 1), writes y; the last chunk writes state.
template <int MPL, bool OUTPUT>
struct Modes {
    float lr[MPL], li[MPL], rr[MPL], ri[MPL], xr[MPL], xi[MPL];

    // Re(sum_n R_n x_n) over this lane's modes (two chains for ILP)
    __device__ __forceinline__ float re_rx() const {
        float a0 = 0.f, a1 = 0.f;
#pragma unroll
        for (int m = 0; m < MPL; ++m) {
            a0 = fmaf(rr[m], xr[m], a0);
            a1 = fmaf(ri[m], xi[m], a1);
        }
        return a0 - a1;
    }
    // x <- lambda x + u
    __device__ __forceinline__ void advance(float uv) {
#pragma unroll
        for (int m = 0; m < MPL; ++m) {
            const float nr = fmaf(lr[m], xr[m], fmaf(-li[m], xi[m], uv));
            const float ni = fmaf(lr[m], xi[m], li[m] * xr[m]);
            xr[m] = nr;
            xi[m] = ni;
        }
    }
};

template <typename IO, int LPR, int MPL, bool OUTPUT>
__global__ __launch_bounds__(kBlock) void chunk_scan_kernel(
    const float2* __restrict__ lam, const float2* __restrict__ R, const float* __restrict__ h0,
    const IO* __restrict__ u, IO* __restrict__ y, float2* __restrict__ state,
    float2* __restrict__ xs, int64_t B, int64_t D, int64_t d, int64_t T, int64_t C,
    int64_t nchunks, int64_t nk)
{
    constexpr int CW = 64 / LPR;  // channels per wave
    const int lane = threadIdx.x % 64;
    const int64_t wave = static_cast<int64_t>(blockIdx.x) * kWavesPerBlock + threadIdx.x / 64;
    const int64_t ncblk = (D + CW - 1) / CW;
    const int64_t nwaves = nk * B * ncblk;
    if (wave >= nwaves) return;  // whole wave exits together
    const int64_t cblk = wave % ncblk;
    const int64_t bk = wave / ncblk;
    const int64_t b = bk % B;
    const int64_t k = bk / B;

    const int64_t c = cblk * CW + (lane % CW);
    const bool valid = c < D;
    const int64_t cc = valid ? c : D - 1;  // all loads stay in bounds
    const int grp = lane / CW;
    const int64_t n0 = static_cast<int64_t>(grp) * MPL;
    const int64_t Dd = D * d;

    Modes<MPL, OUTPUT> md;
#pragma unroll
    for (int m = 0; m < MPL; ++m) {
        const int64_t n = n0 + m;
        const bool mv = n < d;
        const float2 l2 = mv ? lam[cc * d + n] : make_float2(0.f, 0.f);
        md.lr[m] = l2.x;
        md.li[m] = l2.y;
        md.rr[m] = md.ri[m] = md.xr[m] = md.xi[m] = 0.f;
        if constexpr (OUTPUT) {
            const float2 r2 = mv ? R[cc * d + n] : make_float2(0.f, 0.f);
            md.rr[m] = r2.x;
            md.ri[m] = r2.y;
            if (mv && nchunks > 1) {
                const float2 x2 = xs[(b * nchunks + k) * Dd + cc * d + n];
                md.xr[m] = x2.x;
                md.xi[m] = x2.y;
            }
        }
    }
    const float hz = OUTPUT ? h0[cc] : 0.f;

    const int64_t t0 = k * C;
    const int64_t n = ((t0 + C < T) ? t0 + C : T) - t0;  // steps of this chunk, wave-uniform
    const IO* up = u + (b * T + t0) * D + cc;
    IO* yp = y + (b * T + t0) * D + cc;

    auto one_step = [&](float uv, IO* yt) {
        if constexpr (OUTPUT) {
            float acc = md.re_rx();
#pragma unroll
            for (int off = CW; off < 64; off <<= 1) acc += __shfl_xor(acc, off, 64);
            // Every lane stores: lanes of one row hold bit-identical sums (the
            // butterfly adds commute at each level) and lanes past D repeat
            // channel D-1 exactly, so duplicate stores write the same value.
            io_store(yt, fmaf(hz, uv, acc));
        }
        md.advance(uv);
    };

    int64_t t = 0;
    if (n >= 2 * kPf) {
        // main loop: block t computed while block t + kPf is in flight
        float ub[kPf];
#pragma unroll
        for (int s = 0; s < kPf; ++s) ub[s] = io_load(up + s * D);
        for (; t + 2 * kPf <= n; t += kPf) {
            float un[kPf];
#pragma unroll
            for (int s = 0; s < kPf; ++s) un[s] = io_load(up + (kPf + s) * D);
#pragma unroll
            for (int s = 0; s < kPf; ++s) one_step(ub[s], yp + s * D);
#pragma unroll
            for (int s = 0; s < kPf; ++s) ub[s] = un[s];
            up += kPf * D;
            yp += kPf * D;
        }
        // block t is loaded (t + kPf <= n)
#pragma unroll
        for (int s = 0; s < kPf; ++s) one_step(ub[s], yp + s * D);
        t += kPf;
        up += kPf * D;
        yp += kPf * D;
    }
    for (; t < n; ++t) {  // tail (< 2 kPf steps)
        one_step(io_load(up), yp);
        up += D;
        yp += D;
    }

    // end state: s_k (state pass) or x_T (last chunk of the output pass)
    float2* dst = nullptr;
    if constexpr (OUTPUT) {
        if (k == nchunks - 1) dst = state + (b * D + cc) * d;
    } else {
        dst = xs + (b * nchunks + k) * Dd + cc * d;
    }
    if (dst != nullptr && valid) {
#pragma unroll
        for (int m = 0; m < MPL; ++m) {
            const int64_t nn = n0 + m;
            if (nn < d) dst[nn] = make_float2(md.xr[m], md.xi[m]);
        }
    }
}

template <typename IO, int LPR, int MPL, bool OUTPUT>
hipError_t launch_scan(const float2* lam, const float2* R, const float* h0, const void* u,
                       void* y, float2* state, float2* xs, int64_t B, int64_t D, int64_t d,
                       int64_t T, int64_t C, int64_t nchunks, int64_t nk, hipStream_t stream)
{
    constexpr int CW = 64 / LPR;
    const int64_t ncblk = (D + CW - 1) / CW;
    const int64_t nwaves = nk * B * ncblk;
    const int64_t grid = (nwaves + kWavesPerBlock - 1) / kWavesPerBlock;
    if (grid == 0) return hipSuccess;
    if (grid > 0x7fffffff) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((chunk_scan_kernel<IO, LPR, MPL, OUTPUT>),
                       dim3(static_cast<uint32_t>(grid)), dim3(kBlock), 0, stream, lam, R, h0,
                       static_cast<const IO*>(u), static_cast<IO*>(y), state, xs, B, D, d, T, C,
                       nchunks, nk);
    return hipGetLastError();
}

template <typename IO, bool OUTPUT>
hipError_t dispatch_scan(int lpr, int mpl, const float2* lam, const float2* R, const float* h0,
                         const void* u, void* y, float2* state, float2* xs, int64_t B,
                         int64_t D, int64_t d, int64_t T, int64_t C, int64_t nchunks,
                         int64_t nk, hipStream_t stream)
{
#define LH_SCAN(L, M)                                                                       \
    if (lpr == L && mpl == M)                                                               \
        return launch_scan<IO, L, M, OUTPUT>(lam, R, h0, u, y, state, xs, B, D, d, T, C,    \
                                             nchunks, nk, stream);
    // d <= 16: one lane per row, mpl = next power of two >= d
    LH_SCAN(1, 1)
    LH_SCAN(1, 2)
    LH_SCAN(1, 4)
    LH_SCAN(1, 8)
    LH_SCAN(1, 16)
    // d > 16: 16 modes per lane over lpr = ceil(d / 16) (power of two) lanes
    LH_SCAN(2, 16)
    LH_SCAN(4, 16)
    LH_SCAN(8, 16)
    LH_SCAN(16, 16)
    LH_SCAN(32, 16)
    LH_SCAN(64, 16)
#undef LH_SCAN
    return hipErrorInvalidValue;
}

// 1-D grid for n threads; false when it would exceed the grid limit
inline bool grid_for(int64_t n, dim3* g)
{
    const int64_t blocks = (n + kBlock - 1) / kBlock;
    if (blocks > 0x7fffffff) return false;
    *g = dim3(static_cast<uint32_t>(blocks));
    return true;
}

}  // namespace

namespace {

constexpr int64_t kMaxSegments = 64;

// The named plan of an automatic call at sizes that the explicit requests take.  It
// fixes the workspace, which callers hold, so the rule stays as it is whatever the
// kernel's tiling: the whole prompt where its (16 channels, 32 rows) tiles fill the
// GPU, or where it walks at most 7/5 of the chunks of 32 steps that the busiest CU
// walks in the two passes of the segmented plan, counted in workgroups of `cw`
// channels and 16 or 32 rows.
int named_auto(int64_t B, int64_t D, int64_t d, int64_t T, bool bf16_io, int64_t slots)
{
    if (d == 64 && B < 4 && B * T <= 1024) return 0;
    if ((D + 15) / 16 * ((B + 31) / 32) >= 256) return 1;
    if (slots >= 2) {
        auto walk = [&](int64_t rows, int64_t chunks, bool states_only) {
            const int64_t cw = d == 64 ? 4 : (d == 16 && bf16_io ? 16 : 8) * (states_only ? 2 : 1);
            const int64_t groups = d == 16 && !bf16_io && rows > 16 ? 2 : 1;
            const int64_t wgs = (D + cw - 1) / cw * ((rows + 16 * groups - 1) / (16 * groups));
            return (wgs + 255) / 256 * chunks * groups;
        };
        const int64_t chunks = T / slots / 32;
        const int64_t segmented =
            walk(B * (slots - 1), chunks, true) + walk(B * slots, chunks, false);
        return 5 * walk(B, (T + 31) / 32, false) <= 7 * segmented ? 1 : 2;
    }
    return d == 64 && (B >= 4 || (D + 3) / 4 * ((B + 15) / 16) >= 256) ? 1 : 0;
}

// Time of the VALU scan p in microseconds: launches, the steps (a wave's latency or
// the issue of all waves on a SIMD, per mode of a lane and halving of the lane
// sum), or the memory traffic; in one pass the steps outside the blocks of 16 and the
// scattered state as well, in chunks a carry that walks them.
double scan_us(int64_t B, int64_t D, int64_t d, int64_t T, bool bf16_io, const PrefillPlan& p)
{
    const int64_t cw = 64 / p.lpr, waves = B * ((D + cw - 1) / cw) * std::max<int64_t>(p.nchunks, 1);
    const double per_simd = double((waves + 1023) / 1024), lg = __builtin_ctz(p.lpr);
    const double mem = double(B) * double(T) * double(D) * (bf16_io ? 4 : 8);
    if (p.nchunks <= 1) {
        const double step = std::max(0.0016 + 0.0079 * p.mpl + 0.0627 * lg,
                                     per_simd * (0.0004 + 0.0081 * p.mpl + 0.0316 * lg));
        const double tail = double(T < 32 ? T : T % 16);
        return 7.1 + std::max(step * double(T) + 0.025 * tail, 0.117e-6 * mem) +
               0.64e-6 * 8 * double(B) * double(D) * double(d);
    }
    const double step = std::max(0.0216 * p.mpl + 0.0558 * lg,
                                 per_simd * (0.0092 + 0.0164 * p.mpl + 0.0385 * lg));
    return 11.9 + 0.27 * double(p.nchunks) + std::max(step * double(p.C), 0.261e-6 * mem);
}

// Whether sizes that no explicit request names run faster on the matrix cores
// than in the VALU scan p.  The constants of both estimates were fitted to the times
// of both at 360 shapes (B = 1..300, D = 64..4096, d = 1..64, T = 8..16384, both
// types; errors 13% and 14% root mean square); 3% go to the scan, which served these
// sizes first.  There the choice is more than 3% slower than the scan at 9 shapes
// (1.34x at most, of 15.7 us) and misses faster matrix cores at 24 (an earlier
// estimate: 25, up to 1.7x, and 18).
// Narrow banks on short prompts stay on the scan, also where the matrix cores are
// faster (B = 2, D = 70, d = 16, T = 300: 34 us against 12 us): the size of their
// workspace is the one that lh_prefill_workspace_bytes has always given.
bool mfma_faster(int64_t B, int64_t D, int64_t d, int64_t T, bool bf16_io, const PrefillPlan& p)
{
    if (D < 96 && B * T < 1024) return false;
    return mfma_us(B, D, d, T, bf16_io, p.cut) < 0.97 * scan_us(B, D, d, T, bf16_io, p);
}

}  // namespace

bool make_prefill_plan(int64_t B, int64_t D, int64_t d, int64_t T, int64_t request, int io,
                       PrefillPlan* plan)
{
    if (io < 0) {  // workspace for either input type
        // (a type with no plan for these sizes, such as bfloat16 under the
        // forced matrix-core plan at d = 64, adds nothing)
        PrefillPlan pf, pb;
        const bool f = make_prefill_plan(B, D, d, T, request, 0, &pf);
        const bool b = make_prefill_plan(B, D, d, T, request, 1, &pb);
        if (!f && !b) return false;
        *plan = f ? pf : pb;
        if (f && b && pb.ws_bytes > plan->ws_bytes) plan->ws_bytes = pb.ws_bytes;
        return true;
    }
    if (B < 1 || D < 1 || d < 1 || d > 1024 || T < 0 || request < -2) return false;
    // element counts must fit comfortably in int64 (and the byte sizes too)
    const int64_t lim = INT64_C(1) << 58;
    if (B > lim / D || B * D > lim / (T > d ? (T > 0 ? T : 1) : d)) return false;

    PrefillPlan p{};
    if (d <= 16) {
        p.lpr = 1;
        p.mpl = 1;
        while (p.mpl < d) p.mpl *= 2;
    } else {
        p.mpl = 16;
        p.lpr = 1;
        while (p.lpr * 16 < d) p.lpr *= 2;
    }
    if (T == 0) {
        p.C = 0;
        p.nchunks = 0;
    } else if (request > 0) {
        p.C = request < T ? request : T;
        p.nchunks = (T + p.C - 1) / p.C;
    } else {
        // Automatic: keep one sequential pass when the (b, c) rows alone give
        // at least 2 waves per SIMD (1024 SIMDs); otherwise cut time into
        // chunks so that about 4 waves per SIMD run, with chunks >= 64 steps.
        const int64_t cw = 64 / p.lpr;
        const int64_t waves = B * ((D + cw - 1) / cw);
        const int64_t kFull = 2048, kTarget = 4096;
        if (waves >= kFull) {
            p.C = T;
        } else {
            const int64_t want = (kTarget + waves - 1) / waves;
            int64_t C = (T + want - 1) / want;
            if (C < 64) C = 64;
            C = (C + 7) / 8 * 8;
            p.C = C < T ? C : T;
        }
        p.nchunks = (T + p.C - 1) / p.C;
    }
    p.off_pow = 0;
    p.off_xin = 0;
    const size_t pow_bytes = static_cast<size_t>(D) * d * sizeof(float2);
    p.off_xin = (pow_bytes + 255) / 256 * 256;
    p.scan_bytes = 0;
    if (p.nchunks > 1)
        p.scan_bytes = p.off_xin + static_cast<size_t>(B) * p.nchunks * D * d * sizeof(float2);
    p.ws_bytes = p.scan_bytes;

    // matrix cores
    p.forced = request == -1 || request == -2;
    const bool bf = io == 1;
    const bool supported = mfma_supported(B, D, d, T, bf);
    const int64_t slots = supported ? mfma_segments(B, D, d, T) : 0;
    if (p.forced && (!supported || (request == -2 && slots < 2))) return false;
    p.named = p.forced ? -static_cast<int>(request)
              : request == 0 && supported ? named_auto(B, D, d, T, bf, slots)
                                          : 0;
    const bool possible = mfma_possible(B, D, d, T, bf);
    if (p.named == 1) {
        p.mfma = possible;
        const size_t mb = mfma_workspace_bytes(D, d);
        if (p.forced || mb > p.ws_bytes) p.ws_bytes = mb;
        // an automatic call is cut into segments too where its workspace, sized
        // for the scan, has room for their states
        p.cut = mfma_cut(B, D, d, T, bf, p.forced ? 1 : slots);
        if (p.cut.nseg > 1) {
            const size_t off =
                (p.off_xin + static_cast<size_t>(B) * p.cut.nseg * D * d * sizeof(float2) + 255) /
                256 * 256;
            if (off + mfma_table_bytes(bf, true, D, d) <= p.ws_bytes)
                p.off_mfma = off;
            else
                p.cut = mfma_cut(B, D, d, T, bf, 1);
        }
    } else if (p.named == 2) {
        p.mfma = possible;
        p.cut = mfma_cut(B, D, d, T, bf, slots);
        const size_t xin_bytes = static_cast<size_t>(B) * slots * D * d * sizeof(float2);
        p.off_mfma = (p.off_xin + xin_bytes + 255) / 256 * 256;
        p.ws_bytes = p.off_mfma + mfma_workspace_bytes(D, d);
    } else if (request == 0 && possible) {
        // any other size: the same kernel where it is the faster one
        p.cut = mfma_cut(B, D, d, T, bf, kMaxSegments);
        if (mfma_faster(B, D, d, T, bf, p)) {
            p.mfma = true;
            size_t off = 0;
            if (p.cut.nseg > 1)
                off = (p.off_xin + static_cast<size_t>(B) * p.cut.nseg * D * d * sizeof(float2) + 255) /
                      256 * 256;
            p.off_mfma = off;
            p.ws_bytes = off + mfma_table_bytes(bf, false, D, d);
        }
    }
    if (!p.mfma && p.ws_bytes < p.scan_bytes) p.ws_bytes = p.scan_bytes;
    *plan = p;
    return true;
}

hipError_t launch_prefill(const float2* lam, const float2* R, const float* h0, const void* u,
                          bool bf16_io, int64_t B, int64_t D, int64_t d, int64_t T,
                          float2* state, void* y, const PrefillPlan& p, void* workspace,
                          hipStream_t stream)
{
    (void)hipGetLastError();  // clear a stale error so the status below is ours
    dim3 g_state, g_pow;
    if (!grid_for(B * D * d, &g_state) || !grid_for(D * d, &g_pow))
        return hipErrorInvalidConfiguration;
    if (T == 0) {
        hipLaunchKernelGGL(zero_kernel, g_state, dim3(kBlock), 0, stream, state, B * D * d);
        return hipGetLastError();
    }
    if (p.mfma) {
        char* ws = static_cast<char*>(workspace);
        float2* lamC = reinterpret_cast<float2*>(ws + p.off_pow);
        float2* xs = reinterpret_cast<float2*>(ws + p.off_xin);
        void* mws = ws + p.off_mfma;
        // The named plans take two terms where their outputs allow it; where the VALU
        // scan is what callers had (other sizes, unaligned u or y), three everywhere.
        MfmaCut cut = p.cut;
        cut.two_terms = p.named != 0 && (reinterpret_cast<uintptr_t>(u) |
                                         reinterpret_cast<uintptr_t>(y)) % 16 == 0;
        if (!cut.two_terms &&
            (cut.nseg > 1 ? p.off_mfma : 0) + mfma_table_bytes(bf16_io, false, D, d) > p.ws_bytes)
            cut = mfma_cut(B, D, d, T, bf16_io, 1);  // a named plan's segments left less room
        if (cut.nseg == 1) mws = ws;
        hipError_t e;
        if ((e = launch_mfma_setup(lam, R, h0, D, d, bf16_io, cut.two_terms, mws, stream)) != hipSuccess)
            return e;
        if (cut.nseg > 1) {
            hipLaunchKernelGGL(pow_kernel, g_pow, dim3(kBlock), 0, stream, lam, lamC, D * d,
                               cut.seg_len);
            if ((e = hipGetLastError()) != hipSuccess) return e;
            if ((e = launch_mfma_pass(false, lam, R, h0, u, bf16_io, B, D, d, T, cut, xs, state, y,
                                      mws, stream)) != hipSuccess)
                return e;
            hipLaunchKernelGGL(carry_kernel, g_state, dim3(kBlock), 0, stream, lamC, xs, B, D * d,
                               int64_t(cut.nseg));
            if ((e = hipGetLastError()) != hipSuccess) return e;
        }
        return launch_mfma_pass(true, lam, R, h0, u, bf16_io, B, D, d, T, cut, xs, state, y, mws, stream);
    }
    float2* lamC = nullptr;
    float2* xs = nullptr;
    hipError_t e;
    if (p.nchunks > 1) {
        lamC = reinterpret_cast<float2*>(static_cast<char*>(workspace) + p.off_pow);
        xs = reinterpret_cast<float2*>(static_cast<char*>(workspace) + p.off_xin);
        hipLaunchKernelGGL(pow_kernel, g_pow, dim3(kBlock), 0, stream, lam, lamC, D * d, p.C);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        e = bf16_io ? dispatch_scan<bf16, false>(p.lpr, p.mpl, lam, R, h0, u, y, state, xs, B, D,
                                                 d, T, p.C, p.nchunks, p.nchunks - 1, stream)
                    : dispatch_scan<float, false>(p.lpr, p.mpl, lam, R, h0, u, y, state, xs, B,
                                                  D, d, T, p.C, p.nchunks, p.nchunks - 1, stream);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(carry_kernel, g_state, dim3(kBlock), 0, stream, lamC, xs, B, D * d,
                           p.nchunks);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return bf16_io ? dispatch_scan<bf16, true>(p.lpr, p.mpl, lam, R, h0, u, y, state, xs, B, D, d,
                                               T, p.C, p.nchunks, p.nchunks, stream)
                   : dispatch_scan<float, true>(p.lpr, p.mpl, lam, R, h0, u, y, state, xs, B, D,
                                                d, T, p.C, p.nchunks, p.nchunks, stream);
}

}  // namespace lh
