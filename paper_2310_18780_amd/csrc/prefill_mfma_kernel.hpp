// The matrix-core prefill kernel and its tilings (see prefill_mfma.hip for the
// method, the tables and the choice of a tiling).  Included by one translation
// unit per input type, which instantiate the launchers declared at the end.
#pragma once

#include "lh_internal.hpp"
#include "prefill_mfma.hpp"

namespace lh {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

constexpr int kC = kMfmaChunk;  // steps per chunk
constexpr int kN = 16;          // MFMA columns
constexpr int kWaves = 8;       // per workgroup, two per SIMD
constexpr int kThreads = 64 * kWaves;
struct Yes { static constexpr bool value = true; };
struct No { static constexpr bool value = false; };

// nearest bfloat16 values of a pair (one packed conversion), and what they leave
__device__ __forceinline__ bf16x2 to_bf16x2(float a, float b)
{
    return __builtin_convertvector(f32x2{a, b}, bf16x2);
}

__device__ __forceinline__ f32x2 residual(float a, float b, bf16x2 h)
{
    const f32x2 back = __builtin_convertvector(h, f32x2);
    return f32x2{a - back.x, b - back.y};
}

__device__ __forceinline__ uint32_t bits(bf16x2 v) { return __builtin_bit_cast(uint32_t, v); }

__device__ __forceinline__ f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// a value that is the same in every lane, in scalar registers
__device__ __forceinline__ int64_t scalar64(int64_t v)
{
    const uint32_t lo = __builtin_amdgcn_readfirstlane(uint32_t(v));
    const uint32_t hi = __builtin_amdgcn_readfirstlane(uint32_t(uint64_t(v) >> 32));
    return int64_t(uint64_t(hi) << 32 | lo);
}

// Workgroup barrier that orders LDS only: waits for this wave's LDS accesses
// (lgkmcnt(0); vmcnt and expcnt left at their maximum in the s_waitcnt
// encoding) and leaves global accesses in flight, unlike __syncthreads(), whose
// fence also drains every outstanding global access.
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xc07f);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// A wave's LDS accesses execute in order, so values that its own lanes exchange
// through LDS need no barrier; this only keeps the compiler from moving the
// accesses across each other.
__device__ __forceinline__ void wave_order()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
    asm volatile("" ::: "memory");
}

__device__ __forceinline__ float2 cmul(float2 a, float2 b)
{
    return make_float2(fmaf(a.x, b.x, -a.y * b.y), fmaf(a.x, b.y, a.y * b.x));
}

__device__ __forceinline__ float2 add(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }

// B operand of W X_in: 8 state components as NT bfloat16 terms
template <int NT>
__device__ __forceinline__ void split8(const f32x4 a, const f32x4 b, bf16x8 (&out)[NT])
{
    float v[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int i = 0; i < 8; i += 2) {
            const bf16x2 h = to_bf16x2(v[i], v[i + 1]);
            out[t][i] = h.x;
            out[t][i + 1] = h.y;
            if (t + 1 < NT) {
                const f32x2 r = residual(v[i], v[i + 1], h);
                v[i] = r.x;
                v[i + 1] = r.y;
            }
        }
}

// S: time chunks per row among the 16 columns.  OUT = false is the state pass
// of the segmented plan (end states only).  X3: three terms of every float32 operand
// and entry state, else two where the outputs allow it.
template <typename IO, int DM, int S, bool OUT, bool X3>
__global__ __launch_bounds__(kThreads) void mfma_prefill_kernel(MfmaArgs p)
{
    using Cf = MfmaTiling<sizeof(IO) == 2, DM, X3>;
    constexpr bool BF = sizeof(IO) == 2;
    constexpr int ES = int(sizeof(IO));
    constexpr int CPW = Cf::kCpw, CW = Cf::kCw, NF = Cf::kFrags;
    constexpr int R = kN / S;                  // rows per workgroup
    constexpr int CPQ = 8 / ES;                // channels per 8-byte piece
    constexpr int PB = CW * ES;                // bytes of one (row, step)
    constexpr int PQ = PB / 8;                 // pieces per (row, step)
    constexpr int NITEM = R * (S * kC / 4) * PQ;  // (row, four steps, piece) items, at most one per thread
    static_assert(NITEM <= kThreads, "one item per thread");
    constexpr int NTU = BF ? 1 : 3;            // bfloat16 terms of u
    constexpr int NTW = BF && !X3 ? 2 : 3;     // of W
    constexpr int NTX = X3 ? 3 : 2;            // of the entry states
    constexpr int LPC = 16 * DM;               // modes per channel = scan lanes
    constexpr int RHX = 64 / (CPW * LPC) > 0 ? 64 / (CPW * LPC) : 1;
    constexpr int RH = RHX < R ? RHX : R;      // row groups of the scan
    constexpr int RL = R / RH;                 // rows per scan lane
    // LDS: u terms [term][channel][step / 8][column][step % 8], the columns of a
    // channel permuted by its piece (column ^ piece % 8); entry states and end
    // states [wave][channel][column][mode]; outputs [column][step][channel].  The
    // order of the first and the paddings of the others spread a wave's accesses
    // over the banks.
    constexpr int UCH = kN * kC;               // bfloat16 per (term, channel)
    constexpr int UB = NTU * CW * UCH;
    constexpr int XST = 2 * LPC + 4;           // floats per (channel, column)
    constexpr int YCOL = kC * PB + 8;          // bytes per column
    __shared__ __attribute__((aligned(16))) __bf16 ubuf[2][UB];
    constexpr bool kLocal = S == 1;            // a column is a row: its states stay in registers
    __shared__ __attribute__((aligned(16))) float xbuf[kWaves][kLocal ? 4 * CPW * LPC : CPW * kN * XST];
    __shared__ __attribute__((aligned(16))) unsigned char ybuf[2][OUT ? kN * YCOL : 16];
    __shared__ int lost_any;  // whether a state of the workgroup is not finite at its end

    // ---- workgroup -> (channel group, row group).  The CPL channel groups of a
    // 128-byte line of u and y form a line group; logical index (line group, row
    // group, member) is cut into eight contiguous ranges, one per XCD (workgroup
    // i runs on XCD i mod 8), so that an XCD's L2 holds its channels' tables
    // and the workgroups sharing lines run together.
    constexpr int CPL = 128 / PB > 1 ? 128 / PB : 1;
    const int lin = int(blockIdx.x % 8) * p.per_xcd + int(blockIdx.x / 8);
    const int rest = lin / CPL;
    const int lg = rest / p.nrg;
    const int cg = lg * CPL + (lin - rest * CPL);
    if (cg >= p.ncg) return;  // whole workgroup
    const int rg = rest - lg * p.nrg;
    const int D = p.D, d = p.d;
    // the last group is moved back into range: it then repeats channels of its
    // neighbour with the same operations, so both store the same values
    const int c0 = max(0, min(cg * CW, D - CW));
    // rows: batch rows, or (batch row b, segment k) pairs b * sv + k of the
    // segmented plan (R = 1); rows past the last repeat it
    const int sv = S == kN ? (OUT ? p.nseg : p.nseg - 1) : 1;
    const int nrow = p.B * sv;
    const int row0 = rg * R;
    const int seg = S == kN ? row0 % sv : 0;
    const int64_t TL =  // steps of the row(s)
        S == kN ? scalar64(min(p.seg_len, p.T - seg * p.seg_len)) : p.T;

    const int tid = threadIdx.x;
    const int w = tid / 64, lane = tid % 64;
    const int g = lane / 16, n = lane % 16;
    if (X3 && tid == 0) lost_any = 0;

    bf16x8 A[CPW][NF];
#pragma unroll
    for (int k = 0; k < CPW; ++k) {
        const bf16x8* src = static_cast<const bf16x8*>(p.frag) +
                            int64_t(min(c0 + w * CPW + k, D - 1)) * NF * 64 + lane;
#pragma unroll
        for (int f = 0; f < NF; ++f)
            if (OUT || (f >= Cf::kP && f < Cf::kW)) A[k][f] = src[f * 64];
    }

    // ---- scan lanes: lane -> (row group, channel, mode)
    const int sq = lane / LPC, sm = lane % LPC;
    const int sk = sq % CPW, srh = sq / CPW;
    const bool scan_on = srh < RH;
    const int sc = min(c0 + w * CPW + sk, D - 1);
    const float4 lp = static_cast<const float4*>(p.lamc)[int64_t(sc) * LPC + sm];
    // The rounding of lambda^C (lp.z, lp.w relative to it) is put right every kSteps
    // chunks, for the whole state as if all of it had taken kSteps products since: what
    // entered later is over-corrected, by at most kSteps roundings of lambda^C (2.4e-7
    // relative; with poles so fast that little older remains it shows, and every 16
    // chunks came to 1e-6).
    constexpr int kSteps = 4;
    constexpr int kCorrect = S >= kSteps ? 1 : kSteps / S;  // tiles between corrections
    const float2 ec = cmul(make_float2(kSteps * lp.z, kSteps * lp.w), make_float2(lp.x, lp.y));
    const float2 ec2 = cmul(ec, make_float2(lp.x, lp.y));
    float xr[RL], xi[RL];
#pragma unroll
    for (int r = 0; r < RL; ++r) {
        xr[r] = xi[r] = 0.f;
        if (OUT && S == kN && p.nseg > 1 && sm < d) {  // entry state of the segment
            const int64_t slot = int64_t(row0 / sv) * p.nseg + seg;
            const float2 v = p.xs[(slot * D + sc) * d + sm];
            xr[r] = v.x;
            xi[r] = v.y;
        }
    }

    // ---- this thread's item of a tile: 8 bytes of channels from cst on (moved
    // back into range like c0) at steps 4 qd .. 4 qd + 3 of row `irow`
    const bool has = NITEM == kThreads || tid < NITEM;
    const int it = has ? tid : 0;
    const int ip = it % PQ, qd = (it / PQ) % (S * kC / 4), irow = it / (PQ * (S * kC / 4));
    const int cst = min(c0 + ip * CPQ, D - CPQ);
    const int icol = irow * S + qd / (kC / 4), istep = 4 * (qd % (kC / 4));
    constexpr int TS = S * kC;  // steps per tile
    const int ntile = int((TL + TS - 1) / TS);
    // 32-bit offsets from the first row's start (of this segment)
    const int64_t base =
        scalar64((int64_t(row0 / sv) * p.T + (S == kN ? seg * p.seg_len : 0)) * D * ES);
    const char* const ubase = static_cast<const char*>(p.u) + base;
    char* const ybase = static_cast<char*>(p.y) + base;
    const uint32_t des = uint32_t(D) * ES;
    const uint32_t vrow =
        uint32_t(S == kN ? 0 : min(row0 + irow, nrow - 1) - row0) * uint32_t(p.T) * des + cst * ES;
    uint32_t vo[4];  // offsets of the item's steps
#pragma unroll
    for (int s = 0; s < 4; ++s) vo[s] = vrow + (4 * qd + s) * des;

    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    // A tile's place in u: start address and last valid offset of a row; steps
    // (and tiles) past the end repeat the last step.
    struct Place {
        const char* p;
        uint32_t lim;
    };
    auto place = [&](int tile) {
        const int64_t t = min(int64_t(tile) * TS, TL - 1);
        return Place{ubase + t * des, uint32_t(min((TL - 1 - t) * des, int64_t(0x7fffffff)))};
    };
    auto load = [&](const Place& at, int s) {
        u32x2 v;
        __builtin_memcpy(&v, at.p + min(vo[s], vrow + at.lim), 8);
        return v;
    };
    // a pair of steps (istep + 2 h, + 1) of the item
    auto stage_u = [&](u32x2 s0, u32x2 s1, int h, __bf16* ub) {
        if (!has) return;
        const int ch = cst - c0, step = istep + 2 * h;
        __bf16* dst = ub + ch * UCH + step / 8 * (kN * 8) + ((icol ^ (ch / CPQ & 7)) * 8) + step % 8;
#pragma unroll
        for (int j = 0; j < CPQ; ++j) {
            if constexpr (BF) {
                const uint32_t w0 = s0[j / 2], w1 = s1[j / 2];
                *reinterpret_cast<uint32_t*>(dst + j * UCH) =
                    j % 2 == 0 ? __builtin_amdgcn_perm(w1, w0, 0x05040100u)
                               : __builtin_amdgcn_perm(w1, w0, 0x07060302u);
            } else {
                f32x2 v = {__uint_as_float(s0[j]), __uint_as_float(s1[j])};
#pragma unroll
                for (int t = 0; t < 3; ++t) {
                    const bf16x2 hi = to_bf16x2(v.x, v.y);
                    *reinterpret_cast<uint32_t*>(dst + (t * CW + j) * UCH) = bits(hi);
                    if (t < 2) v = residual(v.x, v.y, hi);
                }
            }
        }
    };
    // outputs of a tile: the same items
    auto write_y = [&](int tile, const unsigned char* yb, bool last) {
        if (!has) return;
        const unsigned char* src = yb + icol * YCOL + istep * PB + (cst - c0) * ES;
        char* const dst = ybase + int64_t(tile) * TS * des;
#pragma unroll
        for (int s = 0; s < 4; ++s)
            if (!last || int64_t(tile) * TS + 4 * qd + s < TL) {
                const u32x2 v = *reinterpret_cast<const u32x2*>(src + s * PB);
                __builtin_memcpy(dst + vo[s], &v, 8);
            }
    };
    // u of a staged tile at step j of column col of channel k of this wave
    const int fch = w * CPW / CPQ & 7;
    auto u_at = [&](const __bf16* ub, int k, int col, int j) {
        const __bf16* src = ub + (w * CPW + k) * UCH + j / 8 * (kN * 8) + (col ^ fch) * 8 + j % 8;
        float v = static_cast<float>(src[0]);
        if constexpr (!BF)
            v += static_cast<float>(src[CW * UCH]) + static_cast<float>(src[2 * CW * UCH]);
        return v;
    };

    float* const xw = xbuf[w];
    // U operands of channel k: [term a | term b] of steps 8 (g % 2) ..
    struct Operands {
        bf16x8 u[NTU];
    };
    auto load_u = [&](int k, const __bf16* ub) {
        Operands o;
        const __bf16* src = ub + (w * CPW + k) * UCH + (g & 1) * (kN * 8) + (n ^ fch) * 8;
        o.u[0] = *reinterpret_cast<const bf16x8*>(src);
        if constexpr (!BF) {
            o.u[1] = *reinterpret_cast<const bf16x8*>(src + CW * UCH);
            o.u[2] = *reinterpret_cast<const bf16x8*>(src + (g < 2 ? 2 * CW * UCH : 0));
        }
        return o;
    };
    // Products with U, one instruction each, the smallest first, so that the sum is
    // rounded at its full size as few times as possible.  With float32 u
    // a1 u3 + a3 u1, (a1 + a2) u2, (a1 + a2) u1; with bfloat16 u [a3 | 0] u (of T only
    // with three terms) and [a1 | a2] u.
    constexpr int NPP = BF ? 2 : 3, NPT = BF && !X3 ? 1 : NPP;
    auto mul_u = [&](f32x4 acc, int k, int frag, const Operands& o, int i, int n) {
        const int j = n - 1 - i;  // 0: the largest
        return mfma(A[k][frag + (BF ? j : j < 2 ? 0 : 1)], o.u[BF ? 0 : j], acc);
    };
    auto mul_t = [&](f32x4 acc, int k, const Operands& o, int i) {
        return mul_u(acc, k, 0, o, i, NPT);
    };
    auto mul_p = [&](f32x4 acc, int k, int f, const Operands& o, int i) {
        return mul_u(acc, k, Cf::kP + 2 * f, o, i, NPP);
    };

    // ---- S = 1: the states of column n in the accumulator layout, X[k][f] holding
    // modes 8 f + 2 g and 8 f + 2 g + 1 of channel k as (re, im, re, im)
    // (their lambda^C and the correction of its rounding are read from LDS)
    f32x4 X[kLocal ? CPW : 1][2 * DM];
    float* const corr = xw;
    float* const lam_lds = xw + 2 * CPW * LPC;
    if constexpr (kLocal) {
#pragma unroll
        for (int k = 0; k < CPW; ++k) {
            const float4* src = static_cast<const float4*>(p.lamc) +
                                int64_t(min(c0 + w * CPW + k, D - 1)) * LPC;
#pragma unroll
            for (int f = 0; f < 2 * DM; ++f) {
                const int at = 2 * (k * LPC + 8 * f + 2 * g);
                const float4 a = src[8 * f + 2 * g], b = src[8 * f + 2 * g + 1];
                X[k][f] = f32x4{0.f, 0.f, 0.f, 0.f};
                if (n == 0) {
                    *reinterpret_cast<f32x4*>(corr + at) = f32x4{a.z, a.w, b.z, b.w};
                    *reinterpret_cast<f32x4*>(lam_lds + at) = f32x4{a.x, a.y, b.x, b.y};
                }
            }
        }
        wave_order();
    }
    auto lambda_c = [&](int k, int f) {
        return *reinterpret_cast<const f32x4*>(lam_lds + 2 * (k * LPC + 8 * f + 2 * g));
    };
    // (l.x + i l.y)(x.x + i x.y) and the same of the second mode
    auto mul_lambda = [](const f32x4 l, const f32x4 x) {
        return f32x4{fmaf(l[0], x[0], -l[1] * x[1]), fmaf(l[0], x[1], l[1] * x[0]),
                     fmaf(l[2], x[2], -l[3] * x[3]), fmaf(l[2], x[3], l[3] * x[2])};
    };

    auto store_tile_y = [&](const f32x4 (&Y)[CPW], unsigned char* yb) {
                    // row (step) 4 g + i of column n, this wave's CPW channels side by side
                    unsigned char* dst = yb + n * YCOL + 4 * g * PB + w * CPW * ES;
        #pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        if constexpr (BF && CPW == 4) {
                            *reinterpret_cast<uint2*>(dst + i * PB) = make_uint2(
                                bits(to_bf16x2(Y[0][i], Y[1][i])), bits(to_bf16x2(Y[2][i], Y[3][i])));
                        } else if constexpr (BF && CPW == 2) {
                            *reinterpret_cast<uint32_t*>(dst + i * PB) = bits(to_bf16x2(Y[0][i], Y[1][i]));
                        } else if constexpr (BF) {
                            io_store(reinterpret_cast<bf16*>(dst + i * PB), Y[0][i]);
                        } else if constexpr (CPW == 2) {
                            *reinterpret_cast<float2*>(dst + i * PB) = make_float2(Y[0][i], Y[1][i]);
                        } else {
                            *reinterpret_cast<float*>(dst + i * PB) = Y[0][i];
                        }
                    }
    };

    // Y = T U + W X_in of channel k, X_in given as the 2 DM accumulator tiles of P,
    // and with STEP those tiles advanced by a chunk.  Independent chains of
    // products are issued in turn, so that an instruction rarely waits for the
    // one before it.
    auto products = [&](int k, const Operands& o, f32x4 (&x)[2 * DM], auto step) {
        constexpr bool STEP = decltype(step)::value;
        // (W term, X term) pairs, the smallest first: all with i + j < 3 that both have,
        // but with bfloat16 u and y and two terms not (1, 1), lost in the rounding of
        // the outputs ([64, 4096, 2048] d = 16: 615 us with it, 583 us without; with
        // float32 the error of the outputs is 1.5 times as large without it)
        constexpr int kTa[6] = {0, 2, 1, 1, 0, 0};
        constexpr int kTb[6] = {2, 0, 1, 0, 1, 0};
        constexpr int kFirst = X3 ? 0 : BF ? 3 : 1, NW = 6 - kFirst;
        constexpr int NY = DM == 1 ? 1 : 2;  // chains of Y
        f32x4 y[NY] = {};
#pragma unroll
        for (int q = 0; q < DM; ++q) {
            bf16x8 xb[NTX];
            split8<NTX>(x[2 * q], x[2 * q + 1], xb);
            if constexpr (STEP)
#pragma unroll
                for (int f = 2 * q; f < 2 * q + 2; ++f) x[f] = mul_lambda(lambda_c(k, f), x[f]);
            constexpr int ROUNDS = NPT > NW ? NPT : NW;
#pragma unroll
            for (int i = 0; i < ROUNDS; ++i) {
                if (q == 0 && i < NPT) y[0] = mul_t(y[0], k, o, i);
                if (i < NW)
                    y[(q + 1) % NY] = mfma(A[k][Cf::kW + q * NTW + kTa[kFirst + i]],
                                           xb[kTb[kFirst + i]], y[(q + 1) % NY]);
                if (STEP && i < NPP)
#pragma unroll
                    for (int f = 2 * q; f < 2 * q + 2; ++f) x[f] = mul_p(x[f], k, f, o, i);
            }
        }
        if constexpr (NY == 2) y[0] += y[1];
        return y[0];
    };

    // The loads of a tile are issued over the tile before it in two pairs of steps,
    // so that about 8 to 16 KiB of them are in flight: the first pair is staged at
    // mid-tile, the second at its end, each three quarters of a tile after its
    // loads.
    u32x2 r[4];
    const int64_t nfull = TL / kC;         // whole chunks of a row
    const int tr = int(TL - nfull * kC);   // steps of the last, partial chunk
    const int nwhole = int(TL / TS);       // tiles without it
#pragma unroll
    for (int s = 0; s < 4; ++s) r[s] = load(place(0), s);
    stage_u(r[0], r[1], 0, ubuf[0]);
    stage_u(r[2], r[3], 1, ubuf[0]);
    Place next = place(1);  // of the tile being loaded
    r[0] = load(next, 0);
    r[1] = load(next, 1);
    lds_barrier();

    // quarter points of a tile; the scheduler keeps global accesses there
    auto quarter = [&](int tile, int q, auto first) {
        __builtin_amdgcn_sched_barrier(0x78f);
        if (q == 1) {
            r[2] = load(next, 2);
            r[3] = load(next, 3);
        } else if (q == 2) {
            stage_u(r[0], r[1], 0, ubuf[(tile + 1) & 1]);
            // the last tile's outputs, after the second pair's loads: the wait for
            // those, in issue order, leaves them in flight
            if constexpr (OUT && !decltype(first)::value)
                write_y(tile - 1, ybuf[(tile - 1) & 1], false);
        } else {
            next = place(tile + 2);
            r[0] = load(next, 0);
            r[1] = load(next, 1);
        }
        __builtin_amdgcn_sched_barrier(0x78f);
    };

    // S = 1: one tile; every state stays in its lane
    auto local_tile = [&](int tile, auto first, auto whole) {
        const __bf16* ub = ubuf[tile & 1];
        if constexpr (!decltype(first)::value)
            if (tile % kCorrect == 0) {  // lambda^C's rounding of the last tiles
#pragma unroll
                for (int k = 0; k < CPW; ++k)
#pragma unroll
                    for (int f = 0; f < 2 * DM; ++f) {
                        const f32x4 e =
                            *reinterpret_cast<const f32x4*>(corr + 2 * (k * LPC + 8 * f + 2 * g));
                        X[k][f] += float(kSteps) * mul_lambda(e, X[k][f]);
                    }
            }
        f32x4 Y[CPW];
#pragma unroll
        for (int k = 0; k < CPW; ++k) {
            if (CPW == 4 && k > 0) quarter(tile, k, first);
            if (CPW == 2 && k == 0) quarter(tile, 1, first);
            if (CPW == 2 && k == 1) {
                quarter(tile, 2, first);
                quarter(tile, 3, first);
            }
            if (CPW == 1) quarter(tile, 1, first);
            Y[k] = products(k, load_u(k, ub), X[k], whole);
            if (CPW == 1) quarter(tile, 2, first);
            if (CPW == 1) quarter(tile, 3, first);
        }
        if constexpr (!decltype(whole)::value) {  // the last, partial chunk step by step
#pragma unroll
            for (int k = 0; k < CPW; ++k) {
                const float2* l1 = p.lam + int64_t(min(c0 + w * CPW + k, D - 1)) * d;
                f32x4 l[2 * DM];  // all loads before the chain of steps
#pragma unroll
                for (int f = 0; f < 2 * DM; ++f) {
                    const int m0 = 8 * f + 2 * g;
                    const float2 a = m0 < d ? l1[m0] : make_float2(0.f, 0.f);
                    const float2 b = m0 + 1 < d ? l1[m0 + 1] : make_float2(0.f, 0.f);
                    l[f] = f32x4{a.x, a.y, b.x, b.y};
                }
                float uv = u_at(ub, k, n, 0);
                for (int j = 0; j < tr; ++j) {
                    const float un = u_at(ub, k, n, min(j + 1, kC - 1));
#pragma unroll
                    for (int f = 0; f < 2 * DM; ++f)
                        X[k][f] = mul_lambda(l[f], X[k][f]) + f32x4{uv, 0.f, uv, 0.f};
                    uv = un;
                }
            }
        }
        store_tile_y(Y, ybuf[tile & 1]);
    };

    // S > 1: one tile; end states to LDS, scan over the columns of each row,
    // entry states back
    auto scan_tile = [&](int tile, auto first, auto whole) {
        const __bf16* ub = ubuf[tile & 1];
#pragma unroll
        for (int k = 0; k < CPW; ++k) {
            const Operands o = load_u(k, ub);
            float* dst = xw + (k * kN + n) * XST + 4 * g;
#pragma unroll
            for (int f = 0; f < 2 * DM; ++f) {
                f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int i = 0; i < NPP; ++i) acc = mul_p(acc, k, f, o, i);
                *reinterpret_cast<f32x4*>(dst + 16 * f) = acc;
            }
        }
        quarter(tile, 1, first);
        wave_order();
        if (scan_on) {
            float2* xp = reinterpret_cast<float2*>(xw + (sk * kN + srh * RL * S) * XST) + sm;
            auto advance = [&](int r, float2 z) {
                const float nr = fmaf(lp.x, xr[r], fmaf(-lp.y, xi[r], z.x));
                xi[r] = fmaf(lp.x, xi[r], fmaf(lp.y, xr[r], z.y));
                xr[r] = nr;
            };
            auto due = [&](int s) {
                return s % kSteps == 0 && (s > 0 || (!decltype(first)::value && tile % kCorrect == 0));
            };
            if constexpr (decltype(whole)::value) {
                // the correction of the state before one column joins the sum of the next
                // one, as its smallest term (added to the state by itself it would cost a
                // rounding of it) and out of the chain of the walk, which a long walk waits
                // for; the short one has no registers for it
                constexpr bool kLate = S >= kSteps;
                float2 late[kLate ? RL : 1];
#pragma unroll
                for (int s = 0; s < S; ++s)
#pragma unroll
                    for (int r = 0; r < RL; ++r) {
                        float2* e = xp + (r * S + s) * (XST / 2);
                        float2 z = *e;
                        if constexpr (OUT) *e = make_float2(xr[r], xi[r]);
                        if constexpr (kLate) {
                            if (s > 0 && due(s - 1)) z = add(z, late[r]);
                            if (due(s)) late[r] = cmul(ec2, make_float2(xr[r], xi[r]));
                        } else if (due(s)) {
                            z = add(z, cmul(ec, make_float2(xr[r], xi[r])));
                        }
                        advance(r, z);
                    }
            } else {  // whole chunks, then the remaining steps one by one
                const float2 l1 = sm < d ? p.lam[int64_t(sc) * d + sm] : make_float2(0.f, 0.f);
                const int left = int(nfull - int64_t(tile) * S);
                for (int s = 0; s < left; ++s)
#pragma unroll
                    for (int r = 0; r < RL; ++r) {
                        float2* e = xp + (r * S + s) * (XST / 2);
                        float2 z = *e;
                        *e = make_float2(xr[r], xi[r]);
                        if (due(s)) z = add(z, cmul(ec, make_float2(xr[r], xi[r])));
                        advance(r, z);
                    }
#pragma unroll
                for (int r = 0; r < RL; ++r)
                    xp[(r * S + left) * (XST / 2)] = make_float2(xr[r], xi[r]);
                for (int j = 0; j < tr; ++j) {  // the rows of a lane side by side
                    float uv[RL];
#pragma unroll
                    for (int r = 0; r < RL; ++r) uv[r] = u_at(ub, sk, (srh * RL + r) * S + left, j);
#pragma unroll
                    for (int r = 0; r < RL; ++r) {
                        const float nr = fmaf(l1.x, xr[r], fmaf(-l1.y, xi[r], uv[r]));
                        xi[r] = fmaf(l1.x, xi[r], l1.y * xr[r]);
                        xr[r] = nr;
                    }
                }
            }
        }
        wave_order();
        quarter(tile, 2, first);
        if (!OUT || CPW == 1) quarter(tile, 3, first);
        if constexpr (OUT) {
            f32x4 Y[CPW];
#pragma unroll
            for (int k = 0; k < CPW; ++k) {
                if (CPW > 1 && k == CPW / 2) quarter(tile, 3, first);
                const float* src = xw + (k * kN + n) * XST + 4 * g;
                f32x4 xin[2 * DM];
#pragma unroll
                for (int f = 0; f < 2 * DM; ++f)
                    xin[f] = *reinterpret_cast<const f32x4*>(src + 16 * f);
                Y[k] = products(k, load_u(k, ub), xin, No{});
            }
            store_tile_y(Y, ybuf[tile & 1]);
        }
    };
    auto any_tile = [&](int tile, auto first, auto whole) {
        if constexpr (kLocal)
            local_tile(tile, first, whole);
        else
            scan_tile(tile, first, whole);
        __builtin_amdgcn_sched_barrier(0x78f);
        stage_u(r[2], r[3], 1, ubuf[(tile + 1) & 1]);
        lds_barrier();
    };

    // The first tile (no outputs to store yet) and a last, partial one are peeled
    // off, so that the loop holds no other path.
    if (nwhole > 0) {
        any_tile(0, Yes{}, Yes{});
        for (int tile = 1; tile < nwhole; ++tile) any_tile(tile, No{}, Yes{});
        if (ntile > nwhole) any_tile(nwhole, No{}, No{});
    } else {
        any_tile(0, Yes{}, No{});
    }
    if constexpr (OUT) write_y(ntile - 1, ybuf[(ntile - 1) & 1], true);

    // ---- x_T (of the last segment), or the end state of the segment, and the (row,
    // channel) pairs whose state is not finite: bit row * CPW + channel of the wave
    uint64_t lost = 0;
    if constexpr (kLocal) {
#pragma unroll
        for (int k = 0; k < CPW; ++k) {
            const int c = c0 + w * CPW + k, row = row0 + n;
            const bool on = c < D && row < nrow;
            float2* dst = p.state + (int64_t(row) * D + c) * d;
            float z = 0.f;  // not zero after a value that is not finite
#pragma unroll
            for (int f = 0; f < 2 * DM; ++f)
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    if (on && 8 * f + 2 * g + h < d) {
                        const float2 v = make_float2(X[k][f][2 * h], X[k][f][2 * h + 1]);
                        dst[8 * f + 2 * g + h] = v;
                        if constexpr (X3) z += 0.f * v.x + 0.f * v.y;
                    }
            if constexpr (X3) {
                uint64_t bad = __ballot(z != 0.f);
                bad = (bad | bad >> 16 | bad >> 32 | bad >> 48) & 0xffff;
                for (int r = 0; bad != 0 && r < R; ++r) lost |= (bad >> r & 1) << (r * CPW + k);
            }
        }
    } else {
        const bool on = scan_on && sm < d && w * CPW + sk < D;
#pragma unroll
        for (int r = 0; r < RL; ++r) {
            const int row = row0 + srh * RL + r;
            if constexpr (X3) {
                const float z = 0.f * xr[r] + 0.f * xi[r];
                const uint64_t bad = __ballot(on && row < nrow && z != 0.f);
                for (int q = 0; bad != 0 && q < RH * CPW; ++q)
                    if ((bad >> (q * LPC) & (~UINT64_C(0) >> (64 - LPC))) != 0)
                        lost |= UINT64_C(1) << ((q / CPW * RL + r) * CPW + q % CPW);
            }
            if (!on || row >= nrow || (OUT && seg != sv - 1)) continue;
            float2* dst = OUT ? p.state + (int64_t(row / sv) * D + sc) * d
                              : p.xs + ((int64_t(row / sv) * p.nseg + seg) * D + sc) * d;
            dst[sm] = make_float2(xr[r], xi[r]);
        }
    }

    // ---- A product multiplies every input of its chunk, also by zeros, so an input
    // that is not finite (or that its nearest bfloat16 is not) spoils outputs before
    // it, and leaves a state that is not finite for good.  Such a row and channel is
    // stepped again from its start, one lane per mode, once all stores of the
    // workgroup to it are out (write_y spreads a row over the waves); the others keep
    // their results.  Not in the two-term kernels, whose plans always lost the outputs
    // of the chunk (and where this code costs 1-4% of the time, through the registers).
    if constexpr (!X3) return;
    if (lane == 0 && lost != 0) lost_any = 1;
    lds_barrier();
    if (lost_any == 0) return;
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    constexpr int NG = 64 / LPC;  // pairs at a time
    const int q = lane / LPC, m = lane % LPC;
    for (int p0 = 0; p0 < R * CPW; p0 += NG) {
        const uint64_t these = lost >> p0 & (~UINT64_C(0) >> (64 - NG));
        if (these == 0) continue;
        const bool on = q < NG && (these >> q & 1) != 0;
        const int pair = on ? p0 + q : 0, row = min(row0 + pair / CPW, nrow - 1);
        const int c = min(c0 + w * CPW + pair % CPW, D - 1);
        const bool mode = on && m < d;
        const float2 l1 = mode ? p.lam[int64_t(c) * d + m] : make_float2(0.f, 0.f);
        const float2 r1 = mode ? p.R[int64_t(c) * d + m] : make_float2(0.f, 0.f);
        const float h1 = p.h0[c];
        const int64_t at = (int64_t(row / sv) * p.nseg + seg) * D + c;  // of segment states
        float2 x = make_float2(0.f, 0.f);
        if (OUT && S == kN && p.nseg > 1 && mode) x = p.xs[at * d + m];
        const int64_t first = (int64_t(row / sv) * p.T + (S == kN ? seg * p.seg_len : 0)) * D + c;
        for (int64_t t0 = 0; t0 < TL; t0 += LPC) {
            const int cnt = int(min(int64_t(LPC), TL - t0));
            const int64_t mine = first + (t0 + min(m, cnt - 1)) * D;
            const float ub = io_load(static_cast<const IO*>(p.u) + mine);
            float yb = 0.f;
            for (int j = 0; j < cnt; ++j) {
                const float uv = __shfl(ub, q * LPC + j, 64);
                if constexpr (OUT) {
                    float v = mode ? fmaf(r1.x, x.x, -r1.y * x.y) : 0.f;
                    for (int o = 1; o < (LPC == 48 ? 64 : LPC); o *= 2) v += __shfl_xor(v, o, 64);
                    if (m == j) yb = fmaf(h1, uv, v);
                }
                x = make_float2(fmaf(l1.x, x.x, fmaf(-l1.y, x.y, uv)), fmaf(l1.x, x.y, l1.y * x.x));
            }
            if (OUT && on && m < cnt) io_store(static_cast<IO*>(p.y) + mine, yb);
        }
        if (!mode) continue;
        if constexpr (!OUT)
            p.xs[at * d + m] = x;
        else if (seg == sv - 1)
            p.state[(int64_t(row / sv) * D + c) * d + m] = x;
    }
}

template <typename IO, int DM, int S, bool OUT, bool X3>
hipError_t launch_tiled(MfmaArgs a, hipStream_t stream)
{
    using Cf = MfmaTiling<sizeof(IO) == 2, DM, X3>;
    constexpr int PB = Cf::kCw * int(sizeof(IO)), CPL = 128 / PB > 1 ? 128 / PB : 1, R = kN / S;
    const int64_t rows = int64_t(a.B) * (S == kN ? (OUT ? a.nseg : a.nseg - 1) : 1);
    const int64_t ncg = (int64_t(a.D) + Cf::kCw - 1) / Cf::kCw, nrg = (rows + R - 1) / R;
    const int64_t per_xcd = ((ncg + CPL - 1) / CPL * CPL * nrg + 7) / 8;
    if (8 * per_xcd > 0x7fffffff || rows > 0x7fffffff) return hipErrorInvalidConfiguration;
    a.ncg = int(ncg);
    a.nrg = int(nrg);
    a.per_xcd = int(per_xcd);
    hipLaunchKernelGGL((mfma_prefill_kernel<IO, DM, S, OUT, X3>), dim3(uint32_t(8 * per_xcd)),
                       dim3(kThreads), 0, stream, a);
    return hipGetLastError();
}

template <typename IO, int DM, bool X3>
hipError_t launch_s(int s, bool outputs, const MfmaArgs& a, hipStream_t stream)
{
    if (!outputs) return launch_tiled<IO, DM, 16, false, X3>(a, stream);
    switch (s) {
        case 1: return launch_tiled<IO, DM, 1, true, X3>(a, stream);
        case 2: return launch_tiled<IO, DM, 2, true, X3>(a, stream);
        case 4: return launch_tiled<IO, DM, 4, true, X3>(a, stream);
        case 16: return launch_tiled<IO, DM, 16, true, X3>(a, stream);
        default: return hipErrorInvalidValue;
    }
}

template <typename IO, int DM>
hipError_t launch_dm(int s, bool outputs, const MfmaArgs& a, hipStream_t stream)
{
    if (!a.two_terms) return launch_s<IO, DM, true>(s, outputs, a, stream);
    // the orders of the explicit plans
    if constexpr (DM <= 2 || (DM == 4 && sizeof(IO) == 4))
        if (a.d == 16 * DM) return launch_s<IO, DM, false>(s, outputs, a, stream);
    return hipErrorInvalidValue;
}

template <typename IO>
hipError_t launch_io(int dm, int s, bool outputs, const MfmaArgs& a, hipStream_t stream)
{
    switch (dm) {
        case 1: return launch_dm<IO, 1>(s, outputs, a, stream);
        case 2: return launch_dm<IO, 2>(s, outputs, a, stream);
        case 3: return launch_dm<IO, 3>(s, outputs, a, stream);
        case 4: return launch_dm<IO, 4>(s, outputs, a, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace
}  // namespace lh
