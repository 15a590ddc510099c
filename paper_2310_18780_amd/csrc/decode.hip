// Decode step of the distilled modal recurrence (Proposition
// "modal_realization", Sec. 3.4; real output as in App. B.1):
//
//   y[b,c]       = Re(sum_n R[c,n] x[b,c,n]) + h0[c] u[b,c]
//   x[b,c,n]    <- lambda[c,n] x[b,c,n] + u[b,c]          (in place)
//
// One pass over the [B, D, d] complex64 state: read once, written once, so the
// kernel is bound by memory bandwidth (16 bytes of state traffic per mode
// against 12 flops).
//
// Lanes path (d even up to 128 in 16-byte aligned arrays, else d up to 64): the
// modes of a (b, c) row sit two (one) to a lane on LPR consecutive lanes, LPR the
// power of two that holds them, one 16-byte (8-byte) access each; lanes past d hold
// zeros, so any order reads and writes contiguous spans of the state.  (Against the
// loop over strided modes, one row per thread, that served orders other than powers
// of two, per token of a stack of banks replayed from a graph: B = 37, D = 1001, d =
// 10, 8 banks 48.6 -> 37.0 us; B = 1, D = 4077, d = 60, 15 banks 180 -> 59 us; B =
// 231, D = 704, d = 37, 6 banks 306 -> 175 us.)  The row sum is a butterfly over
// those lanes (DPP within 16 lanes).  Each thread serves NB batch rows of the same (c,
// modes): lambda and R are loaded once for the NB rows, and every thread has NB
// independent state loads in flight before it computes.  NB = 8
// where that still gives 2048 wavefronts (two per SIMD), else 4 where that
// does, else 2: small states are latency-bound, and more wavefronts with
// fewer rows each finish sooner (B = 16, D = 768, d = 16: 1.95 us per step
// with NB = 2 against 2.51 us with NB = 8; B = 64, D = 2048: 6.0 us with
// NB = 8 against 6.3 us with NB = 4).  NB = 1 where pairs of rows leave fewer than 512
// wavefronts (B = 4, D = 512, d = 24: 2.50 us against 2.73 us; at 512, B = 4, D = 1024, d =
// 32: 2.65 against 2.56 us), with LPR >= 32 not more than 512 (B = 4, D = 512, d = 17: 2.40
// us against 2.69 us), and for a single row, and no larger NB than the rows need (B = 2, D = 4096, d = 33: 3.85 us with 2,
// 5.23 us with 8, six of them idle).  Up to 32 single modes (8-byte accesses) take at most
// 2 rows while the state is small (kFewRowsBytes; B = 64, D = 2048, d = 5: 5.51 us
// against 5.90 us with 8; d = 9, 9.4 MB: 8.71 and 7.52 us).  A workgroup is one wavefront
// (64 / LPR channels x NB batch rows) up to LPR = 16; with LPR >= 32 (two
// channels or fewer per wavefront) it is four wavefronts, so that
// a workgroup covers 8 channels (B = 256, D = 2048, d = 64: 71 us per step
// against 76 us with one-wavefront workgroups).
//
// Cache policy: the state is written with the non-temporal hint, and read
// with it when the whole state fits the L2s with room to spare (at most
// kStreamStateBytes, 16 MiB: half of the 8 XCDs' 4 MB L2s).  An in-place
// pass that reads its lines with ordinary loads leaves them in the caches to
// be written back later; a state streaming from HBM (as the states of a
// model's layers together do) then runs about a quarter slower than a copy
// of the same bytes, and with non-temporal loads at the copy's rate.  A
// state that fits the L2s and is stepped again right away stays there either
// way (16 MiB: within 1%).  A larger state stepped again right away keeps
// part of itself in the 256 MB Infinity Cache only when read with ordinary
// loads (32 MiB: 11.0 us per step against 11.8 us; 256 MiB: 76 us against
// 87 us), so those take ordinary loads.  y_t is stored with ordinary stores:
// its 16-byte pieces per wavefront and batch row are merged into whole lines
// in the L2 before they reach HBM.
//
// Workgroups are ordered so that XCD x (workgroup i runs on XCD i mod 8)
// owns one contiguous range of channel tiles: its lambda / R rows, its slice
// of every batch row of the state, and whole 128-byte lines of u_t and y_t
// stay with one L2.
//
// Generic path (larger d, a grid past its limits, or 1 < d <= 16 in single modes on a
// state of at most kStridedBytes): lanes take single modes j, j + LPR, ... (LPR = next
// power of two >= d, <= 64) or pairs, one batch row per thread.  Its four-wavefront
// workgroups step such small states in 0.8-0.95 of the lanes path's time, layers
// replayed from a graph (B = 128, D = 512: d = 5 3.68 us against 4.65 us, d = 7 3.82
// against 4.74; B = 32, D = 1024, d = 15, 3.9 MB: 3.87 against 4.82); from about 4.5 MB
// on the lanes path with two rows per thread is level or faster (B = 128, D = 512, d =
// 9, 4.7 MB: 5.43 us against 5.52 us).
#include "lh_internal.hpp"

namespace lh {
namespace {

constexpr int kBlock = 256;  // generic path

// lanes path: threads per workgroup for LPR lanes per row
constexpr int pairs_block(int lpr) { return lpr >= 32 ? 256 : 64; }
constexpr int kXcds = 8;
constexpr int kMaxRowsPerThread = 8;
constexpr int64_t kMinWaves = 2048;  // wavefronts the row count per thread is chosen for
constexpr int64_t kStreamStateBytes = INT64_C(16) << 20;  // non-temporal state loads up to this size
constexpr int64_t kFewRowsBytes = INT64_C(8) << 20;  // single modes, d <= 32: at most two rows per thread up to this size
constexpr int64_t kStridedBytes = INT64_C(4) << 20;  // single modes, 1 < d <= 16: the generic path up to this size

typedef float f4v __attribute__((ext_vector_type(4)));

// 16-byte accesses.  NT is a template argument, not a run-time flag: with a
// flag, both branches would store the same value to the same address and the
// compiler merges them into one plain access before the flag is known,
// dropping the non-temporal hint.
template <bool NT>
__device__ __forceinline__ float4 load4(const float2* p)
{
    const f4v* q = reinterpret_cast<const f4v*>(p);
    f4v v;
    if constexpr (NT)
        v = __builtin_nontemporal_load(q);
    else
        v = *q;
    return make_float4(v.x, v.y, v.z, v.w);
}

template <bool NT>
__device__ __forceinline__ void store4(float2* p, float4 a)
{
    f4v* q = reinterpret_cast<f4v*>(p);
    const f4v v = {a.x, a.y, a.z, a.w};
    if constexpr (NT)
        __builtin_nontemporal_store(v, q);
    else
        *q = v;
}

// Butterfly step of a row sum over LPR lanes: after the steps for offsets
// 1 .. off/2 every aligned group of `off` lanes holds one partial sum, so any
// lane permutation that pairs each group with its neighbour group completes
// the step.  Within a row of 16 lanes this is DPP on the VALU (quad_perm for
// 1 and 2, half-row mirror for 4, row mirror for 8); wider steps use a shuffle.
template <int OFF>
__device__ __forceinline__ float butterfly(float v)
{
    const int x = __builtin_bit_cast(int, v);
    int p;
    if constexpr (OFF == 1)
        p = __builtin_amdgcn_mov_dpp(x, 0xB1, 0xF, 0xF, false);   // quad_perm [1,0,3,2]
    else if constexpr (OFF == 2)
        p = __builtin_amdgcn_mov_dpp(x, 0x4E, 0xF, 0xF, false);   // quad_perm [2,3,0,1]
    else if constexpr (OFF == 4)
        p = __builtin_amdgcn_mov_dpp(x, 0x141, 0xF, 0xF, false);  // row_half_mirror
    else if constexpr (OFF == 8)
        p = __builtin_amdgcn_mov_dpp(x, 0x140, 0xF, 0xF, false);  // row_mirror
    else
        return v + __shfl_xor(v, OFF, 64);
    return v + __builtin_bit_cast(float, p);
}

template <int LPR>
__device__ __forceinline__ float row_sum(float v)
{
    if constexpr (LPR >= 2) v = butterfly<1>(v);
    if constexpr (LPR >= 4) v = butterfly<2>(v);
    if constexpr (LPR >= 8) v = butterfly<4>(v);
    if constexpr (LPR >= 16) v = butterfly<8>(v);
    if constexpr (LPR >= 32) v = butterfly<16>(v);
    if constexpr (LPR >= 64) v = butterfly<32>(v);
    return v;
}

// complex multiply-add of two modes held as (re0, im0, re1, im1)
__device__ __forceinline__ float4 step_pair(float4 l, float4 x, float uv)
{
    float4 n;
    n.x = fmaf(l.x, x.x, fmaf(-l.y, x.y, uv));
    n.y = fmaf(l.x, x.y, l.y * x.x);
    n.z = fmaf(l.z, x.z, fmaf(-l.w, x.w, uv));
    n.w = fmaf(l.z, x.w, l.w * x.z);
    return n;
}

__device__ __forceinline__ float re_dot_pair(float4 r, float4 x)
{
    return fmaf(r.x, x.x, fmaf(-r.y, x.y, fmaf(r.z, x.z, -r.w * x.w)));
}

// The modes that a lane holds: two (16 bytes) or one (8 bytes, as a float4 whose
// second half is zero and drops out of the compiled code).
template <int VEC, bool NT>
__device__ __forceinline__ float4 load_modes(const float2* p)
{
    if constexpr (VEC == 2) {
        return load4<NT>(p);
    } else {
        typedef float f2v __attribute__((ext_vector_type(2)));
        const f2v* q = reinterpret_cast<const f2v*>(p);
        f2v v;
        if constexpr (NT)
            v = __builtin_nontemporal_load(q);
        else
            v = *q;
        return make_float4(v.x, v.y, 0.f, 0.f);
    }
}

template <int VEC>
__device__ __forceinline__ void store_modes(float2* p, float4 a)
{
    if constexpr (VEC == 2) {
        store4<true>(p, a);
    } else {
        typedef float f2v __attribute__((ext_vector_type(2)));
        __builtin_nontemporal_store(f2v{a.x, a.y}, reinterpret_cast<f2v*>(p));
    }
}

// Lanes path: LPR lanes per row of VEC modes each, NB rows per thread, 2-D grid of
// (channel tile, batch group) workgroups.  FULL: d == VEC LPR; else lanes past d
// hold zeros and touch no memory.  gridDim.x is the tile count padded to a multiple
// of 8; workgroup x runs on XCD x % 8, which owns tiles [(x % 8) T8, (x % 8 + 1) T8)
// with T8 = gridDim.x / 8.  NTL: non-temporal state loads.
template <typename IO, int LPR, int VEC, bool FULL, bool NTL, int NB>
__global__ __launch_bounds__(pairs_block(LPR)) void step_lanes_kernel(
    const float2* __restrict__ lam, const float2* __restrict__ R, const float* __restrict__ h0,
    float2* __restrict__ state, const IO* __restrict__ u, IO* __restrict__ y, int B, int D, int dr,
    int ntiles)
{
    constexpr int kRows = pairs_block(LPR) / LPR;  // channels per workgroup
    const int d = FULL ? VEC * LPR : dr;
    const int ct = int(blockIdx.x % kXcds) * int(gridDim.x / kXcds) + int(blockIdx.x / kXcds);
    const int b0 = blockIdx.y * NB;
    if (ct >= ntiles) return;  // padding tiles
    const int j = threadIdx.x % LPR;
    const int c = ct * kRows + threadIdx.x / LPR;
    const bool cvalid = c < D;
    const int cc = cvalid ? c : D - 1;  // every address stays in bounds
    const bool on = FULL || VEC * j < d;  // d is a multiple of VEC

    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    const int64_t at = int64_t(cc) * d + VEC * j;
    const float4 l4 = on ? load_modes<VEC, false>(lam + at) : zero;
    const float4 r4 = on ? load_modes<VEC, false>(R + at) : zero;
    float4 x[NB];
    float uv[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int b = (b0 + i < B) ? b0 + i : B - 1;
        const int64_t row = int64_t(b) * D + cc;
        x[i] = on ? load_modes<VEC, NTL>(state + row * d + VEC * j) : zero;
        uv[i] = io_load(u + row);
    }
    const float hz = h0[cc];
    // a use of every u value here keeps all the loads above issued together:
    // left alone, the compiler sinks the first row's u load into its
    // conditional store block, where it is issued only after the first wait
#pragma unroll
    for (int i = 0; i < NB; ++i) asm volatile("" ::"v"(uv[i]));
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int b = b0 + i;
        const float acc = row_sum<LPR>(re_dot_pair(r4, x[i]));
        const float4 n4 = step_pair(l4, x[i], uv[i]);
        if (cvalid && b < B) {
            const int64_t row = int64_t(b) * D + c;
            if (on) store_modes<VEC>(state + row * d + VEC * j, n4);
            if (j == 0) io_store(y + row, fmaf(hz, uv[i], acc));
        }
    }
}

// Generic path.  VEC = 2: each lane owns pairs m = 2 (j + i LPR), requires
// d % (2 LPR) == 0 and 16-byte alignment; VEC = 1: modes j, j + LPR, ...
template <typename IO, int LPR, int VEC>
__global__ __launch_bounds__(kBlock) void step_generic_kernel(
    const float2* __restrict__ lam, const float2* __restrict__ R, const float* __restrict__ h0,
    float2* __restrict__ state, const IO* __restrict__ u, IO* __restrict__ y, int64_t B,
    int64_t D, int64_t d, int64_t nblocks)
{
    constexpr int kRows = kBlock / LPR;
    const int64_t lb = blockIdx.x;
    if (lb >= nblocks) return;
    const int64_t ct = lb / B;
    const int64_t b = lb - ct * B;
    const int j = threadIdx.x % LPR;
    const int64_t c = ct * kRows + threadIdx.x / LPR;
    const bool valid = c < D;
    const int64_t cc = valid ? c : D - 1;

    const float uv = io_load(u + b * D + cc);
    const float2* lrow = lam + cc * d;
    const float2* rrow = R + cc * d;
    float2* xrow = state + (b * D + cc) * d;
    float acc = 0.f;
    if constexpr (VEC == 2) {
        const int64_t ni = d / (2 * LPR);
        for (int64_t i = 0; i < ni; ++i) {
            const int64_t m = 2 * (j + i * LPR);
            const float4 x4 = load4<false>(xrow + m);
            acc += re_dot_pair(load4<false>(rrow + m), x4);
            const float4 n4 = step_pair(load4<false>(lrow + m), x4, uv);
            if (valid) store4<false>(xrow + m, n4);
        }
    } else {
        for (int64_t m = j; m < d; m += LPR) {
            const float2 l2 = lrow[m];
            const float2 r2 = rrow[m];
            const float2 x2 = xrow[m];
            acc = fmaf(r2.x, x2.x, acc);
            acc = fmaf(-r2.y, x2.y, acc);
            float2 n2;
            n2.x = fmaf(l2.x, x2.x, fmaf(-l2.y, x2.y, uv));
            n2.y = fmaf(l2.x, x2.y, l2.y * x2.x);
            if (valid) xrow[m] = n2;
        }
    }
    acc = row_sum<LPR>(acc);
    if (valid && j == 0) io_store(y + b * D + c, fmaf(h0[c], uv, acc));
}

// Batch rows per thread of the lanes path (see the file comment).
int pairs_rows_per_thread(int lpr, int vec, int64_t B, int64_t D, int64_t d)
{
    const int64_t waves_per_group = (D * lpr + 63) / 64;
    auto waves = [&](int nb) { return (B + nb - 1) / nb * waves_per_group; };
    const int most = vec == 1 && d <= 32 && 8 * B * D * d <= kFewRowsBytes ? 2 : kMaxRowsPerThread;
    for (int nb = most; nb > 2; nb /= 2)
        if (nb / 2 < B && waves(nb) >= kMinWaves) return nb;
    return B > 1 && waves(2) >= kMinWaves / 4 + (lpr >= 32) ? 2 : 1;
}

// 2-D grid of the lanes path; false when it does not fit the grid limits
bool pairs_grid(int lpr, int nb, int64_t B, int64_t D, dim3* g, int* ntiles)
{
    const int64_t rows_per_block = pairs_block(lpr) / lpr;
    const int64_t nt = (D + rows_per_block - 1) / rows_per_block;
    const int64_t nbg = (B + nb - 1) / nb;
    const int64_t ntp = (nt + kXcds - 1) / kXcds * kXcds;
    if (ntp > 0x7fffffff || nbg > 65535) return false;
    *g = dim3(uint32_t(ntp), uint32_t(nbg));
    *ntiles = int(nt);
    return true;
}

// One call's sizes and pointers, for the nest of template choices below.
struct Step {
    const float2 *lam, *R;
    const float* h0;
    float2* state;
    const void* u;
    void* y;
    int B, D, d;
    dim3 grid;
    int ntiles;
    hipStream_t stream;
};

template <typename IO, int LPR, int VEC, bool FULL, bool NTL>
hipError_t launch_nb(int nb, const Step& s)
{
#define LH_NB(N)                                                                             \
    case N:                                                                                  \
        hipLaunchKernelGGL((step_lanes_kernel<IO, LPR, VEC, FULL, NTL, N>), s.grid,          \
                           dim3(pairs_block(LPR)), 0, s.stream, s.lam, s.R, s.h0, s.state,   \
                           static_cast<const IO*>(s.u), static_cast<IO*>(s.y), s.B, s.D, s.d, \
                           s.ntiles);                                                        \
        return hipGetLastError();
    switch (nb) {
        LH_NB(8)
        LH_NB(4)
        LH_NB(2)
        LH_NB(1)
        default: return hipErrorInvalidValue;
    }
#undef LH_NB
}

template <typename IO, int LPR, int VEC, bool FULL>
hipError_t launch_ntl(bool ntl, int nb, const Step& s)
{
    return ntl ? launch_nb<IO, LPR, VEC, FULL, true>(nb, s)
               : launch_nb<IO, LPR, VEC, FULL, false>(nb, s);
}

template <typename IO, int LPR>
hipError_t launch_vec(int vec, bool ntl, int nb, const Step& s)
{
    const bool full = s.d == vec * LPR;
    if (vec == 2) {
        if (full) return launch_ntl<IO, LPR, 2, true>(ntl, nb, s);
        if constexpr (LPR >= 4) return launch_ntl<IO, LPR, 2, false>(ntl, nb, s);
        return hipErrorInvalidValue;  // 2 LPR - d < LPR: none below 4
    }
    // single modes have no fully unrolled form: odd d never fills LPR > 1
    return launch_ntl<IO, LPR, 1, false>(ntl, nb, s);
}

template <typename IO>
hipError_t launch_lanes(int lpr, int vec, bool ntl, int nb, const Step& s)
{
    switch (lpr) {
        case 1: return launch_vec<IO, 1>(vec, ntl, nb, s);
        case 2: return launch_vec<IO, 2>(vec, ntl, nb, s);
        case 4: return launch_vec<IO, 4>(vec, ntl, nb, s);
        case 8: return launch_vec<IO, 8>(vec, ntl, nb, s);
        case 16: return launch_vec<IO, 16>(vec, ntl, nb, s);
        case 32: return launch_vec<IO, 32>(vec, ntl, nb, s);
        case 64: return launch_vec<IO, 64>(vec, ntl, nb, s);
        default: return hipErrorInvalidValue;
    }
}

template <typename IO, int VEC>
hipError_t launch_generic(int lpr, const float2* lam, const float2* R, const float* h0,
                          float2* state, const void* u, void* y, int64_t B, int64_t D, int64_t d,
                          hipStream_t stream)
{
    const int64_t rows_per_block = kBlock / lpr;
    const int64_t nblocks = (D + rows_per_block - 1) / rows_per_block * B;
    if (nblocks > 0x7fffffff) return hipErrorInvalidConfiguration;
    const IO* uu = static_cast<const IO*>(u);
    IO* yy = static_cast<IO*>(y);
#define LH_GEN(L)                                                                            \
    case L:                                                                                  \
        hipLaunchKernelGGL((step_generic_kernel<IO, L, VEC>), dim3(uint32_t(nblocks)),       \
                           dim3(kBlock), 0, stream, lam, R, h0, state, uu, yy, B, D, d,      \
                           nblocks);                                                         \
        break;
    switch (lpr) {
        LH_GEN(1)
        LH_GEN(2)
        LH_GEN(4)
        LH_GEN(8)
        LH_GEN(16)
        LH_GEN(32)
        LH_GEN(64)
        default:
            return hipErrorInvalidValue;
    }
#undef LH_GEN
    return hipGetLastError();
}

}  // namespace

hipError_t launch_step(const float2* lam, const float2* R, const float* h0, float2* state,
                       const void* u_t, void* y_t, bool bf16_io, int64_t B, int64_t D,
                       int64_t d, bool aligned16, hipStream_t stream)
{
    (void)hipGetLastError();  // clear a stale error so the status below is this launch's
    const int64_t pairs = d / 2;
    const int vec = d % 2 == 0 && aligned16 ? 2 : 1;
    int fast_lpr = 1;
    while (int64_t(fast_lpr) * vec < d) fast_lpr *= 2;
    const bool small_odd = vec == 1 && d > 1 && d <= 16 && 8 * B * D * d <= kStridedBytes;
    if (fast_lpr <= 64 && !small_odd && B < (INT64_C(1) << 31) && D < (INT64_C(1) << 31)) {
        const int nb = pairs_rows_per_thread(fast_lpr, vec, B, D, d);
        Step s{lam, R, h0, state, u_t, y_t, int(B), int(D), int(d), dim3(), 0, stream};
        if (pairs_grid(fast_lpr, nb, B, D, &s.grid, &s.ntiles)) {
            const bool ntl = 8 * B * D * d <= kStreamStateBytes;
            return bf16_io ? launch_lanes<bf16>(fast_lpr, vec, ntl, nb, s)
                           : launch_lanes<float>(fast_lpr, vec, ntl, nb, s);
        }
    }
    // generic layouts
    int lpr = 1;
    const bool vec2 = d % 2 == 0 && aligned16;
    if (vec2) {
        while (lpr < 32 && pairs % (2 * lpr) == 0) lpr *= 2;
        return bf16_io ? launch_generic<bf16, 2>(lpr, lam, R, h0, state, u_t, y_t, B, D, d, stream)
                       : launch_generic<float, 2>(lpr, lam, R, h0, state, u_t, y_t, B, D, d,
                                                  stream);
    }
    while (lpr < 64 && lpr < d) lpr *= 2;
    return bf16_io ? launch_generic<bf16, 1>(lpr, lam, R, h0, state, u_t, y_t, B, D, d, stream)
                   : launch_generic<float, 1>(lpr, lam, R, h0, state, u_t, y_t, B, D, d, stream);
}

}  // namespace lh
