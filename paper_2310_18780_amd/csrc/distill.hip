// Distillation objective of the modal form (Sec. 3.2, "Modal canonical form"):
// per channel c, poles in polar form lambda_n = A_n e^{i theta_n}, residues
// R_n, and a real target filter h_1 .. h_L,
//
//   hhat_t = Re sum_n R_n lambda_n^(t-1)          (eq. "modal_impulse", t = 1..L)
//   e_t    = hhat_t - h_t,   loss = sum_t e_t^2
//   d loss / dR_n     = 2 conj(sum_t e_t lambda_n^(t-1))          (as d/dRe R + i d/dIm R)
//   d loss / dA_n     = 2 Re(R_n e^{i theta_n} S_n)
//   d loss / dtheta_n = 2 Re(i R_n lambda_n S_n),   S_n = sum_t e_t (t-1) lambda_n^(t-2)
//
// and, optionally, the materialised filter hhat (the O(dL) evaluation of
// Lemma "ssmd_impulse").
//
// d <= 64: on the matrix cores (distill_mfma_kernel).  With t - 1 = 16 a + b the
// powers factor, lambda^(t-1) = lambda^(16 a) lambda^b, and every sum over the taps
// is a contraction of small matrices, 16 x 16 taps (a tile) at a time:
//
//   hhat[a][b]  = sum_n Re( (R_n lambda_n^(16 a)) lambda_n^b )                 K = 2d
//   F1[n][b]   += sum_(a > 0) lambda_n^(16 (a-1)) e[a][b]                       K = 16
//   F'[n][b]   += sum_a lambda_n^(16 (a-1)) (16 a e[a][b])                      K = 16
//   sum_t e_t lambda^(t-1) = sum_b lambda^b F[b],  F = lambda^16 F1 + e[0]
//   S = sum_b (lambda^(b+15) F'[b] + b lambda^(b-1) F[b])
//
// in float32 (v_mfma_f32_16x16x4_f32, exact products, float32 sums).  The
// accumulators of hhat, rows a and columns b, are the B operand of the second
// contraction as they are (its K index 4 g + i is the row that lane group g holds in
// register i).  The powers of a tile are lambda^(16 alpha) (constant) times
// lambda^(256 k), both from float64 products rounded once, so that no rounding error
// builds up along t.  A workgroup of four waves per channel, each wave every fourth
// tile.  D = 2048, d = 16, L = 4096: 65 -> 28 us (the VALU kernel below issues 23
// instructions per (t, n)), D = 2048, d = 60, L = 1024: 216 -> 49 us, D = 256, d = 16,
// L = 4096: 21 -> 9 us.  Of the 28 us the float32 matrix products are 10 us (24 of 32
// cycles per tile and wave; the counters show the matrix units busy for 0.30 of the time
// and vector instructions issued for 0.46), 10 us the latency of loads and tables before
// the first tile in two rounds of workgroups; more wavefronts per SIMD spill (34-50 us).
//
// d > 64: on the VALU (distill_kernel).  One workgroup of 256 threads per channel.
// The time axis is cut into segments of 256 x 16 steps; in a segment thread k owns 16
// consecutive steps.
// Pass 1 sums the filter over the modes (in chunks of 8, so any d fits the
// registers) for the thread's steps, from start powers lambda^(t0-1) evaluated
// in polar form (the logarithm of A and the angle reduction in float64, then
// float32 exp and sincos) followed by float32 running products over the 16
// steps; it forms e_t, the loss and, if asked, writes hhat.  Pass 2 walks the
// same powers again and accumulates e_t lambda^(t-1) and e_t (t-1)
// lambda^(t-2) per mode; each chunk's sums are reduced over the wave with DPP
// row permutations and the four row sums, then over the four waves in LDS.
// Per-mode constants (lambda in float32, ln A and theta in float64) are formed
// once per workgroup in LDS.  The work is about 20 flops per (t, n) on the VALU.
//
// Both finalise the gradients without dividing by lambda, so A = 0 is exact.  The
// traffic is the target read once.
#include <float.h>

#include <type_traits>

#include "lh_internal.hpp"

namespace lh {
namespace {

constexpr int kThreads = 256;
constexpr int kWavesD = kThreads / 64;
constexpr int kTB = 16;                    // steps per thread in a segment
constexpr int kSeg = kThreads * kTB;       // steps per segment
constexpr int kMC = 8;                     // modes per chunk

__device__ __forceinline__ float wave_sum64(float v)
{
    int x = __builtin_bit_cast(int, v);
    v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(x, 0xB1, 0xF, 0xF, false));  // quad_perm [1,0,3,2]
    x = __builtin_bit_cast(int, v);
    v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(x, 0x4E, 0xF, 0xF, false));  // quad_perm [2,3,0,1]
    x = __builtin_bit_cast(int, v);
    v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(x, 0x141, 0xF, 0xF, false));  // row_half_mirror
    x = __builtin_bit_cast(int, v);
    v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(x, 0x140, 0xF, 0xF, false));  // row_mirror
    x = __builtin_bit_cast(int, v);
    return (__builtin_bit_cast(float, __builtin_amdgcn_readlane(x, 0)) +
            __builtin_bit_cast(float, __builtin_amdgcn_readlane(x, 16))) +
           (__builtin_bit_cast(float, __builtin_amdgcn_readlane(x, 32)) +
            __builtin_bit_cast(float, __builtin_amdgcn_readlane(x, 48)));
}

// lambda^e in polar form: A^e = exp(e ln A) (ln A in float64), the angle
// e theta reduced modulo 2 pi in float64, then float32 exp and sincos; A = 0
// gives 0^0 = 1 and 0 otherwise
__device__ __forceinline__ float2 polar_pow(double lnA, bool zero, double theta, int64_t e)
{
    if (e < 0) return make_float2(0.f, 0.f);
    if (zero) return e == 0 ? make_float2(1.f, 0.f) : make_float2(0.f, 0.f);
    const float mag = __expf(float(double(e) * lnA));
    const double kTwoPi = 6.283185307179586476925286766559;
    const double kInvTwoPi = 0.15915494309189533576888376337251;
    double ang = double(e) * theta;
    ang = fma(-kTwoPi, floor(ang * kInvTwoPi), ang);
    float sn, cs;
    __sincosf(float(ang), &sn, &cs);
    return make_float2(mag * cs, mag * sn);
}

__device__ __forceinline__ float2 cmul(float2 a, float2 b)
{
    return make_float2(fmaf(a.x, b.x, -a.y * b.y), fmaf(a.x, b.y, a.y * b.x));
}

__global__ __launch_bounds__(kThreads) void distill_kernel(
    const float* __restrict__ A, const float* __restrict__ theta, const float2* __restrict__ R,
    const float* __restrict__ target, int d, int64_t L, float* __restrict__ loss,
    float* __restrict__ dA, float* __restrict__ dtheta, float2* __restrict__ dR,
    float* __restrict__ hhat)
{
    const int c = blockIdx.x;
    const int tid = threadIdx.x, lane = tid % 64, wv = tid / 64;
    __shared__ float red[kWavesD][kMC][4];  // per-wave chunk sums: Re/Im of g and S
    __shared__ float acc_s[kWavesD];
    // dynamic LDS: gs [d][4] (sum_t e lambda^(t-1), sum_t e (t-1) lambda^(t-2)),
    // then per mode lambda (float2), ln A and theta (double)
    extern __shared__ __attribute__((aligned(16))) double dyn[];
    double* lnA_s = dyn;
    double* th_s = dyn + d;
    float2* lam_s = reinterpret_cast<float2*>(dyn + 2 * d);
    float* gs = reinterpret_cast<float*>(lam_s + d);
    const float* Ac = A + int64_t(c) * d;
    const float* Tc = theta + int64_t(c) * d;
    const float2* Rc = R + int64_t(c) * d;
    const float* hc = target + int64_t(c) * L;
    for (int i = tid; i < 4 * d; i += kThreads) gs[i] = 0.f;
    for (int n = tid; n < d; n += kThreads) {
        const double a = Ac[n], th = Tc[n];
        lnA_s[n] = a > 0.0 ? log(a) : 0.0;
        th_s[n] = th;
        lam_s[n] = make_float2(float(a * cos(th)), float(a * sin(th)));
    }
    float lacc = 0.f;
    __syncthreads();

    for (int64_t seg0 = 0; seg0 < L; seg0 += kSeg) {
        const int64_t s0 = seg0 + int64_t(tid) * kTB;  // index of t - 1 of the first step
        float hh[kTB];
#pragma unroll
        for (int s = 0; s < kTB; ++s) hh[s] = 0.f;
        // pass 1: hhat over the thread's steps
        for (int n0 = 0; n0 < d; n0 += kMC) {
#pragma unroll
            for (int q = 0; q < kMC; ++q) {
                const int n = n0 + q;
                if (n >= d) break;
                const float2 lam = lam_s[n];
                float2 p = polar_pow(lnA_s[n], Ac[n] == 0.f, th_s[n], s0);
                const float2 r = Rc[n];
#pragma unroll
                for (int s = 0; s < kTB; ++s) {
                    hh[s] = fmaf(r.x, p.x, fmaf(-r.y, p.y, hh[s]));
                    p = cmul(p, lam);
                }
            }
        }
        float e[kTB];
#pragma unroll
        for (int s = 0; s < kTB; ++s) {
            const int64_t t = s0 + s;
            const bool in = t < L;
            e[s] = in ? hh[s] - hc[in ? t : 0] : 0.f;
            lacc = fmaf(e[s], e[s], lacc);
            if (hhat && in) hhat[int64_t(c) * L + t] = hh[s];
        }
        // pass 2: gradient sums, one chunk of modes at a time
        for (int n0 = 0; n0 < d; n0 += kMC) {
            float sums[kMC][4];
#pragma unroll
            for (int q = 0; q < kMC; ++q) {
                const int n = n0 + q;
                sums[q][0] = sums[q][1] = sums[q][2] = sums[q][3] = 0.f;
                if (n >= d) continue;
                const float2 lam = lam_s[n];
                // lambda^(t-2) (0 at t = 1) and lambda^(t-1)
                float2 pm = polar_pow(lnA_s[n], Ac[n] == 0.f, th_s[n], s0 - 1);
                float2 p = s0 == 0 ? make_float2(1.f, 0.f) : cmul(pm, lam);
#pragma unroll
                for (int s = 0; s < kTB; ++s) {
                    const float w = e[s] * float(s0 + s);  // e_t (t - 1)
                    sums[q][0] = fmaf(e[s], p.x, sums[q][0]);
                    sums[q][1] = fmaf(e[s], p.y, sums[q][1]);
                    sums[q][2] = fmaf(w, pm.x, sums[q][2]);
                    sums[q][3] = fmaf(w, pm.y, sums[q][3]);
                    pm = p;
                    p = cmul(p, lam);
                }
            }
#pragma unroll
            for (int q = 0; q < kMC; ++q)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float v = wave_sum64(sums[q][j]);
                    if (lane == 0) red[wv][q][j] = v;
                }
            __syncthreads();
            if (tid < kMC * 4) {
                const int q = tid / 4, j = tid % 4;
                if (n0 + q < d) {
                    float v = 0.f;
#pragma unroll
                    for (int w2 = 0; w2 < kWavesD; ++w2) v += red[w2][q][j];
                    gs[(n0 + q) * 4 + j] += v;
                }
            }
            __syncthreads();
        }
    }
    const float lw = wave_sum64(lacc);
    if (lane == 0) acc_s[wv] = lw;
    __syncthreads();
    if (tid == 0) {
        float v = 0.f;
        for (int w2 = 0; w2 < kWavesD; ++w2) v += acc_s[w2];
        loss[c] = v;
    }
    for (int n = tid; n < d; n += kThreads) {
        const float2 g = make_float2(gs[4 * n], gs[4 * n + 1]);
        const float2 S = make_float2(gs[4 * n + 2], gs[4 * n + 3]);
        const float2 r = Rc[n];
        const double th = th_s[n];
        const float2 unit = make_float2(float(cos(th)), float(sin(th)));
        const float2 lam = lam_s[n];
        const float2 rs = cmul(r, S);
        dR[int64_t(c) * d + n] = make_float2(2.f * g.x, -2.f * g.y);
        dA[int64_t(c) * d + n] = 2.f * cmul(rs, unit).x;
        dtheta[int64_t(c) * d + n] = -2.f * cmul(rs, lam).y;  // Re(i z) = -Im(z)
    }
}

// ---- d <= 64 on the matrix cores
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kTile = 256;      // taps per tile: 16 a x 16 b
constexpr int kMaxTiles = 32;   // tiles whose lambda^(256 k) are held at a time

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// sum over the 16 lanes of a DPP row, in every lane
__device__ __forceinline__ float row_sum16(float v)
{
    int x = __builtin_bit_cast(int, v);
    v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(x, 0xB1, 0xF, 0xF, false));  // quad_perm [1,0,3,2]
    x = __builtin_bit_cast(int, v);
    v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(x, 0x4E, 0xF, 0xF, false));  // quad_perm [2,3,0,1]
    x = __builtin_bit_cast(int, v);
    v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(x, 0x141, 0xF, 0xF, false));  // row_half_mirror
    x = __builtin_bit_cast(int, v);
    return v + __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(x, 0x140, 0xF, 0xF, false));  // row_mirror
}

// DM = ceil(d / 16); modes past d have lambda = R = 0.
template <int DM>
__global__ __launch_bounds__(kThreads) void distill_mfma_kernel(
    const float* __restrict__ A, const float* __restrict__ theta, const float2* __restrict__ R,
    const float* __restrict__ target, int d, int64_t L, float* __restrict__ loss,
    float* __restrict__ dA, float* __restrict__ dtheta, float2* __restrict__ dR,
    float* __restrict__ hhat)
{
    constexpr int dp = 16 * DM;
    __shared__ float2 pw[dp][17];               // lambda^b
    __shared__ float2 p16[dp][17];              // lambda^(16 alpha)
    __shared__ float2 wk[kMaxTiles + 1][dp];    // lambda^(256 (k - 1)) of the tiles k0 - 1 + ...
    __shared__ float red[kWavesD][dp][4];
    __shared__ float loss_s[kWavesD];
    __shared__ float e0_s[16];                  // e of the first 16 taps (a = 0)
    const int c = blockIdx.x, tid = threadIdx.x, lane = tid % 64, w = tid / 64;
    const int g = lane / 16, q = lane % 16;
    const float* Ac = A + int64_t(c) * d;
    const float* Tc = theta + int64_t(c) * d;
    const float2* Rc = R + int64_t(c) * d;
    const float* hc = target + int64_t(c) * L;
    const int64_t ntile = (L + kTile - 1) / kTile;

    // tables, lane = mode: wave 0 lambda^b, wave 1 lambda^(16 alpha), wave 2
    // lambda^(256 k) (in the loop), float64 products rounded once
    double lr = 0.0, li = 0.0;  // lambda^(1, 16 or 256)
    double sn = 0.0, cs = 0.0;  // (wave 0 needs them again at the end)
    if (w < 3 && lane < d) {
        const double a = Ac[lane], th = Tc[lane];
        sincos(th, &sn, &cs);
        lr = a * cs;
        li = a * sn;
        for (int i = 0; i < 4 * w; ++i) {
            const double t = lr * lr - li * li;
            li = 2.0 * lr * li;
            lr = t;
        }
    }
    double kr = 1.0, ki = 0.0;
    auto advance = [&] {
        const double t = kr * lr - ki * li;
        ki = kr * li + ki * lr;
        kr = t;
    };
    if (w < 2 && lane < dp) {
        float2* const row = w == 0 ? pw[lane] : p16[lane];
        for (int b = 0; b < 16; ++b, advance()) row[b] = make_float2(float(kr), float(ki));
    }
    if (w == 2 && lane < dp) wk[0][lane] = make_float2(0.f, 0.f);
    __syncthreads();

    // constant operands: X0[j] = R lambda^(16 alpha) of mode 4 j + g at the row q
    // (alpha = 4 (q % 4) + q / 4, so that register i and lane group g hold alpha =
    // 4 i + g: 64 consecutive taps per register), V[j] = lambda^b of the same mode
    // at b = q, P1[m][i] = lambda^(16 (alpha - 1)) of mode 16 m + q at alpha = 4 i + g;
    // at alpha = 0 lambda^240, which goes with the tile before
    float2 X0[4 * DM], V[4 * DM], P1[DM][4];
#pragma unroll
    for (int j = 0; j < 4 * DM; ++j) {
        const int n = 4 * j + g;
        const float2 r = n < d ? Rc[n] : make_float2(0.f, 0.f);
        X0[j] = cmul(r, p16[n][4 * (q % 4) + q / 4]);
        V[j] = pw[n][q];
    }
#pragma unroll
    for (int m = 0; m < DM; ++m)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            P1[m][i] = p16[16 * m + q][(4 * i + g + 15) % 16];
            // lambda^240 meets zeros in the first tile, also where it overflows (and all
            // taps it would count for, past the 256th, do too)
            if (i == 0 && g == 0)
                P1[m][i] = make_float2(fminf(fmaxf(P1[m][i].x, -FLT_MAX), FLT_MAX),
                                       fminf(fmaxf(P1[m][i].y, -FLT_MAX), FLT_MAX));
        }
    f32x4 F[DM][4];  // Re F1, Im F1, Re F', Im F': rows modes 16 m + 4 g + i, column b = q
#pragma unroll
    for (int m = 0; m < DM; ++m)
#pragma unroll
        for (int z = 0; z < 4; ++z) F[m][z] = f32x4{0.f, 0.f, 0.f, 0.f};
    float lacc = 0.f;
    // Rows of the last tile that take part in F: not those past the last tap, whose
    // powers may overflow where |lambda| > 1 while every power up to lambda^(L-1) is
    // finite (inf times the zero errors there is no zero).
    auto inside = [&](int64_t s0, int i) { return 16 * (4 * i + g) < int(L - s0); };

    for (int64_t k0 = 0; k0 < ntile; k0 += kMaxTiles) {
        const int nk = int(ntile - k0 < kMaxTiles ? ntile - k0 : kMaxTiles);
        if (k0 > 0) __syncthreads();
        if (w == 2 && lane < dp) {
            if (k0 > 0) wk[0][lane] = wk[kMaxTiles][lane];
            for (int k = 0; k < nk; ++k, advance()) wk[k + 1][lane] = make_float2(float(kr), float(ki));
        }
        __syncthreads();
        for (int k = w; k < nk; k += kWavesD) {
            const int64_t s0 = (k0 + k) * kTile;
            float h[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int64_t s = s0 + 16 * (4 * i + g) + q;
                h[i] = hc[s < L ? s : L - 1];
            }
            f32x4 y = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < 4 * DM; ++j) {
                const float2 x = cmul(X0[j], wk[k + 1][4 * j + g]);
                y = mfma4(x.x, V[j].x, y);
                y = mfma4(-x.y, V[j].y, y);
            }
            float e[4], ae[4];  // e and 16 a e
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int64_t s = s0 + 16 * (4 * i + g) + q;
                const bool in = s < L;
                e[i] = in ? y[i] - h[i] : 0.f;
                lacc = fmaf(e[i], e[i], lacc);
                if (hhat && in) hhat[int64_t(c) * L + s] = y[i];
                ae[i] = float(s0 + 16 * (4 * i + g)) * e[i];
            }
            if (s0 == 0 && g == 0) {  // a = 0 has no lambda^(16 (a - 1)): added at the end
                e0_s[q] = e[0];
                e[0] = 0.f;
            }
            auto accumulate = [&](auto edge) {
#pragma unroll
                for (int m = 0; m < DM; ++m) {
                    const float2 a = wk[k + 1][16 * m + q], a0 = wk[k + (g > 0)][16 * m + q];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        float2 p = cmul(P1[m][i], i == 0 ? a0 : a);
                        if constexpr (decltype(edge)::value)
                            if (!inside(s0, i)) p = make_float2(0.f, 0.f);
                        F[m][0] = mfma4(p.x, e[i], F[m][0]);
                        F[m][1] = mfma4(p.y, e[i], F[m][1]);
                        F[m][2] = mfma4(p.x, ae[i], F[m][2]);
                        F[m][3] = mfma4(p.y, ae[i], F[m][3]);
                    }
                }
            };
            if (s0 + kTile > L)  // (in every tile the masks take 1 of the 30 us)
                accumulate(std::true_type{});
            else
                accumulate(std::false_type{});
        }
    }

    // F = lambda^16 F1 + e[0], sums over b, then over the waves; for at most 16 taps
    // (only a = 0) powers that no tap has stay out here too
    __syncthreads();
    const float e0 = w == 0 ? e0_s[q] : 0.f;
    const float fb = float(q);
    auto finish = [&](auto few) {
        constexpr bool FEW = decltype(few)::value;
        const float2 none = make_float2(0.f, 0.f);
#pragma unroll
        for (int m = 0; m < DM; ++m)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int n = 16 * m + 4 * g + i;
                float2 p = pw[n][q];                       // lambda^b
                float2 pb = q > 0 ? pw[n][q - 1] : none;  // lambda^(b-1)
                float2 f = none, fd = none;
                if constexpr (FEW) {
                    if (q >= L) p = pb = none;
                } else {
                    f = cmul(p16[n][1], make_float2(F[m][0][i], F[m][1][i]));
                    fd = cmul(pw[n][15], make_float2(F[m][2][i], F[m][3][i]));
                }
                f.x += e0;
                const float2 gv = cmul(p, f);
                const float2 s1 = cmul(p, fd), s2 = cmul(pb, f);
                const float v0 = row_sum16(gv.x), v1 = row_sum16(gv.y);
                const float v2 = row_sum16(fmaf(fb, s2.x, s1.x)), v3 = row_sum16(fmaf(fb, s2.y, s1.y));
                if (q == 0) {
                    red[w][n][0] = v0;
                    red[w][n][1] = v1;
                    red[w][n][2] = v2;
                    red[w][n][3] = v3;
                }
            }
    };
    if (L > 16)
        finish(std::false_type{});
    else
        finish(std::true_type{});
    const float lw = wave_sum64(lacc);
    if (lane == 0) loss_s[w] = lw;
    __syncthreads();
    if (tid == 0) loss[c] = (loss_s[0] + loss_s[1]) + (loss_s[2] + loss_s[3]);
    if (tid < d) {
        // in float64, once per mode: R S lambda is almost real where one mode explains
        // the error of its taps, and its imaginary part, the gradient in theta, then
        // keeps every rounding of the product
        double v[4];
#pragma unroll
        for (int z = 0; z < 4; ++z)
            v[z] = (double(red[0][tid][z]) + red[1][tid][z]) + (double(red[2][tid][z]) + red[3][tid][z]);
        const float2 r = Rc[tid];
        const double a = Ac[tid];
        const double rx = double(r.x) * v[2] - double(r.y) * v[3];
        const double ry = double(r.x) * v[3] + double(r.y) * v[2];
        dR[int64_t(c) * d + tid] = make_float2(float(2.0 * v[0]), float(-2.0 * v[1]));
        dA[int64_t(c) * d + tid] = float(2.0 * (rx * cs - ry * sn));
        dtheta[int64_t(c) * d + tid] = float(-2.0 * a * (rx * sn + ry * cs));  // Re(i z) = -Im(z)
    }
}

}  // namespace

hipError_t launch_distill(const float* A, const float* theta, const float2* R,
                          const float* target, int64_t D, int64_t d, int64_t L, float* loss,
                          float* dA, float* dtheta, float2* dR, float* hhat, hipStream_t stream)
{
    (void)hipGetLastError();
    if (D > 0x7fffffff || d > 0x7fffffff) return hipErrorInvalidConfiguration;
    // the matrix-core kernel holds the operands of up to 64 modes in registers
    if (d <= 64) {
#define LH_DISTILL(M)                                                                            \
    case M:                                                                                      \
        hipLaunchKernelGGL((distill_mfma_kernel<M>), dim3(uint32_t(D)), dim3(kThreads), 0,       \
                           stream, A, theta, R, target, int(d), L, loss, dA, dtheta, dR, hhat);  \
        break;
        switch ((d + 15) / 16) {
            LH_DISTILL(1)
            LH_DISTILL(2)
            LH_DISTILL(3)
            LH_DISTILL(4)
            default: return hipErrorInvalidValue;
        }
#undef LH_DISTILL
        return hipGetLastError();
    }
    const size_t shm = size_t(d) * (2 * sizeof(double) + sizeof(float2) + 4 * sizeof(float));
    hipLaunchKernelGGL(distill_kernel, dim3(uint32_t(D)), dim3(kThreads), shm, stream, A, theta,
                       R, target, int(d), L, loss, dA, dtheta, dR, hhat);
    return hipGetLastError();
}

}  // namespace lh
