// Internal declarations of liblh: element helpers shared by the kernels and
// the launchers the C ABI layer calls.  Not part of the public interface.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace lh {

// bfloat16 storage type (upper half of a float32)
struct bf16 {
    uint16_t bits;
};

__device__ __forceinline__ float io_load(const float* p) { return *p; }
__device__ __forceinline__ float io_load(const bf16* p) {
    return __uint_as_float(static_cast<uint32_t>(p->bits) << 16);
}
__device__ __forceinline__ void io_store(float* p, float v) { *p = v; }
// float32 -> bfloat16, round to nearest, ties to even (gfx950 converts with
// one v_cvt_pk_bf16_f32; NaN stays NaN).
__device__ __forceinline__ void io_store(bf16* p, float v) {
    p->bits = __builtin_bit_cast(uint16_t, static_cast<__bf16>(v));
}

// Non-temporal variants (written once, not re-read soon): keep the cache for
// data that is.
__device__ __forceinline__ void io_store_nt(float* p, float v) { __builtin_nontemporal_store(v, p); }
__device__ __forceinline__ void io_store_nt(bf16* p, float v) {
    __builtin_nontemporal_store(__builtin_bit_cast(uint16_t, static_cast<__bf16>(v)), &p->bits);
}

// Columns and segments of a matrix-core prefill.
struct MfmaCut {
    int s;            // time chunks per row among the kernel's 16 columns (1, 2, 4 or 16)
    int nseg;         // segments of the prompt (1: the whole prompt in one pass)
    int64_t seg_len;  // steps per segment (a multiple of 256 when nseg > 1)
    int64_t tiles;    // estimated time, in tiles of the busiest CU
    bool two_terms = false;  // the two-term kernels (named plans, 16-byte aligned u and y)
};

// How the prefill of one call is cut up.
struct PrefillPlan {
    int lpr;          // lanes per (b, c) row: the modes of a row are split over lpr lanes
    int mpl;          // modes per lane (power of two <= 16); lpr * mpl >= d
    int64_t C;        // VALU chunk length (time steps per chunk)
    int64_t nchunks;  // ceil(T / C); 0 when T == 0
    size_t off_pow;   // workspace offset of lambda^C          [D, d] complex64
    size_t off_xin;   // workspace offset of chunk (segment) entry states [B, n, D, d] complex64
    size_t ws_bytes;  // total workspace bytes
    size_t scan_bytes;  // workspace of the VALU scan (a plan that is reported as a scan
                        // takes it when the workspace holds no more)
    int named;        // reported plan: 0 scan, 1 matrix cores, 2 segmented matrix cores
    bool mfma;        // runs on the matrix cores, cut as `cut`
    bool forced;      // a matrix-core plan was requested: u and y must be 16-byte aligned
    MfmaCut cut;
    size_t off_mfma;  // workspace offset of the matrix-core tables
};

// The plan of a prefill call.  request: 0 automatic, > 0 the VALU chunked
// scan with this chunk length, -1 the matrix-core plan, -2 the segmented
// matrix-core plan.  Returns false when the sizes are invalid, overflow or do
// not support the request.  io: 0 float32, 1 bfloat16 u/y, -1 either (the
// automatic plan may differ between them; the workspace size is then the
// larger of the two).
bool make_prefill_plan(int64_t B, int64_t D, int64_t d, int64_t T, int64_t request, int io,
                       PrefillPlan* plan);

// Launchers (asynchronous, on `stream`); they return the launch status.
hipError_t launch_prefill(const float2* lam, const float2* R, const float* h0,
                          const void* u, bool bf16_io, int64_t B, int64_t D, int64_t d,
                          int64_t T, float2* state, void* y, const PrefillPlan& plan,
                          void* workspace, hipStream_t stream);

// Matrix-core prefill.  Sizes that the explicit matrix-core requests take (d = 16
// or 32 with D a multiple of 8, or d = 64 with float32 u/y and D a multiple of 4),
// and sizes that the kernel takes.
bool mfma_supported(int64_t B, int64_t D, int64_t d, int64_t T, bool bf16_io);
bool mfma_possible(int64_t B, int64_t D, int64_t d, int64_t T, bool bf16_io);
// Table bytes of the named plans (either input type) and of one input type and kernel.
size_t mfma_workspace_bytes(int64_t D, int64_t d);
size_t mfma_table_bytes(bool bf16_io, bool two_terms, int64_t D, int64_t d);
// Segment slots of the segmented plan's workspace (0 when T does not split into
// segments of a multiple of 32 steps, at least 256 long).
int64_t mfma_segments(int64_t B, int64_t D, int64_t d, int64_t T);
// The cut of a call into columns and at most max_seg segments.
MfmaCut mfma_cut(int64_t B, int64_t D, int64_t d, int64_t T, bool bf16_io, int64_t max_seg);
// Estimated time of a call on the three-term kernels, in microseconds.
double mfma_us(int64_t B, int64_t D, int64_t d, int64_t T, bool bf16_io, const MfmaCut& cut);
// Tables of the filters into the workspace.
hipError_t launch_mfma_setup(const float2* lam, const float2* R, const float* h0, int64_t D,
                             int64_t d, bool bf16_io, bool two_terms, void* workspace,
                             hipStream_t stream);
// One pass: outputs = false writes each segment's end state from zero into slot
// k < nseg - 1 of xs [B, nseg, D, d]; outputs = true runs every segment from its
// entry state in xs (the whole prompt from zero when nseg = 1), writes y and x_T.
hipError_t launch_mfma_pass(bool outputs, const float2* lam, const float2* R, const float* h0,
                            const void* u, bool bf16_io, int64_t B, int64_t D, int64_t d,
                            int64_t T, const MfmaCut& cut, float2* xs, float2* state, void* y,
                            const void* workspace, hipStream_t stream);

hipError_t launch_step(const float2* lam, const float2* R, const float* h0, float2* state,
                       const void* u_t, void* y_t, bool bf16_io, int64_t B, int64_t D,
                       int64_t d, bool aligned16, hipStream_t stream);

// Distillation objective: loss and gradients per channel (targets [D, L]).
hipError_t launch_distill(const float* A, const float* theta, const float2* R,
                          const float* target, int64_t D, int64_t d, int64_t L, float* loss,
                          float* dA, float* dtheta, float2* dR, float* hhat, hipStream_t stream);

// Multi-head decode step (state [B, M, N, N, d]; q, k, v, y [B, M N]).
hipError_t launch_mh_step(const float2* lam, const float2* R, const float* h0, float2* state,
                          const void* q, const void* k, const void* v, void* y, bool bf16_io,
                          int64_t B, int64_t M, int64_t N, int64_t d, bool aligned16,
                          hipStream_t stream);

}  // namespace lh
