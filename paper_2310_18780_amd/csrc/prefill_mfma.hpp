// Shared by the matrix-core prefill's host side and its kernels: the tilings
// and the kernel arguments.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lh {

constexpr int kMfmaChunk = 16;     // steps per chunk
constexpr int kMfmaMaxModes = 64;  // modes per channel, padded to a multiple of 16

// Tiling for DM = ceil(d / 16) sixteens of modes.  A wave owns kCpw channels: as
// many as its A operands leave room for in 256 registers, and as the wave has
// scan lanes for (kCpw 16 DM <= 64).  Float32 u and y at d <= 16 take two
// channels (64-byte pieces of a line), four would need 144 registers of
// operands.  Fragments of 64 x 16 bytes per channel: T, then P (two per 8
// modes), then W (one per term and 16 modes).  With bfloat16 u and y T and W have
// two terms in the two-term kernels (X3 = false), else three.
template <bool BF, int DM, bool X3>
struct MfmaTiling {
    static constexpr int kCpw = BF ? (DM == 1 ? 4 : DM == 2 ? 2 : 1) : (DM <= 2 ? 2 : 1);
    static constexpr int kCw = 8 * kCpw;
    static constexpr int kP = BF && !X3 ? 1 : 2;
    static constexpr int kW = kP + 4 * DM;
    static constexpr int kFrags = kW + (BF && !X3 ? 2 : 3) * DM;
};

inline int mfma_channels(bool bf, int dm)
{
    return 8 * (bf ? (dm == 1 ? 4 : dm == 2 ? 2 : 1) : (dm <= 2 ? 2 : 1));
}

struct MfmaArgs {
    const float2 *lam, *R;
    const float* h0;
    const void* u;
    void* y;
    float2* state;
    const void* frag;  // A operands in lane order
    const void* lamc;  // lambda^16 as float32 high and low parts [D][16 DM] float4
    float2* xs;        // segment states [B, nseg, D, d]
    int64_t T, seg_len;
    int B, D, d, nseg;
    bool two_terms;     // MfmaCut
    int ncg, nrg, per_xcd;  // grid (set by the launcher)
};

// s: time chunks per row among the kernel's 16 columns (1, 2, 4 or 16; 16
// with nseg > 1); outputs = false is the state pass of the segmented plan.
hipError_t launch_mfma_kernel_f32(int dm, int s, bool outputs, const MfmaArgs& a, hipStream_t stream);
hipError_t launch_mfma_kernel_bf16(int dm, int s, bool outputs, const MfmaArgs& a, hipStream_t stream);

}  // namespace lh
