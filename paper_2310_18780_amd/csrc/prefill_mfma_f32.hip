// Matrix-core prefill kernels for float32 u and y.
#include "prefill_mfma_kernel.hpp"

namespace lh {

hipError_t launch_mfma_kernel_f32(int dm, int s, bool outputs, const MfmaArgs& a, hipStream_t stream)
{
    return launch_io<float>(dm, s, outputs, a, stream);
}

}  // namespace lh
