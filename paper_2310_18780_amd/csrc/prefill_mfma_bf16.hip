// Matrix-core prefill kernels for bfloat16 u and y.
#include "prefill_mfma_kernel.hpp"

namespace lh {

hipError_t launch_mfma_kernel_bf16(int dm, int s, bool outputs, const MfmaArgs& a, hipStream_t stream)
{
    return launch_io<bf16>(dm, s, outputs, a, stream);
}

}  // namespace lh
