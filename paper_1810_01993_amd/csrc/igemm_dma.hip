// Implicit-GEMM convolution engine, direct-to-LDS variant: fp16 kernels, and the choice between the two storage types.
#include "igemm_dma_launch.h"

namespace dlk {

hipError_t launch_igemm_dma(const IgemmArgs &a, bool is_bf16, int cfg, hipStream_t stream)
{
    return is_bf16 ? launch_igemm_dma_bf16(a, cfg, stream) : dispatch_dma<F16>(a, cfg, stream);
}

hipError_t launch_igemm_dma_batch(const IgemmBatch &b, bool is_bf16, int cfg, hipStream_t stream)
{
    if (b.n < 1 || b.n > IgemmBatch::MAX) return hipErrorInvalidValue;
    return is_bf16 ? launch_igemm_dma_batch_bf16(b, cfg, stream) : dispatch_dma_batch<F16>(b, cfg, stream);
}

}  // namespace dlk
