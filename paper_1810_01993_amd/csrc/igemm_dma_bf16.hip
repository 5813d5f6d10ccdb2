// Implicit-GEMM convolution engine, direct-to-LDS variant: bf16 kernels.
#include "igemm_dma_launch.h"

namespace dlk {

hipError_t launch_igemm_dma_bf16(const IgemmArgs &a, int cfg, hipStream_t stream) { return dispatch_dma<BF16>(a, cfg, stream); }
hipError_t launch_igemm_dma_batch_bf16(const IgemmBatch &b, int cfg, hipStream_t stream) { return dispatch_dma_batch<BF16>(b, cfg, stream); }

}  // namespace dlk
