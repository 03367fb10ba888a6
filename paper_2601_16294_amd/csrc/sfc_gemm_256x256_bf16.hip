#include "sfc_gemm_kernel.h"
#include "sfc_gemm_variants.h"

namespace sfc {

const void* kernel_256x256_bf16() { return kernel_ptr<256, 256, kWaves, 0, true, kLoadRing>(); }

}  // namespace sfc
