#include "sfc_gemm_kernel.h"
#include "sfc_gemm_variants.h"

namespace sfc {

const void* kernel_256x128(bool ob) {
  return ob ? kernel_ptr<256, 128, kWaves, 0, true, kLoadRing>() : kernel_ptr<256, 128, kWaves, 0, false, kLoadRing>();
}

}  // namespace sfc
