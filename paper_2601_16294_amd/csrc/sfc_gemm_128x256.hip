#include "sfc_gemm_kernel.h"
#include "sfc_gemm_variants.h"

namespace sfc {

const void* kernel_128x256(bool ob) {
  return ob ? kernel_ptr<128, 256, kWaves, 0, true, kLoadRing>() : kernel_ptr<128, 256, kWaves, 0, false, kLoadRing>();
}

}  // namespace sfc
