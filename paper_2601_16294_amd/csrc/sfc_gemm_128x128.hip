#include "sfc_gemm_kernel.h"
#include "sfc_gemm_variants.h"

namespace sfc {

const void* kernel_128x128(bool ob) {
  return ob ? kernel_ptr<128, 128, kWaves, 0, true, kLoadRing>() : kernel_ptr<128, 128, kWaves, 0, false, kLoadRing>();
}

const void* kernel_128x128_deep(bool ob) {
  return ob ? kernel_ptr<128, 128, kWaves, 0, true, kLoadRing, 4>() : kernel_ptr<128, 128, kWaves, 0, false, kLoadRing, 4>();
}

}  // namespace sfc
