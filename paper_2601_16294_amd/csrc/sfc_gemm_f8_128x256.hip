#include "sfc_gemm_kernel.h"
#include "sfc_gemm_variants.h"

namespace sfc {

const void* kernel_f8_128x256(bool ob, int f8) {
  switch (f8) {
    case 1: return ob ? kernel_ptr<128, 256, kWaves, 1, true, true>() : kernel_ptr<128, 256, kWaves, 1, false, true>();
    case 2: return ob ? kernel_ptr<128, 256, kWaves, 2, true, true>() : kernel_ptr<128, 256, kWaves, 2, false, true>();
    case 3: return ob ? kernel_ptr<128, 256, kWaves, 3, true, true>() : kernel_ptr<128, 256, kWaves, 3, false, true>();
    case 4: return ob ? kernel_ptr<128, 256, kWaves, 4, true, true>() : kernel_ptr<128, 256, kWaves, 4, false, true>();
    default: return nullptr;
  }
}

}  // namespace sfc
