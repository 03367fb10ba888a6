#include "sfc_gemm_kernel.h"
#include "sfc_gemm_variants.h"

namespace sfc {

const void* kernel_f8_256x256(bool ob, int f8) {
  switch (f8) {
    case 1: return ob ? kernel_ptr<256, 256, kWaves, 1, true, kLoadRing>() : kernel_ptr<256, 256, kWaves, 1, false, kLoadRing>();
    case 2: return ob ? kernel_ptr<256, 256, kWaves, 2, true, kLoadRing>() : kernel_ptr<256, 256, kWaves, 2, false, kLoadRing>();
    case 3: return ob ? kernel_ptr<256, 256, kWaves, 3, true, kLoadRing>() : kernel_ptr<256, 256, kWaves, 3, false, kLoadRing>();
    case 4: return ob ? kernel_ptr<256, 256, kWaves, 4, true, kLoadRing>() : kernel_ptr<256, 256, kWaves, 4, false, kLoadRing>();
    default: return nullptr;
  }
}

}  // namespace sfc
