#include "sfc_gemm_kernel.h"
#include "sfc_gemm_variants.h"

namespace sfc {

const void* kernel_general(int tile, bool ob) {
  switch (tile) {
    case kT128x128: return ob ? kernel_ptr<128, 128, kWaves, 0, true, false>() : kernel_ptr<128, 128, kWaves, 0, false, false>();
    case kT256x128: return ob ? kernel_ptr<256, 128, kWaves, 0, true, false>() : kernel_ptr<256, 128, kWaves, 0, false, false>();
    case kT128x256: return ob ? kernel_ptr<128, 256, kWaves, 0, true, false>() : kernel_ptr<128, 256, kWaves, 0, false, false>();
    case kT256x256: return ob ? kernel_ptr<256, 256, kWaves, 0, true, false>() : kernel_ptr<256, 256, kWaves, 0, false, false>();
    default: return nullptr;
  }
}

}  // namespace sfc
