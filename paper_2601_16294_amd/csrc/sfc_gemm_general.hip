#include "sfc_gemm_kernel.h"
#include "sfc_gemm_variants.h"

namespace sfc {

template <int LOADS>
static const void* kernel_loads(int tile, bool ob) {
  switch (tile) {
    case kT128x128: return ob ? kernel_ptr<128, 128, kWaves, 0, true, LOADS>() : kernel_ptr<128, 128, kWaves, 0, false, LOADS>();
    case kT256x128: return ob ? kernel_ptr<256, 128, kWaves, 0, true, LOADS>() : kernel_ptr<256, 128, kWaves, 0, false, LOADS>();
    case kT128x256: return ob ? kernel_ptr<128, 256, kWaves, 0, true, LOADS>() : kernel_ptr<128, 256, kWaves, 0, false, LOADS>();
    case kT256x256: return ob ? kernel_ptr<256, 256, kWaves, 0, true, LOADS>() : kernel_ptr<256, 256, kWaves, 0, false, LOADS>();
    default: return nullptr;
  }
}

const void* kernel_any(int tile, bool ob) { return kernel_loads<kLoadAny>(tile, ob); }
const void* kernel_elements(int tile, bool ob) { return kernel_loads<kLoadElements>(tile, ob); }

}  // namespace sfc
