// Choice and launch of the compiled GEMM kernels.
#include "sfc_gemm_variants.h"
#include "sfc_params.h"

namespace sfc {

// fp8 operands (f8 = 1 + a + 2b, a and b the formats of A and B: 0 OCP E4M3,
// 1 OCP E5M2): 256x256 or 128x256 blocks, fast path only.  deep: the 4-deep
// ring of 128x128 blocks (fast path), for grids of at most one block per CU.
static const void* select_kernel(int tile, bool ob, bool vec, int f8, bool deep) {
  if (f8) {
    if (tile == kT256x256) return kernel_f8_256x256(ob, f8);
    return tile == kT128x256 ? kernel_f8_128x256(ob, f8) : nullptr;
  }
  if (deep) return tile == kT128x128 && vec ? kernel_128x128_deep(ob) : nullptr;
  if (!vec) return kernel_general(tile, ob);
  switch (tile) {
    case kT128x128: return kernel_128x128(ob);
    case kT256x128: return kernel_256x128(ob);
    case kT128x256: return kernel_128x256(ob);
    case kT256x256: return ob ? kernel_256x256_bf16() : kernel_256x256_f32();
    default: return nullptr;
  }
}

constexpr int kThreads = 256;   // every kernel: 4 waves

hipError_t launch_gemm(int tile, bool out_bf16, bool vec, const GemmParams& p, int grid,
                       hipStream_t stream, int f8, bool deep) {
  const void* k = select_kernel(tile, out_bf16, vec, f8, deep);
  if (!k) return hipErrorInvalidValue;
  GemmParams local = p;
  void* args[] = {&local};
  return hipLaunchKernel(k, dim3(grid), dim3(kThreads), args, 0, stream);
}

hipError_t gemm_occupancy(int tile, bool out_bf16, bool vec, int* blocks_per_cu, int f8, bool deep) {
  const void* k = select_kernel(tile, out_bf16, vec, f8, deep);
  if (!k) return hipErrorInvalidValue;
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, k, kThreads, 0);
}

}  // namespace sfc
