// Choice and launch of the compiled GEMM kernels.
#include "sfc_gemm_variants.h"
#include "sfc_params.h"

namespace sfc {

// fp8 operands run on 256x256 or 128x256 blocks with ring loads only; the deep
// ring exists for 128x128 blocks only.
static const void* select_kernel(const Variant& v) {
  if (v.f8) {
    if (v.loads != kLoadRing || v.deep) return nullptr;
    if (v.tile == kT256x256) return kernel_f8_256x256(v.out_bf16, v.f8);
    return v.tile == kT128x256 ? kernel_f8_128x256(v.out_bf16, v.f8) : nullptr;
  }
  if (v.deep) return v.tile == kT128x128 && v.loads == kLoadRing ? kernel_128x128_deep(v.out_bf16) : nullptr;
  if (v.loads == kLoadAny) return kernel_any(v.tile, v.out_bf16);
  if (v.loads == kLoadElements) return kernel_elements(v.tile, v.out_bf16);
  switch (v.tile) {
    case kT128x128: return kernel_128x128(v.out_bf16);
    case kT256x128: return kernel_256x128(v.out_bf16);
    case kT128x256: return kernel_128x256(v.out_bf16);
    case kT256x256: return v.out_bf16 ? kernel_256x256_bf16() : kernel_256x256_f32();
    default: return nullptr;
  }
}

constexpr int kThreads = 256;   // every kernel: 4 waves

hipError_t launch_gemm(const Variant& v, const GemmParams& p, int grid, hipStream_t stream) {
  const void* k = select_kernel(v);
  if (!k) return hipErrorInvalidValue;
  GemmParams local = p;
  void* args[] = {&local};
  return hipLaunchKernel(k, dim3(grid), dim3(kThreads), args, 0, stream);
}

hipError_t gemm_occupancy(const Variant& v, int* blocks_per_cu) {
  const void* k = select_kernel(v);
  if (!k) return hipErrorInvalidValue;
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, k, kThreads, 0);
}

}  // namespace sfc
