// Handles of the compiled GEMM kernels, one source file per block shape (so that
// they build in parallel).  ob: bf16 output, else fp32.  f8 as in launch_gemm.
#pragma once

namespace sfc {

const void* kernel_256x256_f32();
const void* kernel_256x256_bf16();
const void* kernel_256x128(bool ob);
const void* kernel_128x256(bool ob);
const void* kernel_128x128(bool ob);
const void* kernel_128x128_deep(bool ob);      // 4-deep ring
const void* kernel_f8_256x256(bool ob, int f8);
const void* kernel_f8_128x256(bool ob, int f8);
const void* kernel_any(int tile, bool ob);       // any alignment, 16-byte loads
const void* kernel_elements(int tile, bool ob);  // any alignment, element loads

}  // namespace sfc
