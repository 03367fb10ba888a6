// Internal interface between the C-ABI layer and the HIP kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sfc {

constexpr int kBK = 64;          // depth of one K block (the paper's bk)

enum TileId { kT128x128 = 0, kT256x128 = 1, kT128x256 = 2, kT256x256 = 3, kNumTiles = 4 };

inline int tile_bm(int t) { return (t == kT256x128 || t == kT256x256) ? 256 : 128; }
inline int tile_bn(int t) { return (t == kT128x256 || t == kT256x256) ? 256 : 128; }

struct GemmParams {
  int64_t M, N, K;
  const uint16_t* A;
  int64_t lda;
  const uint16_t* B;
  int64_t ldb;
  void* out;                 // C (layers == 1) or the fp32 workspace (layers > 1)
  int64_t ldo;               // leading dimension of `out`
  int64_t out_layer_stride;  // elements between layer copies of `out` (0 when layers == 1)
  const int32_t* table;      // gm*gn curve positions -> im*gn + in
  int gm, gn;
  int layers;                // c_eff
  int nk;                    // ceil(K / kBK)
  int64_t tasks;             // gm * gn * layers
  int sched;                 // SFC_SCHED_*
  // Fused reduction (layers > 1 and counters != nullptr): the workgroup that
  // finishes a block's last layer copy sums the copies into C itself.
  int c_bf16;                // C holds bf16 (else fp32)
  int32_t* counters;         // per block (im*gn + in): layer copies finished; zero between launches
  void* C;                   // the final output
  int64_t ldc;
};

// Curve table of a gm x gn grid into dev_out (gm*gn int32), order = SFC_ORDER_*.
hipError_t launch_sfc_order(int gm, int gn, int order, int32_t* dev_out, hipStream_t stream);

// How a kernel brings its operands into LDS.
enum Loads {
  kLoadElements = 0,  // element by element (K or N below 8, or leading dimensions past the 32-bit offsets)
  kLoadRing = 1,      // 16-byte aligned rows, straight from memory into LDS (vector_loads_ok)
  kLoadAny = 2,       // the same at any alignment, a ragged last K block through registers (any_loads_ok)
};

// One compiled GEMM kernel.
struct Variant {
  int tile = kT128x128;
  bool out_bf16 = false;      // epilogue: bf16 C, else fp32
  int loads = kLoadElements;
  // 0: bf16 operands; 1 + a + 2b: A and B hold OCP fp8 bytes of format a and b
  // (0 E4M3, 1 E5M2; lda, ldb in elements = bytes), ring loads only
  int f8 = 0;
  // 128x128 blocks on the ring with 4-deep prefetch (one workgroup per CU),
  // for grids of at most one block per CU
  bool deep = false;
};

// Persistent GEMM.
hipError_t launch_gemm(const Variant& v, const GemmParams& p, int grid, hipStream_t stream);
// Workgroups of the given kernel that fit on one CU.
hipError_t gemm_occupancy(const Variant& v, int* blocks_per_cu);

// One launch of the small-block kernel (sfc_small.hip): blocks of 16*fm rows
// (fm = 1, 2, 4) x 64 columns, `layers` ranges of K.
struct SmallParams {
  int M, N, K;
  int gm, gn, layers;
  int steps;                 // whole 32-deep steps of K that the LDS ring takes
  int tail;                  // 1: one more step, through registers
  const uint16_t* A;
  int64_t lda;
  const uint16_t* B;
  int64_t ldb;
  void* C;
  int64_t ldc;
  float* W;                  // layers > 1: gm*gn*layers copies of 16*fm x 64
  int32_t* counters;         // layers > 1: one per block, zero between launches
};
hipError_t launch_small(const SmallParams& p, int fm, bool out_bf16, hipStream_t stream);

// p[0 .. n) = v (a fill kernel: usable where a memset node is not wanted).
hipError_t launch_fill_i32(int32_t* p, int64_t n, int32_t v, hipStream_t stream);

// C[i][j] = sum_l W[l][i][j] (ascending l, fp32), W dense M x N per layer.
hipError_t launch_reduce(const float* W, int layers, int64_t M, int64_t N, void* C, int64_t ldc,
                         bool out_bf16, hipStream_t stream);

// Register-only MFMA probe (256 workgroups x 4 waves); dev_out holds
// 256*256 + 256 floats (the last 256: shader clock per workgroup in MHz).
hipError_t run_mfma_probe(int random_operands, int iters, float* dev_out, double* ms);

}  // namespace sfc
