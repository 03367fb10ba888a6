// Analytical choice of the block shape and of the number of K layers
// (Section III.B's fine-grained roofline, Eq. 1-4, used as in Section III.C,
// option 2: evaluate every decomposition and keep the fastest).
//
// The paper's model, per core: the critical path is the sum of the BRGEMM
// times on it, each max(G*gamma, beta*(S_A + S_B)) for the panels that come
// from slow memory (Eq. 1; Eq. 2-4 drop the panels already in fast memory),
// plus the reads and writes of C and, with several layers, of the C copies.
// On the GPU a "core" is a CU running `occ` persistent workgroups; one BRGEMM
// is one 64-deep block of one task; fast memory is the L2 of an XCD, which the
// workgroups of that XCD share, and slow memory is HBM.  With the interleaved
// schedule the tasks in flight on one XCD form a compact patch of the curve,
// about sqrt(P) x sqrt(P) blocks for P tasks, so per block a workgroup brings
// (S_A + S_B) / sqrt(P) bytes from HBM (each panel is fetched once per patch).
// Every candidate is evaluated with the same constants; the smallest time wins.
#pragma once
#include <cstdint>

namespace sfc {

// Calibration on MI355X (fast path, bf16 in, fp32 accumulate).
struct ModelConst {
  double flops_per_clk_cu = 4096.0 * 0.74;   // dense bf16 MFMA peak x achieved fraction (256x256)
  double rate[4] = {0.60, 0.80, 0.86, 1.0};  // per shape, relative to 256x256 (index: kT* order)
  double hbm_bytes_per_clk = 3500.0;         // whole chip, at the loaded shader clock
  double launch_clk = 10000.0;               // per kernel launch (about 5 us)
  int xcds = 8;
};

constexpr int kModelMaxLayers = 16;          // the candidates are c = 1, 2, 4, 8, 16

struct ModelChoice {
  int tile;          // kT* index
  int layers;        // effective layer count
  double clk;        // estimated time in shader clocks
};

// Best (tile, layers) for C[M x N] = A[M x K] B[K x N].  occ[t] = workgroups
// per CU of shape t (kT* index).  tile_fixed = -1 and layers_fixed = 0 leave
// the choice free; otherwise only the fixed value is evaluated.
ModelChoice model_choose(int64_t M, int64_t N, int64_t K, int out_bytes, int num_cus,
                         const int occ[4], int tile_fixed, int layers_fixed,
                         const ModelConst& k = ModelConst());

// Whether 256x256 blocks with a half-height strip (strip_width) in the last round
// take over from `ch`, the model's choice of 128x256 blocks in one layer: the model
// prices whole rounds of one shape only, and charges the 128x256 shape's rounds less
// than they take on a full chip.  The strip's two launches are estimated with
// the model's constants and have to win by 4.5 %, and with one round of whole
// blocks at least a quarter of a round has to be left over (a thin remainder costs
// a nearly empty round of 128x256 blocks little, the strip a launch and a round).
// Measured, 128x256 blocks -> 256x256 and strip (us): 6144x6144x4096 bf16 270 -> 244,
// f32 291 -> 265, fp8 153 -> 141; 5120x4096x8192 bf16 307 -> 277; 1300x14336x4096 160 ->
// 149; 3001x7003x5001 313 -> 259; 5500x4096x4096 171 -> 168.  Where the rule says no:
// 3000x7000x2048 89 -> 99, 2800x6144x4096 153 -> 180, 3300x6144x4096 164 -> 182.
// min_cols: what the strip's launch needs (min_columns); f8: nk counts the K blocks of
// fp8 operands.  Without a strip the model's choice stands.
bool strip_beats_128x256(int64_t M, int64_t N, int64_t nk, int out_bytes, int num_cus, const ModelChoice& ch,
                         int64_t min_cols = 1, bool f8 = false, const ModelConst& k = ModelConst());

// The small-block kernel (sfc_small.hip): blocks of 16*fm rows x 64 columns, `layers`
// ranges of K, every block and layer in flight at once (at most one per CU).
struct SmallChoice {
  int fm;            // 1, 2 or 4; 0: the curve kernel is the faster one
  int layers;
  double us;
};

// ca_layers 0 (free) or 1.  Measured on MI355X, calls of the C ABI back to back over
// rotating operands, against the curve kernel (us):
//   512x512x512 f32 8.2 -> 4.6, 333x517x421 bf16 10.8 -> 4.9, 1024^3 bf16 11.6 -> 8.4,
//   16x14336x4096 bf16 28.3 -> 25.7, 1x4096x4096 16.4 -> 10.0, 64x14336x4096 36.7 -> 30.8,
//   256x4096x4096 20.2 -> 17.2, 200x200x5999 f32 (one layer) 64.3 -> 19.0;
// and where the curve kernel stays: 16x16384x16384 92 (small 106), 512x512x32768 34
// (small 44), 1024x2048x512 8.6 (small 11.2: two rounds of workgroups).
SmallChoice small_choose(int64_t M, int64_t N, int64_t K, int out_bytes, int num_cus, int ca_layers);

}  // namespace sfc
