// Analytical choice of the block shape and the layer count (see sfc_model.h).
#include "sfc_model.h"

#include <cmath>

#include "sfc_params.h"
#include "sfc_validate.h"

namespace sfc {

namespace {

int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Estimated shader clocks of one candidate.  pad = output elements computed,
// ragged edges included (the first tie-breaker).
double candidate_clk(int64_t M, int64_t N, int64_t nk, int out_bytes, int num_cus, int occ, int t, int c,
                     const ModelConst& k, double* pad) {
  const int64_t bm = tile_bm(t), bn = tile_bn(t);
  const int64_t tasks = cdiv(M, bm) * cdiv(N, bn) * c;
  const int64_t slots = (int64_t)num_cus * occ;
  const int64_t rounds = cdiv(tasks, slots);
  const int64_t nb = cdiv(nk, c);                       // blocks of the longest layer
  const int64_t active = tasks < slots ? tasks : slots;  // workgroups streaming at once
  // one BRGEMM (64-deep block): G flops, panels S_A + S_B bytes
  const double g = 2.0 * (double)bm * (double)bn * 64.0;
  const double s_ab = 2.0 * 64.0 * (double)(bm + bn);
  // gamma: a workgroup gets 1/w of its CU's MFMA rate, w the workgroups that
  // share the CU: the dispatcher spreads a grid over the CUs before it puts a
  // second workgroup on one (and a grid of at most one 128x128 block per CU
  // runs the one-per-CU kernel)
  int64_t w = cdiv(active, num_cus);
  if (w > occ) w = occ;
  if (w < 1) w = 1;
  const double t_compute = g * (double)w / (k.flops_per_clk_cu * k.rate[t]);
  // beta: HBM shared by the active workgroups; each panel read once per XCD patch
  double patch = (double)active / (double)k.xcds;
  if (patch < 1.0) patch = 1.0;
  const double t_memory = s_ab / std::sqrt(patch) * (double)active / k.hbm_bytes_per_clk;
  const double t_block = t_compute > t_memory ? t_compute : t_memory;   // Eq. 1
  // C written once; with layers, the copies written and read back, then C
  const double mn = (double)M * (double)N;
  const double c_bytes = c == 1 ? mn * out_bytes : 2.0 * c * mn * 4.0 + mn * out_bytes;
  *pad = (double)tasks * (double)(bm * bn);
  return k.launch_clk * (c == 1 ? 1.0 : 2.0) + (double)rounds * (double)nb * t_block +
         c_bytes / k.hbm_bytes_per_clk;
}

}  // namespace

ModelChoice model_choose(int64_t M, int64_t N, int64_t K, int out_bytes, int num_cus, const int occ[4],
                         int tile_fixed, int layers_fixed, const ModelConst& k) {
  static const int order[4] = {kT256x256, kT128x256, kT256x128, kT128x128};
  const int64_t nk = K > 0 ? cdiv(K, 64) : 0;
  ModelChoice best{kT256x256, 1, 1e300};
  double best_pad = 1e300;
  for (int i = 0; i < 4; ++i) {
    const int t = order[i];
    if (tile_fixed >= 0 && t != tile_fixed) continue;
    int last_c = 0;
    for (int c0 = 1; c0 <= kModelMaxLayers; c0 *= 2) {
      if (layers_fixed > 0 && c0 != 1) break;
      int c = layers_fixed > 0 ? layers_fixed : c0;
      if (c > nk) c = nk > 0 ? (int)nk : 1;               // effective layer count
      if (c == last_c) continue;
      last_c = c;
      double pad = 0.0;
      const double clk = candidate_clk(M, N, nk, out_bytes, num_cus, occ[t] < 1 ? 1 : occ[t], t, c, k, &pad);
      // relative tolerance: candidates this close are ties, settled by the
      // padded work, then by the order of evaluation (shape order above, then
      // ascending layer counts)
      const double tol = 1e-9 * best.clk;
      const bool take = clk < best.clk - tol || (clk <= best.clk + tol && pad < best_pad);
      if (take) {
        best = ModelChoice{t, c, clk};
        best_pad = pad;
      }
    }
  }
  return best;
}

bool strip_beats_128x256(int64_t M, int64_t N, int64_t nk, int out_bytes, int num_cus, const ModelChoice& ch,
                         int64_t min_cols, bool f8, const ModelConst& k) {
  if (ch.tile != kT128x256 || ch.layers != 1) return false;
  const int64_t gm = cdiv(M, 256), gn = cdiv(N, 256);
  const int w = strip_width(M, N, 256, 256, num_cus, num_cus, min_cols, f8 ? nk : 0);
  if (w == 0) return false;
  const int64_t full = gm * gn / num_cus, left = gm * gn % num_cus;
  if (full < 2 && 4 * left < num_cus) return false;
  const double g = 2.0 * 256.0 * 256.0 * 64.0 / k.flops_per_clk_cu;
  const double t_main = g / k.rate[kT256x256], t_strip = 0.5 * g / k.rate[kT128x256];
  const double rounds = (double)cdiv(gm * (gn - w), num_cus);
  const double clk = 2.0 * k.launch_clk + (double)nk * (rounds * t_main + t_strip) +
                     (double)M * (double)N * out_bytes / k.hbm_bytes_per_clk;
  return clk < 0.955 * ch.clk;
}

// Both kernels' times in microseconds, from fits to about 70 measured calls (M, N
// 1 .. 2048, K 8 .. 65536): most within 15 %.  The small-block kernel takes 3 us for the
// launch, the first loads and the end; `round` per 256 of K (64 per wave; the first
// value with few workgroups, the second with one on every CU; cold operands, too
// large to lie in a cache, arrive more slowly); operands from memory at 5.2 TB/s
// (128-byte row segments of B; the curve kernel's 512-byte ones reach 6.0); with
// several layers 2.2 us for the count's round trip and the last workgroup's read
// of a block's copies at about 30 bytes per ns.
// Past 150 MB the small-block kernel slows down where a workgroup has many rounds
// (curve kernel in 4 or 8 layers -> small, us: 16x12520x7656 40.0 -> 44.9, 15x14200x8200
// 44.6 -> 48.2, 56x14848x9288 61.9 -> 73.6; below 26 rounds the small one wins: 3x16208x5728
// 35.7 -> 31.5, 15x14624x6224 37.6 -> 34.2; against 16 layers, whose tasks fill the
// curve kernel's rounds badly, up to 40: 3x12256x8552 50.5 -> 39.1, 13x11768x12040 64.2 ->
// 66.0), unless one 16-row block reads whole 128-byte lines (16x13376x6840 37.3 -> 32.8,
// 12x11840x12352 64.5 -> 49.2), and where rows of B lie a multiple of 4 KB apart, which puts a block's segments
// on few channels (16x16384x6144 40.3 -> 41.7, 16x16384x8192 50.9 -> 54.5).
SmallChoice small_choose(int64_t M, int64_t N, int64_t K, int out_bytes, int num_cus, int ca_layers) {
  SmallChoice best{0, 1, 1e300};
  // more blocks than CUs of the tallest shape (a second round of workgroups would
  // cost more than the curve kernel's larger blocks)
  if (K < 8 || cdiv(M, 64) * cdiv(N, 64) > num_cus) return best;
  static const int occ[4] = {2, 1, 1, 1};
  const ModelChoice old = model_choose(M, N, K, out_bytes, num_cus, occ, -1, ca_layers);
  const double in_bytes = 2.0 * ((double)M * (double)K + (double)K * (double)N);
  const double mn = (double)M * (double)N;
  double old_us = old.clk / 2100.0;
  const double old_mem = 4.0 + in_bytes / 6.0e6 + (old.layers > 1 ? 4.0 + old.layers * mn * 8.0 / 4.0e6 : 0.0);
  if (old_mem > old_us) old_us = old_mem;
  static const double kLow[3] = {0.42, 0.50, 0.62}, kHigh[3] = {0.60, 0.66, 0.86}, kCold[3] = {0.90, 0.95, 1.05},
                      kLong[3] = {1.40, 1.48, 1.56};
  const bool large = in_bytes > 150e6;
  const bool whole_lines = N % 64 == 0 && N % 1024 != 0;
  const double stream = large && old.layers <= 4 && N % 2048 == 0 ? 4.9e6 : 5.2e6;
  const int64_t nk = cdiv(K, 64);
  for (int i = 0; i < 3; ++i) {
    const int fm = 1 << i;
    const int64_t tiles = cdiv(M, 16 * fm) * cdiv(N, 64);
    // layers only where the curve kernel would use them too
    const int max_layers = ca_layers == 0 && old.layers > 1 ? kModelMaxLayers : 1;
    for (int c = 1; c <= max_layers && tiles * c <= num_cus; c *= 2) {
      if (c > 1 && nk < 8 * c) break;               // at least two stages per wave
      const double rounds = (double)cdiv(nk, 4 * c);
      const double busy = (double)(tiles * c) / (double)num_cus;
      double per = kLow[i] + (kHigh[i] - kLow[i]) * busy;
      const bool many = large && rounds > (old.layers > 8 ? 40.0 : 25.0) && !(i == 0 && whole_lines);
      const double arrive = many ? kLong[i] : in_bytes > 60e6 ? 1.3 * kCold[i] : in_bytes > 16e6 ? kCold[i] : 0.0;
      if (per < arrive) per = arrive;
      double us = rounds * per;
      if (us < in_bytes / stream) us = in_bytes / stream;
      us += 3.0 + mn * out_bytes / 4.0e6;
      if (c > 1) us += 2.2 + (double)(fm * c) * 4096.0 / 30.0e3;
      if (us < best.us) best = SmallChoice{fm, c, us};
    }
  }
  if (best.us >= old_us) best.fm = 0;
  return best;
}

}  // namespace sfc
