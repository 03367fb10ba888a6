// Small products and few rows (a decode step's tokens times weights): the
// calls whose time is latency, or the one read of B, rather than MFMA work.
//
// One workgroup computes a block of 16*FM rows (FM = 1, 2, 4) x 64 columns.  Its 4
// waves split the block's K range between them, 64-deep stages dealt in turn
// (wave w takes stages w, w+4, ..), and each wave runs on its own: a private ring
// of S stage slots in LDS, filled straight from memory, no barrier until the
// 4 partial blocks are added (waves ascending, fp32).  With several layers each
// layer contracts its own range of stages; the copies are summed, layers
// ascending, by the last workgroup of a block to finish (no workgroup waits).
//
//   * A of a stage is [16*FM][64], whole 128-byte lines, stored as the A blocks of
//     sfc_gemm_kernel.h (a_off): with 64-byte pieces the lines of A took a third
//     of the loads' cache line requests;
//   * B of a stage is [64][64]: whole 128-byte row segments.  Chunk c (8 columns)
//     of row k is stored at chunk c ^ (2*bit1(k) + 4*bit3(k)); a pass of the
//     transposing read touches rows k0..k0+3 and k0+8..k0+11 at two chunks, and
//     the swizzle puts those 16 pieces on the 16 16-byte bank groups;
//   * loads for stages past the range go out with empty descriptors (zeros, no
//     memory is read), so every stage waits for the same count.
//
// Bound: few rows read B once, 128-byte row segments at 5.2 TB/s (16x14336x4096:
// 28.1 -> 25.7 us; the curve kernel's 128-row blocks needed 4 layer copies and a
// reduction launch for the same parallelism).  Small products are a chain of
// launch (~2 us), first loads (~1 us), rounds of 256 of K (0.4-0.9 us) and the sum of
// the partial blocks.  Calls of the C ABI back to back: 512x512x512 f32 8.2 -> 4.6 us,
// 333x517x421 bf16 10.8 -> 4.9 (5.1 both in a kernel trace, which spaces the launches).
//
// Rows of any alignment (see the notes at any_tail in sfc_gemm_kernel.h): the ring
// takes whole stages; where K is no multiple of 32, or a last chunk of a row of B
// would run past N, the last stage's operands are loaded into registers by the
// wave whose turn it is, before its ring starts.
#include "sfc_gemm_kernel.h"

namespace sfc {

constexpr int kSmallN = 64;      // columns of a block

template <int FM, int S>
struct SmallRing {
  static constexpr int A_BYTES = FM * 2048, B_BYTES = 64 * kSmallN * 2;
  static constexpr int SLOT = A_BYTES + B_BYTES;
  static constexpr int WAVE = S * SLOT;                // bytes of a wave's ring
  static constexpr int LOADS = 2 * FM + 8;               // loads per stage and wave
  static constexpr int RS = kSmallN * 4 + 16;          // row stride of a partial block (bytes)
  static_assert((S - 1) * LOADS <= 63, "vmcnt range");
  static_assert(16 * FM * RS <= WAVE, "a partial block fits its wave's ring");
  static_assert(4 * WAVE <= 160 * 1024, "LDS of one CU");
};

// FM loads sharing M0, instruction offsets 0, 1024, ..
template <int N>
__device__ __forceinline__ void small_dma(i32x4 rsrc, uint32_t m0_value, const int* v) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
               :: "s"(m0_value), "v"(v[0]), "s"(rsrc) : "memory");
  if constexpr (N > 1)
    asm volatile("buffer_load_dwordx4 %0, %1, 0 offen offset:1024 lds" :: "v"(v[1]), "s"(rsrc) : "memory");
  if constexpr (N > 2) {
    asm volatile("buffer_load_dwordx4 %0, %1, 0 offen offset:2048 lds" :: "v"(v[2]), "s"(rsrc) : "memory");
    asm volatile("buffer_load_dwordx4 %0, %1, 0 offen offset:3072 lds" :: "v"(v[3]), "s"(rsrc) : "memory");
  }
}

// 16 bytes of fp32 or 8 bytes of bf16 at element alignment.
struct __attribute__((packed, aligned(4))) F32x4Any { f32x4 v; };
struct __attribute__((packed, aligned(2))) Bf16x4Any { bf16x4 v; };

// Columns c .. c+3 of row r of C (those inside it).
template <bool OB>
__device__ __forceinline__ void small_store(const SmallParams& p, int r, int c, const f32x4& v) {
  if (r >= p.M || c >= p.N) return;
  const int64_t at = (int64_t)r * p.ldc + c;
  if constexpr (OB) {
    __bf16* dst = reinterpret_cast<__bf16*>(p.C) + at;
    const bf16x4 b = {(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3]};
    if (c + 4 <= p.N) reinterpret_cast<Bf16x4Any*>(dst)->v = b;
    else
#pragma unroll
      for (int e = 0; e < 3; ++e)
        if (c + e < p.N) dst[e] = b[e];
  } else {
    float* dst = reinterpret_cast<float*>(p.C) + at;
    if (c + 4 <= p.N) reinterpret_cast<F32x4Any*>(dst)->v = v;
    else
#pragma unroll
      for (int e = 0; e < 3; ++e)
        if (c + e < p.N) dst[e] = v[e];
  }
}

// 16 bytes read at device scope: past this chiplet's caches, which may hold older
// lines of the copies, without invalidating them.
__device__ __forceinline__ f32x4 load16_agent(const float* p) {
  typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));
  uint64_t* q = const_cast<uint64_t*>(reinterpret_cast<const uint64_t*>(p));
  const u64x2 w = {__hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
                   __hip_atomic_load(q + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)};
  return __builtin_bit_cast(f32x4, w);
}

template <int FM, int S, bool OB>
__global__ __launch_bounds__(256, 1) void sfc_small_kernel(SmallParams p) {
  using R = SmallRing<FM, S>;
  __shared__ __attribute__((aligned(16))) unsigned char smem[4 * R::WAVE];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // consecutive ranks (one chiplet) share the block's columns of B
  const int cells = p.gm * p.gn;
  const int rank = xcd_rank(blockIdx.x, gridDim.x);
  const int layer = rank / cells, cell = rank - layer * cells;
  const int in = cell / p.gm, im = cell - in * p.gm;
  const int m0 = im * 16 * FM, n0 = in * kSmallN;
  // 64-deep stages of this layer.  The ring takes p.steps whole 32-deep steps of K
  // (its last stage may be half a stage); one more step may go through registers.
  const int all = (p.steps + p.tail + 1) >> 1;
  const int st0 = (int)((int64_t)layer * all / p.layers), st1 = (int)((int64_t)(layer + 1) * all / p.layers);
  const int ring_all = (p.steps + 1) >> 1;
  const int ring1 = st1 < ring_all ? st1 : ring_all;
  const int n = (ring1 - st0 - wave + 3) >> 2;       // this wave's ring stages (may be <= 0)
  // ring stage (of this wave) that is half a stage
  const int half = (p.steps & 1) && ring1 == ring_all && ((ring_all - 1 - st0) & 3) == wave ? n - 1 : -1;
  const bool tail = p.tail && st1 == all && ((all - st0) & 3) == wave;

  // last stage in registers: A fragment i and B fragment j as the MFMA takes them
  bf16x8 ta[FM], tb[4];
  if (tail) {
    const int k0 = p.steps * 32, kc = k0 + 8 * (lane >> 4);
    const int ka = kc < p.K - 8 ? kc : p.K - 8;
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      const int r = m0 + 16 * i + (lane & 15);
      const u32x4 v = reinterpret_cast<const Chunk16*>(p.A + (int64_t)(r < p.M ? r : p.M - 1) * p.lda + ka)->v;
      ta[i] = __builtin_bit_cast(bf16x8, shift_chunk(v, kc - ka));
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int c = n0 + 16 * j + (lane & 15);
      const uint16_t* col = p.B + (c < p.N ? c : p.N - 1);
      i16x8 v;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int k = kc + e;
        const uint16_t x = col[(int64_t)(k < p.K ? k : p.K - 1) * p.ldb];
        v[e] = k < p.K ? (short)x : (short)0;
      }
      tb[j] = __builtin_bit_cast(bf16x8, v);
    }
  }

  f32x4 acc[FM][4];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  const uint32_t ring = lds_addr(smem) + (uint32_t)(wave * R::WAVE);
  if (n > 0) {
    int av[2 * FM], bv[8];
#pragma unroll
    for (int i = 0; i < 2 * FM; ++i) {
      const int r = 8 * i + (lane >> 3);
      const int c = (lane & 7) ^ ((r >> 1) & 7);
      av[i] = m0 + r < p.M ? (int)(r * p.lda * 2) + 16 * c + kBias - 1024 * (i & 3) : kOobOffset;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int k = 8 * i + (lane >> 3);
      const int c = (lane & 7) ^ (((k >> 1) & 1) * 2 + ((k >> 3) & 1) * 4);
      bv[i] = n0 + 8 * c < p.N ? (int)(k * p.ldb * 2) + 16 * c + kBias - 1024 * (i & 3) : kOobOffset;
    }
    const uint32_t ar = (uint32_t)(a_off(lane & 15, lane >> 4) * 2);   // A fragment 0 of step 0; step 1: chunk ^ 4
    // fragment reads: B fragment j, row 8*(l/16) + (l%16)/4 of the stage
    uint32_t br[4];
    {
      const int g = lane >> 4, jj = lane & 15;
      const int k = 8 * g + (jj >> 2), f = ((k >> 1) & 1) * 2 + (g & 1) * 4;
#pragma unroll
      for (int j = 0; j < 4; ++j)
        br[j] = (uint32_t)(R::A_BYTES + k * 128 + (((2 * j + ((jj >> 1) & 1)) ^ f) << 4) + (jj & 1) * 8);
    }
    uint64_t a_at = reinterpret_cast<uint64_t>(p.A + m0 * p.lda + (int64_t)(st0 + wave) * 64) - kBias;
    uint64_t b_at = reinterpret_cast<uint64_t>(p.B + (int64_t)(st0 + wave) * 64 * p.ldb + n0) - kBias;
    const uint64_t b_step = (uint64_t)p.ldb * 2 * 256;   // 4 stages of 64 rows
    int issued = 0;
    uint32_t fill = ring;
    auto issue = [&]() {
      const uint32_t lim = issued < n ? (uint32_t)kOobOffset : 0u;
      if (issued == half) {
        // half a stage: the chunks of A and the rows of B past it read zeros (by
        // lanes: a range of B's rows would cut the chunk that runs past N)
#pragma unroll
        for (int i = 0; i < 2 * FM; ++i)
          if (((lane & 7) ^ (((8 * i + (lane >> 3)) >> 1) & 7)) >= 4) av[i] = kOobOffset;
#pragma unroll
        for (int i = 4; i < 8; ++i) bv[i] = kOobOffset;
      }
      const i32x4 ra = make_rsrc_addr(a_at, lim), rb = make_rsrc_addr(b_at, lim);
#pragma unroll
      for (int i = 0; i < 2 * FM; i += 4) small_dma<(FM == 1 ? 2 : 4)>(ra, fill + (uint32_t)(i * 1024), av + i);
      small_dma<4>(rb, fill + R::A_BYTES, bv);
      small_dma<4>(rb, fill + R::A_BYTES + 4096, bv + 4);
      a_at += 4 * 64 * 2;
      b_at += b_step;
      ++issued;
    };
#pragma unroll
    for (int s = 0; s < S; ++s) {
      fill = ring + (uint32_t)(s * R::SLOT);
      issue();
    }
    uint32_t slot = 0;
    for (int it = 0; it < n; ++it) {
      fill = ring + slot;
      wait_vmem_at_most<(S - 1) * R::LOADS>();
      bf16x8 fa[2][FM], fb[2][4];
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
          fa[ks][i] = *(lds_bf16x8*)(uintptr_t)(fill + (ar ^ (uint32_t)(64 * ks)) + (uint32_t)(i * 2048));
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const uint32_t at = fill + br[j] + (uint32_t)(4096 * ks);
          const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(uintptr_t)at);
          const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(uintptr_t)(at + 512));
          const i16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
          fb[ks][j] = __builtin_bit_cast(bf16x8, v);
        }
      }
      wait_lds_all();          // the slot has been read: load into it
      issue();
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[ks][j], fa[ks][i], acc[i][j], 0, 0, 0);
      slot = slot + R::SLOT == (uint32_t)R::WAVE ? 0u : slot + R::SLOT;
    }
    wait_vmem_at_most<0>();    // the empty loads have written their zeros
  }
  if (tail) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(tb[j], ta[i], acc[i][j], 0, 0, 0);
  }

  // the waves' partial blocks, added in ascending order
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
      lds_write16(ring + (uint32_t)((16 * i + (lane & 15)) * R::RS + (16 * j + 4 * (lane >> 4)) * 4),
                  __builtin_bit_cast(u32x4, acc[i][j]));
  __syncthreads();
  const int row = tid >> 4, c4 = (tid & 15) * 4;      // 4 columns of rows row, row + 16, ..
  f32x4 sum[FM];
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    const uint32_t at = lds_addr(smem) + (uint32_t)((16 * i + row) * R::RS + c4 * 4);
    sum[i] = __builtin_bit_cast(f32x4, lds_read16(at));
#pragma unroll
    for (int w = 1; w < 4; ++w) {
      const f32x4 v = __builtin_bit_cast(f32x4, lds_read16(at + (uint32_t)(w * R::WAVE)));
      sum[i][0] += v[0]; sum[i][1] += v[1]; sum[i][2] += v[2]; sum[i][3] += v[3];
    }
  }
  if (p.layers == 1) {
#pragma unroll
    for (int i = 0; i < FM; ++i) small_store<OB>(p, m0 + 16 * i + row, n0 + c4, sum[i]);
    return;
  }

  // layer copies: [cell][layer][16*FM][64] fp32, stored at device scope (written
  // through this chiplet's L2); the last workgroup of the cell to arrive sums
  // them, layers ascending
  constexpr int TILE = 16 * FM * kSmallN;
  float* own = p.W + ((int64_t)cell * p.layers + layer) * TILE + row * kSmallN + c4;
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));
    const u64x2 w = __builtin_bit_cast(u64x2, sum[i]);
    uint64_t* q = reinterpret_cast<uint64_t*>(own + i * 16 * kSmallN);
    __hip_atomic_store(q, w[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(q + 1, w[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  int* flag = reinterpret_cast<int*>(smem);
  if (tid == 0) *flag = __hip_atomic_fetch_add(p.counters + cell, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  if (*flag != p.layers - 1) return;
  asm volatile("" ::: "memory");   // the loads below come after the count
  const float* all_copies = p.W + (int64_t)cell * p.layers * TILE + row * kSmallN + c4;
#pragma unroll
  for (int i = 0; i < FM; ++i) sum[i] = load16_agent(all_copies + i * 16 * kSmallN);
#pragma unroll 4
  for (int l = 1; l < p.layers; ++l)
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      const f32x4 v = load16_agent(all_copies + (int64_t)l * TILE + i * 16 * kSmallN);
      sum[i][0] += v[0]; sum[i][1] += v[1]; sum[i][2] += v[2]; sum[i][3] += v[3];
    }
#pragma unroll
  for (int i = 0; i < FM; ++i) small_store<OB>(p, m0 + 16 * i + row, n0 + c4, sum[i]);
  if (tid == 0) __hip_atomic_store(p.counters + cell, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int FM, int S>
static const void* small_ptr(bool ob) {
  return ob ? reinterpret_cast<const void*>(&sfc_small_kernel<FM, S, true>)
            : reinterpret_cast<const void*>(&sfc_small_kernel<FM, S, false>);
}

hipError_t launch_small(const SmallParams& p, int fm, bool out_bf16, hipStream_t stream) {
  const void* k = fm == 1 ? small_ptr<1, 2>(out_bf16) : fm == 2 ? small_ptr<2, 2>(out_bf16) : small_ptr<4, 2>(out_bf16);
  SmallParams local = p;
  void* args[] = {&local};
  return hipLaunchKernel(k, dim3((unsigned)(p.gm * p.gn * p.layers)), dim3(256), args, 0, stream);
}

}  // namespace sfc
