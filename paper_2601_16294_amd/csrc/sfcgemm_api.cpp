// C ABI of the SFC-CA GEMM (declarations and contracts in include/sfcgemm.h).
//
// Host-side duties: argument checks (before any HIP call), choice of the block
// shape, the per-device cache of curve tables (built once per grid on the
// device and kept), the per-stream internal workspace for layer copies and
// arrival counters, and the launches.  Nothing here computes any part of the
// product.  No entry point synchronises the device or a stream: new curve
// tables and workspaces are made stream-ordered (events, hipMallocAsync /
// hipFreeAsync).
#include <hip/hip_runtime.h>

#include <map>
#include <mutex>
#include <string>
#include <tuple>

#include "sfc_model.h"
#include "sfc_params.h"
#include "sfc_validate.h"
#include "sfcgemm.h"

namespace {

thread_local std::string g_last_error;

// A curve table on the device, written by a kernel on the stream of the call
// that first needed it; `ready` marks its completion for calls on other streams.
struct Table {
  int32_t* d = nullptr;
  hipEvent_t ready = nullptr;
  bool done = false;        // `ready` has been seen complete
};

// Layer copies of calls that pass no workspace, and arrival counters of reductions
// inside a launch.
struct LayerMem {
  void* ws = nullptr;
  size_t ws_bytes = 0;
  int32_t* counters = nullptr;
  int64_t n_counters = 0;
};

// Library-owned memory of one stream.  Calls on different streams never share it.
// Calls that run at once use `eager`: only work on that stream touches it, it grows
// stream-ordered, and its counters are zero between launches.  Calls recorded into
// a graph use `captured`: the graph keeps the addresses for its replays, so this
// memory is never freed (a larger buffer joins the old one and is at least twice
// its size, so all of them stay below twice the last), is no graph's own (the next
// capture and other graphs use it too), and no replay, on whatever stream, shares
// copies or counters with calls that run at once.
struct StreamMem {
  LayerMem eager, captured;
};

struct DeviceState {
  std::map<std::tuple<int, int, int>, Table> tables;   // (gm, gn, order) -> device table
  std::map<std::tuple<int, int, int>, int32_t*> captured_tables;   // those that graphs write themselves
  std::map<hipStream_t, StreamMem> streams;
  char* scratch = nullptr;   // this device's copy of `scratch` (see sfc_gemm_noalloc_ex)
  int num_cus = 0;
  int occupancy[sfc::kNumTiles][2][3][2] = {};               // [tile][bf16 out][loads][fp8 in], 0 = unknown
  int occupancy_deep[2] = {};                                  // 4-deep 128x128 ring, [bf16 out]
};

std::mutex g_mu;
std::map<int, DeviceState> g_devices;

int set_error(int code, const std::string& msg) {
  g_last_error = msg;
  return code;
}

int hip_fail(hipError_t e, const char* where) {
  return set_error(SFC_ERR_HIP, std::string(where) + ": " + hipGetErrorString(e));
}

// Must be called with g_mu held.
int device_state(DeviceState** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  DeviceState& st = g_devices[dev];
  if (st.num_cus == 0) {
    int cus = 0;
    e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return hip_fail(e, "hipDeviceGetAttribute");
    st.num_cus = cus;
  }
  *out = &st;
  return SFC_OK;
}

// Whether calls on `stream` are being recorded into a graph.
bool is_captured(hipStream_t stream) {
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(stream, &cap) != hipSuccess) {
    (void)hipGetLastError();   // not an error: do not leave it for the next check
    return false;
  }
  return cap != hipStreamCaptureStatusNone;
}

// The relaxed capture mode of this thread: allocations and event queries are refused
// while a stream is captured in the other modes.
struct RelaxedCapture {
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  hipError_t e;
  RelaxedCapture() { e = hipThreadExchangeStreamCaptureMode(&mode); }
  ~RelaxedCapture() {
    if (e == hipSuccess) (void)hipThreadExchangeStreamCaptureMode(&mode);
  }
};

// Memory for a captured call: a plain allocation (one in stream order would become a
// node of the graph and its memory the graph's).
hipError_t captured_malloc(void** out, size_t bytes) {
  RelaxedCapture relaxed;
  return relaxed.e != hipSuccess ? relaxed.e : hipMalloc(out, bytes);
}

// Curve table of a gm x gn grid on the current device.  The first call for a
// grid allocates it and enqueues the generator on `stream` (no wait); a later
// call on another stream waits for that kernel on the device, until the table
// is known to be complete.  A call that is recorded into a graph before that cannot
// wait for it: it records the generator too, into a table that only recorded calls
// use (each replay writes the same values).  Must be called with g_mu held.
int get_table(DeviceState& st, int gm, int gn, int order, hipStream_t stream, const int32_t** out) {
  auto key = std::make_tuple(gm, gn, order);
  auto it = st.tables.find(key);
  const bool known = it != st.tables.end();
  if (known && it->second.done) {
    *out = it->second.d;
    return SFC_OK;
  }
  const bool cap = is_captured(stream);
  if (known) {
    Table& t = it->second;
    hipError_t e;
    {
      RelaxedCapture relaxed;
      e = hipEventQuery(t.ready);
    }
    if (e == hipSuccess) {
      t.done = true;
    } else if (e == hipErrorNotReady) {
      (void)hipGetLastError();   // not an error: do not leave it for the next check
      if (!cap) e = hipStreamWaitEvent(stream, t.ready, 0);
      if (!cap && e != hipSuccess) return hip_fail(e, "hipStreamWaitEvent(curve table)");
    } else {
      return hip_fail(e, "hipEventQuery(curve table)");
    }
    if (t.done || !cap) {
      *out = t.d;
      return SFC_OK;
    }
  }
  if (cap) {
    int32_t*& d = st.captured_tables[key];
    if (!d) {
      void* p = nullptr;
      hipError_t e = captured_malloc(&p, sizeof(int32_t) * (size_t)gm * (size_t)gn);
      if (e != hipSuccess) return hip_fail(e, "hipMalloc(curve table of captured calls)");
      d = static_cast<int32_t*>(p);
    }
    hipError_t e = sfc::launch_sfc_order(gm, gn, order, d, stream);
    if (e != hipSuccess) return hip_fail(e, "curve table");
    *out = d;
    return SFC_OK;
  }
  Table t;
  hipError_t e = hipMalloc(&t.d, sizeof(int32_t) * (size_t)gm * (size_t)gn);
  if (e != hipSuccess) return hip_fail(e, "hipMalloc(curve table)");
  e = sfc::launch_sfc_order(gm, gn, order, t.d, stream);
  if (e == hipSuccess) e = hipEventCreateWithFlags(&t.ready, hipEventDisableTiming);
  if (e == hipSuccess) e = hipEventRecord(t.ready, stream);
  if (e != hipSuccess) {
    // the generator may be queued: the table is kept (never used) rather than freed under it
    return hip_fail(e, "curve table");
  }
  st.tables[key] = t;
  *out = t.d;
  return SFC_OK;
}

// At least `bytes` of layer workspace owned by `stream`.  Outside a capture a
// smaller buffer is released stream-ordered (after the work already queued on the
// stream that uses it) and a larger one allocated in stream order.  Must be called
// with g_mu held.
int stream_workspace(DeviceState& st, hipStream_t stream, size_t bytes, void** out) {
  const bool cap = is_captured(stream);
  LayerMem& m = cap ? st.streams[stream].captured : st.streams[stream].eager;
  if (m.ws_bytes < bytes) {
    void* d = nullptr;
    if (cap) {
      if (bytes < 2 * m.ws_bytes) bytes = 2 * m.ws_bytes;
      hipError_t e = captured_malloc(&d, bytes);
      if (e != hipSuccess) return hip_fail(e, "hipMalloc(workspace of captured calls)");
    } else {
      if (m.ws) {
        hipError_t e = hipFreeAsync(m.ws, stream);
        m.ws = nullptr;
        m.ws_bytes = 0;
        if (e != hipSuccess) return hip_fail(e, "hipFreeAsync(workspace)");
      }
      hipError_t e = hipMallocAsync(&d, bytes, stream);
      if (e != hipSuccess) return hip_fail(e, "hipMallocAsync(workspace)");
    }
    m.ws = d;
    m.ws_bytes = bytes;
  }
  *out = m.ws;
  return SFC_OK;
}

// At least n arrival counters owned by `stream`, all zero when the next
// launch on the stream starts: outside a capture new ones are cleared by a fill
// kernel and every launch leaves those it used at zero; in a capture the fill is
// recorded with each call.  Must be called with g_mu held.
int stream_counters(DeviceState& st, hipStream_t stream, int64_t n, int32_t** out) {
  const bool cap = is_captured(stream);
  LayerMem& m = cap ? st.streams[stream].captured : st.streams[stream].eager;
  if (m.n_counters < n) {
    void* d = nullptr;
    int64_t count = n < 4096 ? 4096 : n;
    if (cap) {
      if (count < 2 * m.n_counters) count = 2 * m.n_counters;
      hipError_t e = captured_malloc(&d, (size_t)count * 4u);
      if (e != hipSuccess) return hip_fail(e, "hipMalloc(counters of captured calls)");
    } else {
      if (m.counters) {
        hipError_t e = hipFreeAsync(m.counters, stream);
        m.counters = nullptr;
        m.n_counters = 0;
        if (e != hipSuccess) return hip_fail(e, "hipFreeAsync(counters)");
      }
      hipError_t e = hipMallocAsync(&d, (size_t)count * 4u, stream);
      if (e != hipSuccess) return hip_fail(e, "hipMallocAsync(counters)");
      e = sfc::launch_fill_i32(static_cast<int32_t*>(d), count, 0, stream);
      if (e != hipSuccess) return hip_fail(e, "counter fill");
    }
    m.counters = static_cast<int32_t*>(d);
    m.n_counters = count;
  }
  if (cap) {
    hipError_t e = sfc::launch_fill_i32(m.counters, n, 0, stream);
    if (e != hipSuccess) return hip_fail(e, "counter fill");
  }
  *out = m.counters;
  return SFC_OK;
}

int get_occupancy(DeviceState& st, const sfc::Variant& v, int* occ) {
  int& o = v.deep ? st.occupancy_deep[v.out_bf16] : st.occupancy[v.tile][v.out_bf16][v.loads][v.f8 != 0];
  if (o == 0) {
    int n = 0;
    hipError_t e = sfc::gemm_occupancy(v, &n);
    if (e != hipSuccess) return hip_fail(e, "occupancy query");
    o = n < 1 ? 1 : n;
  }
  *occ = o;
  return SFC_OK;
}

int tile_from_api(int t) {
  switch (t) {
    case SFC_TILE_128x128: return sfc::kT128x128;
    case SFC_TILE_256x128: return sfc::kT256x128;
    case SFC_TILE_128x256: return sfc::kT128x256;
    case SFC_TILE_256x256: return sfc::kT256x256;
    default: return -1;
  }
}

struct Plan {
  int tile, bm, bn, gm, gn, ce, nk, grid, occ;
  int loads;           // sfc::Loads
  bool deep = false;   // 128x128 blocks with the 4-deep ring (one workgroup per CU)
};

int make_plan(DeviceState& st, int64_t M, int64_t N, int64_t K, const void* A, int64_t lda,
              const void* B, int64_t ldb, bool ob, int ca_layers, int tile_api, Plan* pl, int f8 = 0) {
  int rc = SFC_OK;
  if (f8) {
    // fp8 operands (checked by check_gemm_f8_args): 256x256 or 128x256 blocks,
    // 128-deep K blocks.  A 128-deep fp8 block moves the bytes of a 64-deep
    // bf16 block and takes the same MFMA time, so the free knobs are chosen by
    // the model for the bf16 problem with the same number of blocks, over the
    // two fp8 block shapes (256x256 first: it keeps a tie).
    pl->loads = sfc::kLoadRing;
    int occ[sfc::kNumTiles];
    for (int t = 0; t < sfc::kNumTiles; ++t) occ[t] = 1;
    static const int kF8Tiles[2] = {sfc::kT256x256, sfc::kT128x256};
    for (int t : kF8Tiles) {
      rc = get_occupancy(st, {t, ob, sfc::kLoadRing, f8}, &occ[t]);
      if (rc != SFC_OK) return rc;
    }
    int tile = tile_api == SFC_TILE_AUTO ? -1 : tile_from_api(tile_api);
    int layers = ca_layers;
    if (tile < 0 || ca_layers == SFC_CA_AUTO) {
      const int64_t k_equiv = (K > 0 ? sfc::ceil_div(K, 128) : 0) * sfc::kBK;
      sfc::ModelChoice best{-1, 1, 0.0};
      for (int t : kF8Tiles) {
        if (tile >= 0 && t != tile) continue;
        const sfc::ModelChoice ch = sfc::model_choose(M, N, k_equiv, ob ? 2 : 4, st.num_cus, occ, t, ca_layers);
        if (best.tile < 0 || ch.clk < best.clk) best = ch;
      }
      if (tile < 0 && sfc::strip_beats_128x256(M, N, k_equiv / sfc::kBK, ob ? 2 : 4, st.num_cus, best, 1, true))
        best.tile = sfc::kT256x256;
      tile = best.tile;
      layers = best.layers;
    }
    pl->tile = tile;
    pl->ce = sfc::effective_layers(K, layers, 128);
    pl->bm = sfc::tile_bm(tile);
    pl->bn = sfc::tile_bn(tile);
    pl->gm = (int)sfc::ceil_div(M, pl->bm);
    pl->gn = (int)sfc::ceil_div(N, pl->bn);
    pl->nk = (int)(K > 0 ? sfc::ceil_div(K, 128) : 0);
    rc = get_occupancy(st, {pl->tile, ob && pl->ce == 1, sfc::kLoadRing, f8}, &pl->occ);
    if (rc != SFC_OK) return rc;
    const int64_t tasks = (int64_t)pl->gm * pl->gn * pl->ce;
    const int64_t slots = (int64_t)st.num_cus * pl->occ;
    pl->grid = (int)(tasks < slots ? tasks : slots);
    return SFC_OK;
  }
  // the fast path needs at least one K block per task
  pl->loads = K <= 0 ? sfc::kLoadElements
              : sfc::vector_loads_ok(A, lda, B, ldb, K, N) ? sfc::kLoadRing
              : sfc::any_loads_ok(lda, ldb, K, N) ? sfc::kLoadAny : sfc::kLoadElements;
  if (tile_api == SFC_TILE_AUTO || ca_layers == SFC_CA_AUTO) {
    // the analytical model evaluates the free knobs (block shape, layers)
    int occ[sfc::kNumTiles];
    for (int t = 0; t < sfc::kNumTiles; ++t) {
      rc = get_occupancy(st, {t, ob && ca_layers == 1, pl->loads}, &occ[t]);
      if (rc != SFC_OK) return rc;
    }
    sfc::ModelChoice ch =
        sfc::model_choose(M, N, K, ob ? 2 : 4, st.num_cus, occ,
                          tile_api == SFC_TILE_AUTO ? -1 : tile_from_api(tile_api), ca_layers);
    if (tile_api == SFC_TILE_AUTO && pl->loads != sfc::kLoadElements &&
        sfc::strip_beats_128x256(M, N, sfc::ceil_div(K, sfc::kBK), ob ? 2 : 4, st.num_cus, ch,
                                 sfc::min_columns(pl->loads == sfc::kLoadAny)))
      ch.tile = sfc::kT256x256;
    pl->tile = ch.tile;
    pl->ce = sfc::effective_layers(K, ch.layers, sfc::kBK);
  } else {
    pl->tile = tile_from_api(tile_api);
    pl->ce = sfc::effective_layers(K, ca_layers, sfc::kBK);
  }
  pl->bm = sfc::tile_bm(pl->tile);
  pl->bn = sfc::tile_bn(pl->tile);
  pl->gm = (int)sfc::ceil_div(M, pl->bm);
  pl->gn = (int)sfc::ceil_div(N, pl->bn);
  pl->nk = (int)(K > 0 ? sfc::ceil_div(K, sfc::kBK) : 0);
  // layer copies are fp32 whatever the output type
  const bool kernel_bf16 = ob && pl->ce == 1;
  const int64_t tasks = (int64_t)pl->gm * pl->gn * pl->ce;
  // a grid of at most one 128x128 block per CU runs the deep-ring kernel
  pl->deep = sfc::deep_ring(pl->tile == sfc::kT128x128, pl->loads == sfc::kLoadRing, 0, tasks, st.num_cus);
  rc = get_occupancy(st, {pl->tile, kernel_bf16, pl->loads, 0, pl->deep}, &pl->occ);
  if (rc != SFC_OK) return rc;
  int64_t slots = (int64_t)st.num_cus * pl->occ;
  pl->grid = (int)(tasks < slots ? tasks : slots);
  return SFC_OK;
}

// Wave quantisation of the last round.  With T = gm*gn blocks and S resident
// workgroups the last of ceil(T/S) rounds holds r = T mod S blocks.  When r <= S/2
// and a kernel with half-height blocks of the same width exists, the last
// w = ceil(r/gm) block columns go to a second launch with half-height blocks: their
// 2*gm*w <= S blocks form one round that takes about half as long, and the first
// launch keeps at most floor(T/S) full rounds.  Every element is still one full
// ascending K pass of the same MFMA sequence, so no result bit changes.
struct Split {
  bool on = false;
  int w = 0;      // block columns moved to the strip
  Plan strip;     // the strip's plan (half-height blocks)
};

int plan_tail_split(DeviceState& st, const Plan& pl, int64_t M, int64_t N, bool ob, int f8, Split* sp) {
  sp->on = false;
  if (pl.ce != 1 || pl.loads == sfc::kLoadElements) return SFC_OK;
  int half;
  if (pl.tile == sfc::kT256x256) half = sfc::kT128x256;
  else if (pl.tile == sfc::kT256x128) half = sfc::kT128x128;
  else return SFC_OK;
  int occ2 = 1;
  int rc = get_occupancy(st, {half, ob, pl.loads, f8}, &occ2);
  if (rc != SFC_OK) return rc;
  const int w = sfc::strip_width(M, N, pl.bm, pl.bn, (int64_t)st.num_cus * pl.occ, (int64_t)st.num_cus * occ2,
                                 sfc::min_columns(pl.loads == sfc::kLoadAny), f8 ? pl.nk : 0);
  if (w == 0) return SFC_OK;
  Plan& q = sp->strip;
  q.tile = half;
  q.bm = sfc::tile_bm(half);
  q.bn = sfc::tile_bn(half);
  const int64_t n1 = (int64_t)(pl.gn - w) * pl.bn;
  q.gm = (int)sfc::ceil_div(M, q.bm);
  q.gn = (int)sfc::ceil_div(N - n1, q.bn);
  q.ce = 1;
  q.nk = pl.nk;
  q.occ = occ2;
  // n1 is a multiple of 128, so the strip's B is aligned as B is
  q.loads = pl.loads;
  q.grid = (int)((int64_t)q.gm * q.gn);
  sp->w = w;
  sp->on = true;
  return SFC_OK;
}

// The fused reduction's part of a launch: C and the arrival counters (none:
// the layer copies are summed by the separate reduction kernel).
struct Fuse {
  int32_t* counters = nullptr;
  void* C = nullptr;
  int64_t ldc = 0;
  bool bf16 = false;
};

// One GEMM launch of plan pl into out (C, or the layer copies when pl.ce > 1),
// blocks taken in the order of `table`.  Must be called with g_mu held.
int launch_plan(const Plan& pl, const int32_t* table, int64_t M, int64_t N, int64_t K, const void* A,
                int64_t lda, const void* B, int64_t ldb, void* out, int64_t ldo, int64_t layer_stride,
                bool out_bf16, int sched, const Fuse& fu, hipStream_t stream, int f8) {
  sfc::GemmParams p;
  p.M = M; p.N = N; p.K = K;
  p.A = reinterpret_cast<const uint16_t*>(A); p.lda = lda;
  p.B = reinterpret_cast<const uint16_t*>(B); p.ldb = ldb;
  p.out = out; p.ldo = ldo; p.out_layer_stride = layer_stride;
  p.table = table;
  p.gm = pl.gm; p.gn = pl.gn;
  p.layers = pl.ce;
  p.nk = pl.nk;
  p.tasks = (int64_t)pl.gm * pl.gn * pl.ce;
  p.sched = sched;
  p.c_bf16 = fu.bf16 ? 1 : 0;
  p.counters = fu.counters;
  p.C = fu.C;
  p.ldc = fu.ldc;
  hipError_t e = sfc::launch_gemm({pl.tile, out_bf16, pl.loads, f8, pl.deep}, p, pl.grid, stream);
  if (e != hipSuccess) return hip_fail(e, "GEMM launch");
  return SFC_OK;
}

// Whether a call whose block shape is the library's to choose runs on the
// small-block kernel (fm = 0: no), and how.
sfc::SmallChoice small_choice(const DeviceState& st, int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb, bool ob,
                              int ca_layers) {
  // (K well inside 32 bits: the kernel's K indices run up to a stage past it)
  if (ca_layers > 1 || K > ((int64_t)1 << 30) || !sfc::any_loads_ok(lda, ldb, K, N)) return sfc::SmallChoice{0, 1, 0.0};
  return sfc::small_choose(M, N, K, ob ? 2 : 4, st.num_cus, ca_layers);
}

// The small-block kernel; its layer copies and counters lie in (W, counters), the
// counters zero, or, if W is null, in the stream's own memory.  Must be called
// with g_mu held.
int launch_small_plan(DeviceState& st, int fm, int layers, int64_t M, int64_t N, int64_t K, const void* A, int64_t lda,
                      const void* B, int64_t ldb, void* C, int64_t ldc, bool ob, hipStream_t stream,
                      float* W = nullptr, int32_t* counters = nullptr) {
  sfc::SmallParams p;
  p.M = (int)M; p.N = (int)N; p.K = (int)K;
  p.gm = (int)sfc::ceil_div(M, 16 * fm);
  p.gn = (int)sfc::ceil_div(N, 64);
  p.layers = layers;
  // a step whose rows or row ends the ring may not take goes through registers
  p.tail = (K % 32 != 0 || N % 8 != 0) ? 1 : 0;
  p.steps = (int)sfc::ceil_div(K, 32) - p.tail;
  p.A = reinterpret_cast<const uint16_t*>(A); p.lda = lda;
  p.B = reinterpret_cast<const uint16_t*>(B); p.ldb = ldb;
  p.C = C; p.ldc = ldc;
  p.W = W;
  p.counters = counters;
  const int64_t cells = (int64_t)p.gm * p.gn;
  if (layers > 1 && !W) {
    void* own = nullptr;
    int rc = stream_workspace(st, stream, (size_t)cells * (size_t)layers * (size_t)(16 * fm * 64) * 4u, &own);
    if (rc == SFC_OK) rc = stream_counters(st, stream, cells, &p.counters);
    if (rc != SFC_OK) return rc;
    p.W = static_cast<float*>(own);
  }
  hipError_t e = sfc::launch_small(p, fm, ob, stream);
  if (e != hipSuccess) return hip_fail(e, "small GEMM launch");
  return SFC_OK;
}

// How the layer copies of a call with c_eff > 1 are summed.
enum Reduce { kReduceSeparate = 0, kReduceFused = 1 };

int gemm_impl(int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, const void* B,
              int64_t ldb, void* C, int64_t ldc, int out_type, int ca_layers, int tile, int order,
              int sched, void* ws, size_t ws_bytes, void* stream_ptr, int f8 = 0, int reduce = kReduceSeparate) {
  const sfc::Checked chk =
      f8 ? sfc::check_gemm_f8_args(M, N, K, A, lda, B, ldb, C, ldc, out_type, ca_layers, tile, order, sched, ws,
                                   ws_bytes)
         : sfc::check_gemm_args(M, N, K, A, lda, B, ldb, C, ldc, out_type, ca_layers, tile, order, sched, ws,
                                ws_bytes);
  if (chk.code != SFC_OK) return set_error(chk.code, chk.msg);
  if (M == 0 || N == 0) return SFC_OK;
  hipStream_t stream = reinterpret_cast<hipStream_t>(stream_ptr);
  const bool ob = out_type == SFC_OUT_BF16;
  // K = 0 is accepted with any N, but the fp8 kernels store whole chunks of columns
  // (N a multiple of 16): the zeros of another N come from the element kernels
  if (f8 && K == 0 && N % 16 != 0) f8 = 0;

  std::lock_guard<std::mutex> lock(g_mu);
  DeviceState* st = nullptr;
  int rc = device_state(&st);
  if (rc != SFC_OK) return rc;
  // (a caller's workspace receives the layer copies of the plan: with the layer
  // count left to the library, that is the curve kernel's)
  if (tile == SFC_TILE_AUTO && !f8 && !(ws && ca_layers == SFC_CA_AUTO)) {
    const sfc::SmallChoice sm = small_choice(*st, M, N, K, lda, ldb, ob, ca_layers);
    if (sm.fm)
      return launch_small_plan(*st, sm.fm, sm.layers, M, N, K, A, lda, B, ldb, C, ldc, ob, stream);
  }
  Plan pl;
  rc = make_plan(*st, M, N, K, A, lda, B, ldb, ob, ca_layers, tile, &pl, f8);
  if (rc != SFC_OK) return rc;

  // the block shape is the library's to choose: a half-height strip may take
  // a partial last round
  Split sp;
  if (tile == SFC_TILE_AUTO) {
    rc = plan_tail_split(*st, pl, M, N, ob, f8, &sp);
    if (rc != SFC_OK) return rc;
  }
  const Fuse none;
  if (sp.on) {
    Plan main = pl;
    main.gn -= sp.w;
    const int64_t tasks = (int64_t)main.gm * main.gn;
    const int64_t slots = (int64_t)st->num_cus * main.occ;
    main.grid = (int)(tasks < slots ? tasks : slots);
    const int64_t n1 = (int64_t)main.gn * main.bn;
    const int32_t *t_main = nullptr, *t_strip = nullptr;
    rc = get_table(*st, main.gm, main.gn, order, stream, &t_main);
    if (rc == SFC_OK) rc = get_table(*st, sp.strip.gm, sp.strip.gn, order, stream, &t_strip);
    if (rc != SFC_OK) return rc;
    rc = launch_plan(main, t_main, M, n1, K, A, lda, B, ldb, C, ldc, 0, ob, sched, none, stream, f8);
    if (rc != SFC_OK) return rc;
    const size_t esz = ob ? 2 : 4;
    return launch_plan(sp.strip, t_strip, M, N - n1, K, A, lda, static_cast<const char*>(B) + n1 * (f8 ? 1 : 2), ldb,
                       static_cast<char*>(C) + (size_t)n1 * esz, ldc, 0, ob, sched, none, stream, f8);
  }

  const int32_t* table = nullptr;
  rc = get_table(*st, pl.gm, pl.gn, order, stream, &table);
  if (rc != SFC_OK) return rc;
  if (pl.ce == 1) return launch_plan(pl, table, M, N, K, A, lda, B, ldb, C, ldc, 0, ob, sched, none, stream, f8);

  // layer copies: the caller's workspace, or this stream's own
  void* W = ws;
  if (!W) {
    rc = stream_workspace(*st, stream, (size_t)pl.ce * (size_t)M * (size_t)N * 4u, &W);
    if (rc != SFC_OK) return rc;
  }
  Fuse fu;
  if (reduce == kReduceFused) {
    rc = stream_counters(*st, stream, (int64_t)pl.gm * pl.gn, &fu.counters);
    if (rc != SFC_OK) return rc;
    fu.C = C;
    fu.ldc = ldc;
    fu.bf16 = ob;
  }
  rc = launch_plan(pl, table, M, N, K, A, lda, B, ldb, W, N, M * N, false, sched, fu, stream, f8);
  if (rc != SFC_OK || reduce == kReduceFused) return rc;
  hipError_t e = sfc::launch_reduce(static_cast<const float*>(W), pl.ce, M, N, C, ldc, ob, stream);
  if (e != hipSuccess) return hip_fail(e, "reduction launch");
  return SFC_OK;
}

// ---- the entry point that allocates nothing ---------------------------------------------
// sfc_gemm_noalloc_ex keeps everything it needs beyond the caller's buffers in
// this file-scope device array: the layer copies of a ca_layers > 1 call
// (kNoAllocWsBytes) and the curve tables of its launches (two of at most
// kNoAllocCells entries: the main grid and the half-height strip).  The small-block
// kernel's copies and counters (a block and layer per CU at most) lie in the same
// array, its counters in the first table.  Each
// device holds its own copy until the process ends.  In host code `scratch`
// only names the array: its address on a device comes from
// hipGetSymbolAddress, taken once per device with that device current.
constexpr size_t kNoAllocWsBytes = SFC_NOALLOC_WS_BYTES;
constexpr int64_t kNoAllocCells = SFC_NOALLOC_MAX_BLOCKS;
constexpr size_t kNoAllocTableOffset = kNoAllocWsBytes;
constexpr size_t kScratchBytes = kNoAllocWsBytes + 2 * (size_t)kNoAllocCells * 4;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

// The current device's address of `scratch`.  Must be called with g_mu held.
int scratch_address(DeviceState& st, char** out) {
  if (!st.scratch) {
    void* ptr = nullptr;
    hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress(scratch)");
    st.scratch = static_cast<char*>(ptr);
  }
  *out = st.scratch;
  return SFC_OK;
}

int gemm_noalloc_impl(int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, const void* B, int64_t ldb,
                      void* C, int64_t ldc, int out_type, int ca_layers, int tile, int order, int sched,
                      void* stream_ptr) {
  const sfc::Checked chk =
      sfc::check_gemm_args(M, N, K, A, lda, B, ldb, C, ldc, out_type, ca_layers, tile, order, sched, nullptr, 0);
  if (chk.code != SFC_OK) return set_error(chk.code, chk.msg);
  if (M == 0 || N == 0) return SFC_OK;
  // the layer copies must fit (for SFC_CA_AUTO: the largest count the model picks)
  const size_t need = sfc::ws_size(M, N, K, ca_layers);
  if (need > kNoAllocWsBytes)
    return set_error(SFC_ERR_WORKSPACE, "sfc_gemm_noalloc_ex: the layer copies need " + std::to_string(need) +
                                            " bytes; its workspace holds " + std::to_string(kNoAllocWsBytes));
  hipStream_t stream = reinterpret_cast<hipStream_t>(stream_ptr);
  const bool ob = out_type == SFC_OUT_BF16;

  std::lock_guard<std::mutex> lock(g_mu);
  DeviceState* st = nullptr;
  int rc = device_state(&st);
  if (rc != SFC_OK) return rc;
  char* base = nullptr;
  rc = scratch_address(*st, &base);
  if (rc != SFC_OK) return rc;
  int32_t* tables = reinterpret_cast<int32_t*>(base + kNoAllocTableOffset);
  float* W = reinterpret_cast<float*>(base);

  if (tile == SFC_TILE_AUTO) {
    const sfc::SmallChoice sm = small_choice(*st, M, N, K, lda, ldb, ob, ca_layers);
    const int64_t cells = sfc::ceil_div(M, 16 * (sm.fm ? sm.fm : 1)) * sfc::ceil_div(N, 64);
    if (sm.fm && sm.layers > 1) {
      if (cells > kNoAllocCells || (size_t)(cells * sm.layers) * (size_t)(16 * sm.fm * 64) * 4u > kNoAllocWsBytes)
        return set_error(SFC_ERR_WORKSPACE, "sfc_gemm_noalloc_ex: the planned layer copies exceed its workspace");
      // the table memory holds what the last call left: counters start from zero
      hipError_t e = sfc::launch_fill_i32(tables, cells, 0, stream);
      if (e != hipSuccess) return hip_fail(e, "counter fill");
    }
    if (sm.fm)
      return launch_small_plan(*st, sm.fm, sm.layers, M, N, K, A, lda, B, ldb, C, ldc, ob, stream, W, tables);
  }
  Plan pl;
  rc = make_plan(*st, M, N, K, A, lda, B, ldb, ob, ca_layers, tile, &pl);
  if (rc != SFC_OK) return rc;
  if (pl.ce > 1 && (size_t)pl.ce * (size_t)M * (size_t)N * 4u > kNoAllocWsBytes)
    return set_error(SFC_ERR_WORKSPACE, "sfc_gemm_noalloc_ex: the planned layer copies exceed its workspace");
  Split sp;
  if (tile == SFC_TILE_AUTO) {
    rc = plan_tail_split(*st, pl, M, N, ob, 0, &sp);
    if (rc != SFC_OK) return rc;
  }
  Plan main = pl;
  if (sp.on) {
    main.gn -= sp.w;
    const int64_t tasks = (int64_t)main.gm * main.gn;
    const int64_t slots = (int64_t)st->num_cus * main.occ;
    main.grid = (int)(tasks < slots ? tasks : slots);
  }
  if ((int64_t)main.gm * main.gn > kNoAllocCells || (sp.on && (int64_t)sp.strip.gm * sp.strip.gn > kNoAllocCells))
    return set_error(SFC_ERR_UNSUPPORTED, "sfc_gemm_noalloc_ex: more output blocks than its curve table holds (" +
                                              std::to_string(kNoAllocCells) + ")");
  // the curve tables are written on the stream for every call: the array
  // keeps only what the last call left there
  hipError_t e = sfc::launch_sfc_order(main.gm, main.gn, order, tables, stream);
  if (e != hipSuccess) return hip_fail(e, "curve table");
  const Fuse none;
  if (sp.on) {
    int32_t* t_strip = tables + kNoAllocCells;
    e = sfc::launch_sfc_order(sp.strip.gm, sp.strip.gn, order, t_strip, stream);
    if (e != hipSuccess) return hip_fail(e, "curve table");
    const int64_t n1 = (int64_t)main.gn * main.bn;
    rc = launch_plan(main, tables, M, n1, K, A, lda, B, ldb, C, ldc, 0, ob, sched, none, stream, 0);
    if (rc != SFC_OK) return rc;
    const size_t esz = ob ? 2 : 4;
    return launch_plan(sp.strip, t_strip, M, N - n1, K, A, lda, static_cast<const uint16_t*>(B) + n1, ldb,
                       static_cast<char*>(C) + (size_t)n1 * esz, ldc, 0, ob, sched, none, stream, 0);
  }
  if (pl.ce == 1) return launch_plan(pl, tables, M, N, K, A, lda, B, ldb, C, ldc, 0, ob, sched, none, stream, 0);
  rc = launch_plan(pl, tables, M, N, K, A, lda, B, ldb, W, N, M * N, false, sched, none, stream, 0);
  if (rc != SFC_OK) return rc;
  e = sfc::launch_reduce(W, pl.ce, M, N, C, ldc, ob, stream);
  if (e != hipSuccess) return hip_fail(e, "reduction launch");
  return SFC_OK;
}

}  // namespace

extern "C" {

int sfc_version(void) { return 1; }

const char* sfc_strerror(int code) {
  switch (code) {
    case SFC_OK: return "success";
    case SFC_ERR_INVALID_ARG: return "invalid argument";
    case SFC_ERR_UNSUPPORTED: return "unsupported argument";
    case SFC_ERR_WORKSPACE: return "workspace too small";
    case SFC_ERR_HIP: return "HIP runtime error";
    default: return "unknown error code";
  }
}

const char* sfc_last_error(void) { return g_last_error.c_str(); }

size_t sfc_gemm_ws_size(int64_t M, int64_t N, int64_t K, int ca_layers) {
  return sfc::ws_size(M, N, K, ca_layers);
}

int sfc_tile_order_ex(int gm, int gn, int order, int32_t* out_idx) {
  const sfc::Checked chk = sfc::check_order_args(gm, gn, order, out_idx);
  if (chk.code != SFC_OK) return set_error(chk.code, chk.msg);
  std::lock_guard<std::mutex> lock(g_mu);
  DeviceState* st = nullptr;
  int rc = device_state(&st);
  if (rc != SFC_OK) return rc;
  const int32_t* table = nullptr;
  rc = get_table(*st, gm, gn, order, nullptr, &table);
  if (rc != SFC_OK) return rc;
  // a synchronous copy on the null stream: it follows the generator (get_table
  // made the null stream wait for it if it was enqueued on another stream)
  hipError_t e = hipMemcpy(out_idx, table, sizeof(int32_t) * (size_t)gm * (size_t)gn,
                           hipMemcpyDeviceToHost);
  if (e != hipSuccess) return hip_fail(e, "hipMemcpy(curve table)");
  return SFC_OK;
}

int sfc_tile_order(int gm, int gn, int32_t* out_idx) {
  return sfc_tile_order_ex(gm, gn, SFC_ORDER_HILBERT, out_idx);
}

int sfc_gemm_ex(int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, const void* B,
                int64_t ldb, void* C, int64_t ldc, int out_type, int ca_layers, int tile, int order,
                int sched, void* ws, size_t ws_bytes, void* stream) {
  return gemm_impl(M, N, K, A, lda, B, ldb, C, ldc, out_type, ca_layers, tile, order, sched, ws,
                   ws_bytes, stream);
}

int sfc_gemm_f8_ex(int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, const void* B,
                   int64_t ldb, void* C, int64_t ldc, int out_type, int ca_layers, int tile, int order,
                   int sched, void* ws, size_t ws_bytes, void* stream) {
  return gemm_impl(M, N, K, A, lda, B, ldb, C, ldc, out_type, ca_layers, tile, order, sched, ws,
                   ws_bytes, stream, 1);
}

int sfc_gemm_f8_fmt_ex(int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, const void* B,
                       int64_t ldb, void* C, int64_t ldc, int out_type, int a_format, int b_format,
                       int ca_layers, int tile, int order, int sched, void* ws, size_t ws_bytes, void* stream) {
  if ((a_format != SFC_FP8_E4M3 && a_format != SFC_FP8_E5M2) || (b_format != SFC_FP8_E4M3 && b_format != SFC_FP8_E5M2))
    return set_error(SFC_ERR_INVALID_ARG, "unknown fp8 format");
  return gemm_impl(M, N, K, A, lda, B, ldb, C, ldc, out_type, ca_layers, tile, order, sched, ws,
                   ws_bytes, stream, 1 + a_format + 2 * b_format);
}

int sfc_gemm_noalloc_ex(int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, const void* B,
                        int64_t ldb, void* C, int64_t ldc, int out_type, int ca_layers, int tile, int order,
                        int sched, void* stream) {
  return gemm_noalloc_impl(M, N, K, A, lda, B, ldb, C, ldc, out_type, ca_layers, tile, order, sched, stream);
}

int sfc_gemm_fused_ex(int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, const void* B,
                      int64_t ldb, void* C, int64_t ldc, int out_type, int ca_layers, int tile, int order,
                      int sched, void* ws, size_t ws_bytes, void* stream) {
  return gemm_impl(M, N, K, A, lda, B, ldb, C, ldc, out_type, ca_layers, tile, order, sched, ws,
                   ws_bytes, stream, 0, kReduceFused);
}

int sfc_gemm(int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, const void* B, int64_t ldb,
             void* C, int64_t ldc, int ca_layers, void* stream) {
  return gemm_impl(M, N, K, A, lda, B, ldb, C, ldc, SFC_OUT_F32, ca_layers, SFC_TILE_AUTO,
                   SFC_ORDER_HILBERT, SFC_SCHED_INTERLEAVED, nullptr, 0, stream);
}

int sfc_gemm_bf16out(int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, const void* B,
                     int64_t ldb, void* C, int64_t ldc, int ca_layers, void* stream) {
  return gemm_impl(M, N, K, A, lda, B, ldb, C, ldc, SFC_OUT_BF16, ca_layers, SFC_TILE_AUTO,
                   SFC_ORDER_HILBERT, SFC_SCHED_INTERLEAVED, nullptr, 0, stream);
}

int sfc_probe_mfma(int random_operands, int iterations, double* tflops, double* mhz) {
  if (iterations < 1 || !tflops || !mhz) return set_error(SFC_ERR_INVALID_ARG, "invalid probe arguments");
  const size_t n = 256 * 256 + 256;
  float* d = nullptr;
  hipError_t e = hipMalloc(&d, n * sizeof(float));
  if (e != hipSuccess) return hip_fail(e, "hipMalloc(probe)");
  double ms = 0.0;
  e = sfc::run_mfma_probe(random_operands ? 1 : 0, iterations, d, &ms);
  float clk[256];
  if (e == hipSuccess) e = hipMemcpy(clk, d + 256 * 256, sizeof clk, hipMemcpyDeviceToHost);
  (void)hipFree(d);
  if (e != hipSuccess) return hip_fail(e, "MFMA probe");
  double sum = 0.0;
  for (int i = 0; i < 256; ++i) sum += clk[i];
  *mhz = sum / 256.0;
  // per wave and round: 64 MFMA 16x16x32
  const double flops = 256.0 * 4.0 * (double)iterations * 64.0 * (2.0 * 16 * 16 * 32);
  *tflops = ms > 0.0 ? flops / (ms * 1e-3) / 1e12 : 0.0;
  return SFC_OK;
}

int sfc_gemm_plan(int64_t M, int64_t N, int64_t K, int ca_layers, int tile, int64_t plan[7]) {
  if (!plan) return set_error(SFC_ERR_INVALID_ARG, "plan is NULL");
  if (M <= 0 || N <= 0 || K < 0 || ca_layers < 0 || ca_layers > sfc::kMaxLayers ||
      tile < SFC_TILE_AUTO || tile > SFC_TILE_256x256)
    return set_error(SFC_ERR_INVALID_ARG, "invalid plan arguments");
  std::lock_guard<std::mutex> lock(g_mu);
  DeviceState* st = nullptr;
  int rc = device_state(&st);
  if (rc != SFC_OK) return rc;
  Plan pl;
  // aligned dummy pointers: the plan of the vector-load path
  rc = make_plan(*st, M, N, K, reinterpret_cast<const void*>(256), (K + 7) / 8 * 8,
                 reinterpret_cast<const void*>(256), (N + 7) / 8 * 8, false, ca_layers, tile, &pl);
  if (rc != SFC_OK) return rc;
  plan[0] = pl.bm; plan[1] = pl.bn; plan[2] = pl.gm; plan[3] = pl.gn;
  plan[4] = pl.ce; plan[5] = pl.grid; plan[6] = pl.occ;
  return SFC_OK;
}

int sfc_gemm_f8_plan(int64_t M, int64_t N, int64_t K, int ca_layers, int tile, int64_t plan[7]) {
  if (!plan) return set_error(SFC_ERR_INVALID_ARG, "plan is NULL");
  if (M <= 0 || N <= 0 || K < 0 || ca_layers < 0 || ca_layers > sfc::kMaxLayers ||
      (tile != SFC_TILE_AUTO && tile != SFC_TILE_128x256 && tile != SFC_TILE_256x256))
    return set_error(SFC_ERR_INVALID_ARG, "invalid plan arguments");
  std::lock_guard<std::mutex> lock(g_mu);
  DeviceState* st = nullptr;
  int rc = device_state(&st);
  if (rc != SFC_OK) return rc;
  Plan pl;
  rc = make_plan(*st, M, N, K, nullptr, 0, nullptr, 0, false, ca_layers, tile, &pl, 1);
  if (rc != SFC_OK) return rc;
  plan[0] = pl.bm; plan[1] = pl.bn; plan[2] = pl.gm; plan[3] = pl.gn;
  plan[4] = pl.ce; plan[5] = pl.grid; plan[6] = pl.occ;
  return SFC_OK;
}

int sfc_gemm_model(int64_t M, int64_t N, int64_t K, int out_type, int ca_layers, int tile, int num_cus,
                   const int32_t occupancy[4], int64_t choice[3]) {
  if (!choice || !occupancy) return set_error(SFC_ERR_INVALID_ARG, "NULL model argument");
  if (M < 0 || N < 0 || K < 0 || num_cus < 1 || ca_layers < 0 || ca_layers > sfc::kMaxLayers ||
      tile < SFC_TILE_AUTO || tile > SFC_TILE_256x256 || (out_type != SFC_OUT_F32 && out_type != SFC_OUT_BF16))
    return set_error(SFC_ERR_INVALID_ARG, "invalid model arguments");
  int occ[sfc::kNumTiles];
  for (int t = 0; t < sfc::kNumTiles; ++t) {
    if (occupancy[t] < 1) return set_error(SFC_ERR_INVALID_ARG, "occupancy must be >= 1");
    occ[t] = occupancy[t];
  }
  const sfc::ModelChoice ch = sfc::model_choose(M, N, K, out_type == SFC_OUT_BF16 ? 2 : 4, num_cus, occ,
                                                tile == SFC_TILE_AUTO ? -1 : tile_from_api(tile), ca_layers);
  choice[0] = ch.tile + 1;   // SFC_TILE_* code
  choice[1] = sfc::effective_layers(K, ch.layers, sfc::kBK);
  choice[2] = (int64_t)(ch.clk + 0.5);
  return SFC_OK;
}

}  // extern "C"
