// Host side of the C ABI declared in include/t3.h: argument validation, the launch plan
// (ring order, tile grid, XCD grouping, release granularity) and the kernel launches.
#include "t3.h"

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdlib.h>
#include <stdio.h>

#include <atomic>
#include <mutex>

#include "t3_aux.h"
#include "t3_choice.h"
#include "t3_launch.h"

namespace t3k {
thread_local int32_t last_hip_error = 0;
}

namespace {

using t3k::ceil_div;
using t3k::launch;
using t3k::TileShape;

// preference order of t3_default_tile
constexpr TileShape kTileShapes[] = {{256, 256}, {256, 128}, {128, 256}, {128, 128}};
constexpr int kNumTileShapes = sizeof(kTileShapes) / sizeof(kTileShapes[0]);
constexpr int kDefaultCus = 256;       // compute units of an MI355X (host-only plan queries assume it)
constexpr int kMaxDevices = 64;
constexpr int kReleaseAgents = 32;     // release workgroups per chunk (t3_release_chunks)
constexpr int64_t kMaxCopyBlocks = 1 << 20;   // workgroups of t3_ag_step; more rows are walked
constexpr int kReduceWordsBlocks = 1024;   // workgroups up to which the reduction takes its plan by a vector request
constexpr int kNtMinK = 3072;          // K from which result stores take the streaming hint
constexpr int64_t kMemorySideCacheBytes = 256ll << 20;
// What the launch plan needs to know of the device it launches on, read from the runtime once
// per device (hardware attributes only; they never change while the process lives).
struct DeviceFacts {
  int cus;     // compute units: persistent workgroups are sized to them
  int xcds;    // accelerator dies the dispatcher deals workgroups to, round-robin
};
std::mutex g_facts_mutex;
DeviceFacts g_facts[kMaxDevices];
bool g_facts_known[kMaxDevices];

// Facts of the current device; T3_ERR_HIP if the runtime cannot tell.
t3_status device_facts(DeviceFacts *out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess && (dev < 0 || dev >= kMaxDevices)) e = hipErrorInvalidDevice;
  if (e == hipSuccess) {
    std::lock_guard<std::mutex> lock(g_facts_mutex);
    if (!g_facts_known[dev]) {
      DeviceFacts f{0, 0};
      e = hipDeviceGetAttribute(&f.cus, hipDeviceAttributeMultiprocessorCount, dev);
      if (e == hipSuccess && hipDeviceGetAttribute(&f.xcds, hipDeviceAttributeNumberOfXccs, dev) != hipSuccess) {
        (void)hipGetLastError();
        f.xcds = 1;                // unknown: plan without XCD grouping
      }
      if (e == hipSuccess && f.cus < 1) e = hipErrorInvalidDevice;
      if (e == hipSuccess) {
        g_facts[dev] = f;
        g_facts_known[dev] = true;
      }
    }
    if (e == hipSuccess) *out = g_facts[dev];
  }
  if (e != hipSuccess) {
    t3k::last_hip_error = (int32_t)e;
    return T3_ERR_HIP;
  }
  return T3_OK;
}

// Where tile kernels record their timelines (t3_timeline), for the launches of every thread.
std::atomic<uint64_t *> g_timeline{nullptr};
std::atomic<int64_t> g_timeline_wgs{0};

// Tracker state for t3_gemm_rs_fused_static, the entry point for callers that cannot allocate:
// one array per device (each GPU the library runs on holds its own copy at its own address
// until the process ends).  Host code never uses the array's name as an address: the device
// address is looked up once per device and kept.
constexpr int kStaticMaxTp = T3_STATIC_MAX_TP;
constexpr int kStaticTrackWords = 2 * (3 * kStaticMaxTp + 2) + 2 + t3k::kTailSlots;
static __device__ __align__(256) uint32_t scratch[kStaticTrackWords];
uint32_t *g_scratch_ptr[kMaxDevices];

// Device address of the current device's `scratch`; T3_ERR_HIP if the runtime cannot tell.
t3_status static_track(uint32_t **out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess && (dev < 0 || dev >= kMaxDevices)) e = hipErrorInvalidDevice;
  if (e == hipSuccess) {
    std::lock_guard<std::mutex> lock(g_facts_mutex);
    if (!g_scratch_ptr[dev]) {
      void *ptr = nullptr;
      e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));   // the current device's copy
      if (e == hipSuccess && !ptr) e = hipErrorInvalidSymbol;
      if (e == hipSuccess) g_scratch_ptr[dev] = static_cast<uint32_t *>(ptr);
    }
    if (e == hipSuccess) *out = g_scratch_ptr[dev];
  }
  if (e != hipSuccess) {
    t3k::last_hip_error = (int32_t)e;
    return T3_ERR_HIP;
  }
  return T3_OK;
}

// Flags of the tiles a balanced tail splits, for t3_gemm, which is given no tracker state to
// keep them in: a few sets of flag words per device.  Two launches may share a set only one
// after the other (the second half of a tile clears the flag the first half raised), so behind
// every launch an event is recorded, and a launch that takes a set whose last user may still be
// running is made to wait for that event first: a launch on the same stream would have waited
// anyway, launches on more streams than there are sets get serialised.  A launch whose stream is
// being captured runs without a balanced tail (a replayed graph would use the set while this
// bookkeeping knows nothing of it).
constexpr int kGemmTailSets = 8;
static __device__ __align__(256) uint32_t gemm_tail_flags[kGemmTailSets * t3k::kTailSlots];
struct GemmTail {
  uint32_t *base = nullptr;              // device address of the current device's gemm_tail_flags
  hipEvent_t done[kGemmTailSets] = {};   // recorded behind the last launch that used the set
  hipStream_t stream[kGemmTailSets] = {};
  bool used[kGemmTailSets] = {};
  unsigned next = 0;
};
GemmTail g_gemm_tail[kMaxDevices];

// Launches the plain GEMM `q` (balanced tail wanted) on stream s with a set of flags, or without
// a balanced tail if no set can be had.  The whole sequence runs under the lock, so that the
// event of a set always belongs to its last launch.
template <typename LaunchFn>
t3_status launch_with_gemm_tail(t3k::Plan &q, hipStream_t s, LaunchFn launch_fn) {
  auto plain = [&]() {
    (void)hipGetLastError();
    q.tail_r = q.tail_q = 0;
    q.tail_flags = nullptr;
    return launch_fn(q);
  };
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  int dev = 0;
  if (hipStreamIsCapturing(s, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone ||
      hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices)
    return plain();
  std::lock_guard<std::mutex> lock(g_facts_mutex);
  GemmTail &g = g_gemm_tail[dev];
  if (!g.base) {
    void *ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(gemm_tail_flags)) != hipSuccess || !ptr) return plain();
    g.base = static_cast<uint32_t *>(ptr);
  }
  // the set this stream used last, else the next in turn
  int set = -1;
  for (int i = 0; i < kGemmTailSets; ++i)
    if (g.used[i] && g.stream[i] == s) set = i;
  if (set < 0) set = (int)(g.next++ % kGemmTailSets);
  if (!g.used[set]) {
    if (hipEventCreateWithFlags(&g.done[set], hipEventDisableTiming) != hipSuccess) return plain();
  } else if (hipStreamWaitEvent(s, g.done[set], 0) != hipSuccess) {
    return plain();
  }
  g.used[set] = true;
  g.stream[set] = s;
  q.tail_flags = g.base + set * t3k::kTailSlots;
  const t3_status st = launch_fn(q);
  // (a launch that failed used nothing; a record that fails leaves the older record in place)
  if (st == T3_OK && hipEventRecord(g.done[set], s) != hipSuccess) (void)hipGetLastError();
  return st;
}

// T3_STAGGER="groups,window_ns" from the environment, read once per process.
struct StaggerEnv {
  bool set = false, off = false;
  int groups = 0, window_ns = 0;
};
const StaggerEnv &stagger_env() {
  static const StaggerEnv env = [] {
    StaggerEnv v;
    if (const char *e = getenv("T3_STAGGER")) {
      int eg = 0, ens = 0;
      const int n = sscanf(e, "%d,%d", &eg, &ens);
      if (n == 2 && eg > 1 && ens > 0) {
        v.set = true;
        v.groups = eg;
        v.window_ns = ens;
      } else if (n >= 1 && eg == 0) {
        v.set = v.off = true;
      }
    }
    return v;
  }();
  return env;
}

t3_status check_shape(const t3_problem *p) {
  if (!p) return T3_ERR_NULL;
  if (p->M < 0 || p->N < 0 || p->K < 0 || p->tp < 1 || p->rank < 0 || p->rank >= p->tp)
    return T3_ERR_BAD_SHAPE;
  if (p->N % p->tp != 0) return T3_ERR_BAD_SHAPE;
  return T3_OK;
}

bool tile_supported(int32_t tm, int32_t tn) {
  for (int i = 0; i < kNumTileShapes; ++i)
    if (kTileShapes[i].m == tm && kTileShapes[i].n == tn) return true;
  return false;
}

void default_tile(const t3_problem *p, int cus, int32_t *tm, int32_t *tn) {
  // The TRACKED tile of a caller who names none (workgroup tiles are workgroup_tile's).  A caller
  // sizes counters by it, so the rule stays as it is: cheapest shape by (work padded up to whole
  // tiles) x (cost per product relative to 256 x 256) x (how far the tiles fall short of filling `cus`
  // compute units), 128 x 256 counted in pairs.
  static const double kSlower[kNumTileShapes] = {1.0, 1.21, 1.0, 1.28};
  const int64_t W = p->N / p->tp;
  double best = -1.0;
  *tm = 128;
  *tn = 128;
  for (int i = 0; i < kNumTileShapes; ++i) {
    const int64_t Mt = ceil_div(p->M, kTileShapes[i].m), Wt = ceil_div(W, kTileShapes[i].n);
    const int64_t T = Mt * Wt * p->tp;
    if (T == 0) continue;
    const bool paired = kTileShapes[i].m == 128 && kTileShapes[i].n == 256 && Mt > 1;
    const int64_t rows = paired ? ceil_div(p->M, 256) * 256 : Mt * kTileShapes[i].m;
    const int64_t groups = paired ? ceil_div(Mt, 2) * Wt * p->tp : T;     // workgroup tiles
    const double padded = (double)rows * (double)(Wt * kTileShapes[i].n) / ((double)p->M * (double)W);
    const double score = padded * kSlower[i] * (groups < cus ? (double)cus / (double)groups : 1.0);
    if (best < 0 || score < best) {
      best = score;
      *tm = kTileShapes[i].m;
      *tn = kTileShapes[i].n;
    }
  }
}

t3_status resolve_tile(const t3_problem *p, int32_t *tm, int32_t *tn) {
  if (p->tile_m == 0 && p->tile_n == 0) {
    default_tile(p, kDefaultCus, tm, tn);
    return T3_OK;
  }
  if (!tile_supported(p->tile_m, p->tile_n)) return T3_ERR_BAD_TILE;
  *tm = p->tile_m;
  *tn = p->tile_n;
  return T3_OK;
}

// the kernels test the same flag bits under their own names
static_assert(T3_FLAG_STEP0_STORE_ONLY == t3k::kFlagStep0StoreOnly &&
                  T3_FLAG_FWD_DIRECT == t3k::kFlagFwdDirect &&
                  T3_FLAG_TWO_WRITERS == t3k::kFlagTwoWriters && T3_FLAG_FWD_BF16 == t3k::kFlagFwdBf16,
              "flag bits of the header and of the kernels");
static_assert(sizeof(t3_problem) == 104, "layout documented in the header");
static_assert(T3_TIMELINE_ITEMS == t3k::kTimelineItems, "timeline layout of the header and of the kernels");

inline bool aligned16(const void *q) { return (reinterpret_cast<uintptr_t>(q) & 15u) == 0; }

enum Need { kNeedAB = 1, kNeedR = 2, kNeedC = 4, kNeedFwd = 8, kNeedTrack = 16,
            kNeedTwoWriters = 32 /* the call exists only in two-writer mode */ };

// The flag words of a balanced tail in tracker state: behind the two banks, gen and error.
inline uint32_t *tail_flags_in(uint32_t *track, int32_t tp) { return track + 2 * (3 * (int64_t)tp + 2) + 2; }

// Validates everything and fills the plan.  *empty is set when there is nothing to launch.
t3_status make_plan(const t3_problem *p, t3k::Call call, int need, const void *A, const void *B, const float *C,
                    float *R, void *fwd, uint32_t *track, t3k::Plan *plan, int32_t *tm,
                    int32_t *tn, bool *empty) {
  t3_status st = check_shape(p);
  if (st != T3_OK) return st;
  st = resolve_tile(p, tm, tn);
  if (st != T3_OK) return st;
  const bool fused_like = (need & kNeedTrack) != 0;
  const bool direct = fused_like && (p->flags & T3_FLAG_FWD_DIRECT);
  const bool two_writers = fused_like && (p->flags & T3_FLAG_TWO_WRITERS);
  if ((need & kNeedAB) && (!A || !B)) return T3_ERR_NULL;
  if ((need & kNeedR) && !R) return T3_ERR_NULL;
  if ((need & kNeedC) && !C) return T3_ERR_NULL;
  if ((need & kNeedTrack) && !track) return T3_ERR_NULL;
  if ((need & kNeedFwd) && p->tp > 1 && !fwd && !(two_writers && (need & kNeedAB)))
    return T3_ERR_NULL;                         // (the fused call releases nothing with two writers)
  if (p->flags & ~(T3_FLAG_STEP0_STORE_ONLY | T3_FLAG_FWD_DIRECT | T3_FLAG_TWO_WRITERS |
                   T3_FLAG_FWD_BF16))
    return T3_ERR_UNSUPPORTED;
  if (two_writers && direct) return T3_ERR_UNSUPPORTED;   // both writers must target R
  if ((need & kNeedTwoWriters) && !two_writers) return T3_ERR_UNSUPPORTED;
  // split-K: several workgroups add into one tile, so it needs the atomic updates of two-writer
  // mode, and every part needs at least one full K-slab of 64
  const int32_t split_k = p->split_k > 1 ? p->split_k : 1;
  if (p->split_k < 0) return T3_ERR_BAD_SHAPE;
  if (split_k > 1 && fused_like && (!two_writers || split_k > p->K / 64 || split_k > 64))
    return T3_ERR_UNSUPPORTED;
  // the unfused reduction kernel has no second writer to wait for
  if (two_writers && (need & kNeedC) && (need & kNeedFwd) && !(need & kNeedTwoWriters))
    return T3_ERR_UNSUPPORTED;

  const int64_t W = p->N / p->tp;
  if (need & kNeedAB) {
    if (p->b_layout != T3_B_NK && p->b_layout != T3_B_KN) return T3_ERR_BAD_SHAPE;
    if (p->a_layout != T3_A_MK && p->a_layout != T3_A_KM) return T3_ERR_BAD_SHAPE;
    if (p->reserved != 0) return T3_ERR_BAD_SHAPE;
    const bool kn = p->b_layout == T3_B_KN, km = p->a_layout == T3_A_KM;
    if (p->lda < (km ? p->M : p->K) || p->ldb < (kn ? p->N : p->K)) return T3_ERR_BAD_SHAPE;
    if (p->K % 8 || p->lda % 8 || p->ldb % 8 || !aligned16(A) || !aligned16(B)) return T3_ERR_ALIGN;
    // A stored K x M: 16-byte pieces run along M, and whole K-slabs of 64 only
    if (km && p->M % 8) return T3_ERR_ALIGN;
    if (km && p->K % 64) return T3_ERR_UNSUPPORTED;
    // B stored K x N: 16-byte pieces run along N, so chunks must be cut on multiples of 8
    // columns, and the transposed operand path takes whole K-slabs of 64 only
    if (kn && W % 8) return T3_ERR_ALIGN;
    if (kn && p->K % 64) return T3_ERR_UNSUPPORTED;
    // kernels address A and B with 32-bit element offsets
    if ((int64_t)(km ? p->K : p->M) * p->lda >= (1ll << 31) ||
        (int64_t)(kn ? p->K : p->N) * p->ldb >= (1ll << 31))
      return T3_ERR_UNSUPPORTED;
  }
  // kernels address R, C and a forward slot with 32-bit byte offsets
  if (need & kNeedR) {
    if (p->ldr < p->N) return T3_ERR_BAD_SHAPE;
    if (p->ldr % 4 || W % 4 || !aligned16(R)) return T3_ERR_ALIGN;
    if ((int64_t)p->M * p->ldr * 4 >= (1ll << 32)) return T3_ERR_UNSUPPORTED;
  }
  if (need & kNeedC) {
    if (p->ldc < p->N) return T3_ERR_BAD_SHAPE;
    if (p->ldc % 4 || W % 4 || !aligned16(C)) return T3_ERR_ALIGN;
    if ((int64_t)p->M * p->ldc * 4 >= (1ll << 32)) return T3_ERR_UNSUPPORTED;
  }
  if ((need & kNeedFwd) && fwd && !aligned16(fwd)) return T3_ERR_ALIGN;
  // bfloat16 forward slots move 8 elements per 16-byte access
  if ((need & kNeedFwd) && fused_like && (p->flags & T3_FLAG_FWD_BF16) && W % 8) return T3_ERR_ALIGN;

  // (the last refusals, before the device is asked anything: tracked tiles, which the issue order, the tile
  // range and the tracker's thresholds are counted in, fit 31 bits, with split-K in as many parts too; the workgroup tiles
  // of arrays below 4 GiB always do)
  const int64_t T_t = ceil_div(p->M, *tm) * ceil_div(W, *tn) * p->tp;
  if (T_t >= (1ll << 31)) return T3_ERR_UNSUPPORTED;
  if (two_writers && T_t * split_k >= (1ll << 31)) return T3_ERR_UNSUPPORTED;
  if ((need & kNeedTwoWriters) && (need & kNeedC) && p->upstream_agents < 0) return T3_ERR_BAD_SHAPE;

  DeviceFacts dev{kDefaultCus, t3k::kNumXcd};
  if (T_t) {                                     // (nothing is launched otherwise: no device needed)
    st = device_facts(&dev);
    if (st != T3_OK) return st;
  }
  const t3k::LaunchShape shape = t3k::launch_shape(p, call, {*tm, *tn}, dev.cus);
  *tm = shape.tile.m;
  *tn = shape.tile.n;
  const int64_t Mt = shape.Mt, Wt = shape.Wt, tpc = shape.tpc;
  *empty = shape.begin >= shape.limit;           // (no tiles, or an empty range of them)

  t3k::Plan &q = *plan;
  q = t3k::Plan{};                               // (callers give memory with an earlier call's plan in it, and not every kernel has every field set)
  q.A = static_cast<const uint16_t *>(A);
  q.B = static_cast<const uint16_t *>(B);
  q.C = C;
  q.R = R;
  q.fwd = static_cast<float *>(fwd);     // (bfloat16 under T3_FLAG_FWD_BF16)
  q.track = track;
  q.lda = p->lda;
  q.ldb = p->ldb;
  q.ldr = p->ldr;
  q.ldc = p->ldc;
  q.limit = shape.limit;
  q.begin = shape.begin;
  q.M = p->M;
  q.N = p->N;
  q.K = p->K;
  q.P = p->tp;
  q.rank = p->rank;
  q.W = (int32_t)W;
  q.own = (p->rank + p->tp - 1) % p->tp;
  q.Mt = (int32_t)Mt;
  q.Wt = (int32_t)Wt;
  q.tpc = (int32_t)tpc;
  q.tile_m = *tm;
  q.tile_n = *tn;
  q.tracked = (int32_t)shape.tracked_tpc;
  q.flags = fused_like ? p->flags : 0u;

  const t3k::XcdBlocks blocks = t3k::xcd_blocks(p, shape, dev.xcds);
  q.xcd_nbm = blocks.by_rows;
  q.xcd_bmk = blocks.rows;
  q.xcd_bnk = blocks.columns;
  const int64_t range_steps = tpc > 0 ? ceil_div(q.limit, tpc) - q.begin / tpc : 0;

  // (an empty problem has no tiles to divide by)
  q.by_tpc = t3k::fast_div((uint32_t)(tpc > 0 ? tpc : 1));
  q.by_column = t3k::fast_div((uint32_t)(tpc == 0 ? 1 : (q.xcd_nbm ? q.xcd_bmk : Mt)));

  const int64_t resident = shape.resident;
  q.stage0 = (int32_t)shape.stage0;
  q.total_blocks = (int32_t)shape.total_blocks;
  // Start-up phase offsets (see stagger_start); T3_STAGGER="groups,window_ns" overrides them ("0" turns them off).
  {
    t3k::StartOffsets o = t3k::start_offsets(p, call, shape);
    const StaggerEnv &env = stagger_env();
    if (env.set) o = env.off ? t3k::StartOffsets{0, 0.0} : t3k::StartOffsets{env.groups, (double)env.window_ns};
    if (o.groups > 1 && o.window_ns >= 100.0) {
      q.stagger_groups = o.groups;
      q.stagger_ticks = (int32_t)(o.window_ns / 10.0 / o.groups);   // 100 MHz ticks between consecutive groups
      q.stagger_blocks = (int32_t)resident;
    }
  }
  q.expected_done = (int32_t)(q.limit - q.begin);
  // updates expected per element (Sec. 4.2.1): with two writers the launches of both count in
  // one bank, which closes when the tiles of both have been counted
  q.upd_first = q.upd_rest = 1;
  q.split_k = 1;
  if (two_writers) {
    q.split_k = split_k;                        // local updates per element = parts of K (Sec. 7.7)
    const bool step0 = (p->flags & T3_FLAG_STEP0_STORE_ONLY) != 0;
    q.upd_rest = split_k + 1;
    q.upd_first = split_k + (step0 ? 0 : 1);
    const int64_t up_begin = (step0 && q.begin < tpc) ? (tpc < q.limit ? tpc : q.limit) : q.begin;
    q.expected_done = (int32_t)((q.limit - q.begin) * split_k + (q.limit - up_begin));
  }
  // K walks start at a different slab on every XCD (see the kernels' `koff`)
  q.k_groups = dev.xcds > 1 ? dev.xcds : 0;
  q.by_groups = t3k::fast_div((uint32_t)(q.k_groups > 1 ? q.k_groups : 1));
  q.resident = (int32_t)resident;
  // Results leave the XCD's L2 at once (streaming hint) where that L2 is better spent on slabs
  // of A and B: long K loops, or an output that the memory-side cache cannot hold anyway.
  // The plain GEMM of 16384 x 3072 x 1536 and the reduction that reads C next: 275 us with the hint, 257
  // without.  (The wide-tile kernel streams fused results always: 4096 x 12288 x 1536 166 us with, 174
  // without; gemm_tile_kernel loses 6 % there with it, and gains 3 % where K or the output is large.)
  q.nt_out = (!two_writers &&
              (p->K >= kNtMinK || 4ll * p->M * p->N > kMemorySideCacheBytes)) ? 1 : 0;
  q.timeline = g_timeline.load();
  {
    const int64_t wgs = g_timeline_wgs.load();
    q.timeline_wgs = (int32_t)(wgs > (1ll << 30) ? (1ll << 30) : wgs);
  }
  q.wide = shape.kernel == t3k::kWideTile;
  if (q.wide) {
    q.order = t3k::tile_order(p, call, shape, t3k::xcd_rows(p, call, shape, blocks));
    q.granule = (p->flags & T3_FLAG_FWD_BF16) && fused_like ? 32 : 16;
    q.overlap = t3k::column_overlap(p, call, shape.tile, Wt);
  }
  q.col_align = q.wide ? t3k::column_align(p, call, shape.tile, Wt) : 0;
  q.tail_r = (int32_t)shape.tail_r;
  q.tail_q = (int32_t)shape.tail_q;
  q.tail_flags = track ? tail_flags_in(track, p->tp) : nullptr;   // (t3_gemm brings its own)
  // Counting.  Groups pay where many tiles finish together; up to 32 ring steps x 8 groups, 16 x 16
  // or 8 x 32 fit the words.
  q.whole_chunks = !two_writers && tpc > 0 && q.begin % tpc == 0 && q.limit % tpc == 0;
  q.sub_groups = 1;
  q.sub_shift = 0;
  if (q.whole_chunks && track && !q.tail_r && range_steps <= 32 && tpc >= 24) {
    q.sub_groups = 8;
    for (int g = 16; g <= 32 && tpc >= 8 * g && range_steps * g <= t3k::kTailSlots; g *= 2) {
      q.sub_groups = g;
      ++q.sub_shift;
    }
  }
  return T3_OK;
}

inline unsigned grid_size(const t3k::Plan &q) { return (unsigned)q.total_blocks; }

t3_status launch_gemm(int mode, const t3k::Plan &q, int32_t tm, int32_t tn, bool b_kn, bool a_km, hipStream_t s) {
  using namespace t3k;
  if (q.wide) {
    if (mode == kModeFused && q.overlap)
      return a_km ? (b_kn ? launch_wide_overlap_km_kn(q, tm, tn, s) : launch_wide_overlap_km(q, tm, tn, s))
                  : (b_kn ? launch_wide_overlap_kn(q, tm, tn, s) : launch_wide_overlap(q, tm, tn, s));
    if (mode == kModeFused)
      return a_km ? (b_kn ? launch_wide_fused_km_kn(q, tm, tn, s) : launch_wide_fused_km(q, tm, tn, s))
                  : (b_kn ? launch_wide_fused_kn(q, tm, tn, s) : launch_wide_fused(q, tm, tn, s));
    Plan g = q;
    g.ldr = q.ldc;                      // C through R
    return a_km ? (b_kn ? launch_wide_gemm_km_kn(g, tm, tn, s) : launch_wide_gemm_km(g, tm, tn, s))
                : (b_kn ? launch_wide_gemm_kn(g, tm, tn, s) : launch_wide_gemm_nk(g, tm, tn, s));
  }
  if (tm < 128)
    return mode == kModeFused ? launch_small_fused(q, tm, tn, b_kn, a_km, s) : launch_small_gemm(q, tm, tn, b_kn, a_km, s);
  if (mode == kModeFused)
    return a_km ? (b_kn ? launch_fused_km_kn(q, tm, tn, s) : launch_fused_km(q, tm, tn, s))
                : (b_kn ? launch_fused_kn(q, tm, tn, s) : launch_fused(q, tm, tn, s));
  return a_km ? (b_kn ? launch_gemm_km_kn(q, tm, tn, s) : launch_gemm_km(q, tm, tn, s))
              : (b_kn ? launch_gemm_kn(q, tm, tn, s) : launch_gemm_nk(q, tm, tn, s));
}

}  // namespace

extern "C" {

const char *t3_status_string(t3_status s) {
  switch (s) {
    case T3_OK: return "ok";
    case T3_ERR_NULL: return "null pointer";
    case T3_ERR_BAD_SHAPE: return "bad shape";
    case T3_ERR_BAD_TILE: return "unsupported tile shape";
    case T3_ERR_ALIGN: return "misaligned pointer or leading dimension";
    case T3_ERR_UNSUPPORTED: return "unsupported request";
    case T3_ERR_HIP: return "HIP runtime error";
  }
  return "unknown status";
}

int32_t t3_last_hip_error(void) { return t3k::last_hip_error; }

t3_status t3_chunk_order(int32_t tp, int32_t rank, int32_t *order, int32_t *own) {
  if (!order || !own) return T3_ERR_NULL;
  if (tp < 1 || rank < 0 || rank >= tp) return T3_ERR_BAD_SHAPE;
  for (int32_t s = 0; s < tp; ++s) order[s] = (rank + s) % tp;
  *own = (rank + tp - 1) % tp;
  return T3_OK;
}

t3_status t3_default_tile(const t3_problem *p, int32_t *tile_m, int32_t *tile_n) {
  if (!tile_m || !tile_n) return T3_ERR_NULL;
  const t3_status st = check_shape(p);
  if (st != T3_OK) return st;
  default_tile(p, kDefaultCus, tile_m, tile_n);
  return T3_OK;
}

t3_status t3_tiles_per_chunk(const t3_problem *p, int64_t *tpc) {
  if (!tpc) return T3_ERR_NULL;
  t3_status st = check_shape(p);
  if (st != T3_OK) return st;
  int32_t tm, tn;
  st = resolve_tile(p, &tm, &tn);
  if (st != T3_OK) return st;
  *tpc = ceil_div(p->M, tm) * ceil_div(p->N / p->tp, tn);
  return T3_OK;
}

t3_status t3_tile_of(const t3_problem *p, int64_t t, int32_t *s, int32_t *c, int32_t *mi,
                     int32_t *nj) {
  if (!s || !c || !mi || !nj) return T3_ERR_NULL;
  int64_t tpc;
  const t3_status st = t3_tiles_per_chunk(p, &tpc);
  if (st != T3_OK) return st;
  if (t < 0 || t >= tpc * p->tp) return T3_ERR_BAD_SHAPE;
  int32_t tm, tn;
  resolve_tile(p, &tm, &tn);
  const int64_t Mt = ceil_div(p->M, tm);
  const int64_t q = t % tpc;
  *s = (int32_t)(t / tpc);
  *c = (p->rank + *s) % p->tp;
  *mi = (int32_t)(q % Mt);
  *nj = (int32_t)(q / Mt);
  return T3_OK;
}

int64_t t3_track_words(int32_t tp) { return tp < 1 ? 0 : 2 * (3ll * tp + 2) + 2 + t3k::kTailSlots; }

t3_status t3_track_reset(int32_t tp, uint32_t *track, void *stream) {
  if (!track) return T3_ERR_NULL;
  if (tp < 1 || tp > (1 << 20)) return T3_ERR_BAD_SHAPE;
  return launch(t3k::track_reset_kernel, dim3(1), dim3(256), static_cast<hipStream_t>(stream), track,
                (int)tp);
}

t3_status t3_gemm_rs_fused(const t3_problem *p, const void *A, const void *B, float *R,
                           void *fwd, uint32_t *track, void *stream) {
  t3k::Plan q;
  int32_t tm, tn;
  bool empty = false;
  const t3_status st = make_plan(p, t3k::kCallFused, kNeedAB | kNeedR | kNeedFwd | kNeedTrack, A, B, nullptr, R,
                                 fwd, track, &q, &tm, &tn, &empty);
  if (st != T3_OK) return st;
  if (empty) return T3_OK;
  return launch_gemm(t3k::kModeFused, q, tm, tn, p->b_layout == T3_B_KN, p->a_layout == T3_A_KM,
                                      static_cast<hipStream_t>(stream));
}

t3_status t3_gemm_rs_fused_static(const t3_problem *p, const void *A, const void *B, float *R,
                                  void *fwd, uint32_t *track_copy, void *stream) {
  if (!p) return T3_ERR_NULL;
  if (p->tp > kStaticMaxTp) return T3_ERR_UNSUPPORTED;   // the static tracker state holds no more
  if (p->flags & T3_FLAG_TWO_WRITERS) return T3_ERR_UNSUPPORTED;   // needs a tracker that outlives the call
  // validate everything first (a non-null stand-in for the tracker pointer: nothing reads it)
  t3k::Plan q;
  int32_t tm, tn;
  bool empty = false;
  uint32_t stand_in = 0;
  t3_status st = make_plan(p, t3k::kCallFused, kNeedAB | kNeedR | kNeedFwd | kNeedTrack, A, B, nullptr, R, fwd,
                           &stand_in, &q, &tm, &tn, &empty);
  if (st != T3_OK) return st;
  uint32_t *track = nullptr;
  st = static_track(&track);
  if (st != T3_OK) return st;
  q.track = track;
  q.tail_flags = tail_flags_in(track, p->tp);
  hipStream_t s = static_cast<hipStream_t>(stream);
  // the array keeps the last call's contents: every call starts from a cleared tracker
  st = launch(t3k::track_reset_kernel, dim3(1), dim3(256), s, track, (int)p->tp);
  if (st != T3_OK) return st;
  if (!empty) {
    st = launch_gemm(t3k::kModeFused, q, tm, tn, p->b_layout == T3_B_KN, p->a_layout == T3_A_KM, s);
    if (st != T3_OK) return st;
  }
  if (track_copy)
    st = launch(t3k::track_copy_kernel, dim3(1), dim3(256), s, (const uint32_t *)track, track_copy,
                (int)t3_track_words(p->tp));
  return st;
}

t3_status t3_gemm(const t3_problem *p, const void *A, const void *B, float *C, void *stream) {
  // (flags and split_k are ignored: make_plan sees no tracker for this call)
  t3k::Plan q;
  int32_t tm, tn;
  bool empty = false;
  const t3_status st = make_plan(p, t3k::kCallGemm, kNeedAB | kNeedC, A, B, C, nullptr, nullptr, nullptr, &q,
                                 &tm, &tn, &empty);
  if (st != T3_OK) return st;
  if (empty) return T3_OK;
  q.R = C;   // the GEMM kernel's output pointer, addressed with ldc
  hipStream_t s = static_cast<hipStream_t>(stream);
  const bool b_kn = p->b_layout == T3_B_KN, a_km = p->a_layout == T3_A_KM;
  auto go = [&](const t3k::Plan &plan) { return launch_gemm(t3k::kModeGemm, plan, tm, tn, b_kn, a_km, s); };
  return q.tail_r ? launch_with_gemm_tail(q, s, go) : go(q);
}

t3_status t3_rs_reduce(const t3_problem *p, const float *C, float *R, void *fwd,
                       uint32_t *track, void *stream) {
  t3k::Plan q;
  int32_t tm, tn;
  bool empty = false;
  const t3_status st = make_plan(p, t3k::kCallReduce, kNeedC | kNeedR | kNeedFwd | kNeedTrack, nullptr, nullptr, C,
                                 R, fwd, track, &q, &tm, &tn, &empty);
  if (st != T3_OK) return st;
  if (empty) return T3_OK;
  const int64_t W = p->N / p->tp, elements = (int64_t)(tm < p->M ? tm : p->M) * (tn < W ? tn : W);
  const bool one = elements <= 4 * t3k::kReduceBatch * t3k::kReduceThreads;
  auto kernel = q.total_blocks <= kReduceWordsBlocks ? (one ? t3k::reduce_tile_kernel<true, true> : t3k::reduce_tile_kernel<false, true>)
                                                     : (one ? t3k::reduce_tile_kernel<true, false> : t3k::reduce_tile_kernel<false, false>);
  return launch(kernel, dim3(grid_size(q)), dim3(t3k::kThreads),
                static_cast<hipStream_t>(stream), q);
}

t3_status t3_upstream_update(const t3_problem *p, const float *incoming, float *R,
                             uint32_t *track, void *stream) {
  t3k::Plan q;
  int32_t tm, tn;
  bool empty = false;
  const t3_status st = make_plan(p, t3k::kCallOther, kNeedC | kNeedR | kNeedTrack | kNeedTwoWriters, nullptr, nullptr,
                                 incoming, R, nullptr, track, &q, &tm, &tn, &empty);
  if (st != T3_OK) return st;
  if (empty) return T3_OK;
  unsigned blocks = grid_size(q);
  if (p->upstream_agents > 0 && (unsigned)p->upstream_agents < blocks)
    blocks = (unsigned)p->upstream_agents;     // the rest of the positions are walked in a loop
  const dim3 grid(blocks), block(t3k::kThreads);
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (tm == 256 && tn == 256)
    return launch(t3k::upstream_update_kernel<256, 256>, grid, block, s, q);
  else if (tm == 256 && tn == 128)
    return launch(t3k::upstream_update_kernel<256, 128>, grid, block, s, q);
  else if (tm == 128 && tn == 256)
    return launch(t3k::upstream_update_kernel<128, 256>, grid, block, s, q);
  return launch(t3k::upstream_update_kernel<128, 128>, grid, block, s, q);
}

t3_status t3_release_chunks(const t3_problem *p, const float *R, void *fwd,
                            const uint32_t *track, void *stream) {
  t3k::Plan q;
  int32_t tm, tn;
  bool empty = false;
  const t3_status st = make_plan(p, t3k::kCallOther, kNeedR | kNeedFwd | kNeedTrack | kNeedTwoWriters, nullptr,
                                 nullptr, nullptr, const_cast<float *>(R), fwd,
                                 const_cast<uint32_t *>(track), &q, &tm, &tn, &empty);
  if (st != T3_OK) return st;
  if (p->tp < 2 || p->M == 0 || p->N == 0) return T3_OK;
  q.agents = kReleaseAgents;
  q.rows_per_agent = (int32_t)ceil_div(p->M, q.agents);
  return launch(t3k::release_ready_kernel, dim3((unsigned)(q.agents * (p->tp - 1))),
                dim3(t3k::kThreads), static_cast<hipStream_t>(stream), q);
}

t3_status t3_timeline(uint64_t *stamps, int64_t words) {
  if (stamps && words < 0) return T3_ERR_BAD_SHAPE;
  if (stamps && (reinterpret_cast<uintptr_t>(stamps) & 7u)) return T3_ERR_ALIGN;
  // (the count first when switching off, the pointer first when switching on: a launch planned
  // in between records nothing rather than out of bounds)
  if (!stamps) {
    g_timeline.store(nullptr);
    g_timeline_wgs.store(0);
    return T3_OK;
  }
  g_timeline_wgs.store(0);
  g_timeline.store(stamps);
  g_timeline_wgs.store(words / (4 * T3_TIMELINE_ITEMS));
  return T3_OK;
}

t3_status t3_ag_step(const t3_problem *p, int32_t step, const float *upstream_R, int64_t ld_up,
                     float *R, void *stream) {
  const t3_status st = check_shape(p);
  if (st != T3_OK) return st;
  if (step < 0 || step >= p->tp - 1) return T3_ERR_BAD_SHAPE;
  if (!upstream_R || !R) return T3_ERR_NULL;
  const int64_t W = p->N / p->tp;
  if (p->ldr < p->N || ld_up < p->N) return T3_ERR_BAD_SHAPE;
  if (p->ldr % 4 || ld_up % 4 || W % 4 || !aligned16(R) || !aligned16(upstream_R)) return T3_ERR_ALIGN;
  if (p->M == 0 || W == 0) return T3_OK;
  const int64_t c = (p->rank + step) % p->tp;    // what the upstream neighbour owned, or got a step ago
  DeviceFacts dev;
  const t3_status known = device_facts(&dev);
  if (known != T3_OK) return known;
  const t3k::CopyShape shape = t3k::copy_shape(p->M, W, dev.cus);
  auto kernel = t3k::ag_copy_kernel<256, 8, 8>;
  if (shape.team == 256 && shape.batch == 1) kernel = t3k::ag_copy_kernel<256, 1, 1>;
  if (shape.team == 64 && shape.batch == 8)
    kernel = shape.in_flight == 8 ? t3k::ag_copy_kernel<64, 8, 8> : (shape.in_flight == 2 ? t3k::ag_copy_kernel<64, 8, 2> : t3k::ag_copy_kernel<64, 8, 1>);
  if (shape.team == 64 && shape.batch == 4) kernel = shape.in_flight == 4 ? t3k::ag_copy_kernel<64, 4, 4> : t3k::ag_copy_kernel<64, 4, 1>;
  if (shape.team == 16) kernel = t3k::ag_copy_kernel<16, 4, 4>;
  if (shape.team == 4) kernel = t3k::ag_copy_kernel<4, 4, 4>;
  const int64_t blocks = shape.workgroups < kMaxCopyBlocks ? shape.workgroups : kMaxCopyBlocks;
  return launch(kernel, dim3((unsigned)blocks), dim3(t3k::kThreads), static_cast<hipStream_t>(stream),
                upstream_R + c * W, ld_up, R + c * W, (int64_t)p->ldr, (int32_t)p->M, (int32_t)W, blocks * (t3k::kThreads / shape.team));
}

}  // extern "C"
