// What every kernel of the library shares: the launch plan, the walk over tiles, the tracker
// (track & trigger, Sec. 4.2 of the T3 paper) and the memory accesses with a cache policy.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "t3_choice.h"
#include "t3_div.h"

#ifndef T3_MH
#define T3_MH 2            // row passes per MFMA k-step of a 128-row wavefront tile (2 or 4)
#endif

namespace t3k {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((address_space(3))) void *lds_void_ptr;

constexpr int kThreads = 256;
constexpr uint32_t kEmpty = 0xFFFFFFFFu;
constexpr int kSpinLimit = 1 << 22;   // polls for the other half of a split tile before the wait gives up
constexpr int kTimelineItems = 16;     // pieces of work per workgroup a timeline records

constexpr uint32_t kFlagStep0StoreOnly = 1u;
constexpr uint32_t kFlagFwdDirect = 2u;
constexpr uint32_t kFlagTwoWriters = 4u;
constexpr uint32_t kFlagFwdBf16 = 8u;

enum Mode { kModeGemm = 0, kModeFused = 1 };

// s_waitcnt immediates (gfx9 encoding: vmcnt[3:0] | expcnt << 4 | lgkmcnt << 8 | vmcnt[5:4] << 14)
constexpr int kWaitVm0 = 0x0F70;
constexpr int kWaitLgkm0 = 0xF0FF;    // and-mask that turns a wait into "... and lgkmcnt(0)"
constexpr int kWaitAll = 0;
__host__ __device__ constexpr int wait_vm(int n) { return 0x0F70 | (n & 15) | ((n >> 4) << 14); }

// Everything a kernel needs, passed by value.
struct Plan {
  const uint16_t *A;
  const uint16_t *B;
  const float *C;    // reduce kernel input
  float *R;          // fused / reduce: incoming in, sums out.  gemm: the C output
  float *fwd;
  uint32_t *track;
  int64_t lda, ldb, ldr, ldc;
  int64_t limit;     // tiles with issue index >= limit do nothing
  int64_t begin;     // nor do tiles with issue index < begin
  int32_t M, N, K, P, rank, W, own;
  // The grid of WORKGROUP tiles: rows, columns, tiles per chunk.  `begin` and `limit` are counted
  // in these.  Where the launch covers whole ring steps they are cut as suits the chip, whatever
  // the tracked tile of the problem; tracked = the tracked tiles of a chunk, which is what its
  // counter holds once it is complete.
  int32_t Mt, Wt, tpc, tracked;
  int32_t tile_m, tile_n;              // the workgroup tile, for the reduction kernel
  int32_t xcd_nbm, xcd_bmk, xcd_bnk;   // XCD grouping of a stage's tiles; xcd_nbm == 0: none
  FastDiv by_tpc, by_column;           // by tpc; by xcd_bmk, or Mt without grouping
  int32_t agents, rows_per_agent;      // release_ready_kernel: workgroups per chunk, rows of each
  int32_t expected_done;               // grid positions of this launch that do work
  int32_t stage0, total_blocks;        // first ring step of the range, grid positions (tiles) from there
  int32_t resident;                    // tile workgroups the chip holds at once
  int32_t upd_first, upd_rest;         // updates expected per element of chunk order[0] / the others
  int32_t split_k;                     // >= 1: workgroups that share a tile, each taking a part of K (Sec. 7.7)
  int32_t stagger_blocks, stagger_groups, stagger_ticks;   // start-up phase offsets (see stagger_start)
  FastDiv by_groups;                   // by k_groups
  int32_t k_groups;                    // > 1: workgroup w starts its K loop (w % k_groups) / k_groups of the way in
  int32_t col_align;                   // 15: tile columns start at 64-byte granules of R, 0: at multiples of the tile (wide-tile kernel)
  int32_t overlap, granule;            // columns by which a chunk's tile columns overlap, elements of a granule (wide-tile kernel, see column_overlap)
  int32_t nt_out;                      // results leave with the streaming hint (wide-tile kernel: the plain GEMM's)
  // Timeline (a profiling aid, normally null): workgroup w < timeline_wgs writes, for its i-th
  // piece of work, i < kTimelineItems, four wall-clock readings (100 MHz) at
  // timeline[(w * kTimelineItems + i) * 4 + ...]: piece taken; accumulators set up (the
  // incoming partial in place); main loop done; results handed to the memory system.
  uint64_t *timeline;
  int32_t timeline_wgs;
  // Balanced tail (persistent launches): the last tail_r grid positions, which would keep only
  // tail_r of the workgroups busy for a whole tile time, are each split into two halves of K
  // (see work_item).  0: off.  tail_q = full rounds of the grid before them; tail_flags = one
  // word per split tile, 0 between launches.
  int32_t tail_r, tail_q;
  uint32_t *tail_flags;
  // Counting (see track_issue): a chunk's tiles in sub_groups (a power of two) groups, `done` by
  // whole chunks; sub_shift places the groups' words.
  int32_t sub_groups, sub_shift, whole_chunks;
  int32_t wide;                        // the wide-tile kernel serves the launch (host side only)
  uint32_t flags;
  TileOrder order;                     // which tile a grid position is (wide-tile kernel; rows 0, as for all the other kernels: decode_block)
};

struct Tile {
  int s, c, mi, nj;
};

// The plan in vector registers, a word per lane: one request for all of the kernel's argument, and a read of a lane
// for each word where it is wanted.  As scalar loads the words come in batches, one behind the other, as the code needs
// them, from lines nobody has touched yet.  The small-tile kernel in one round, in us, by scalar loads and this way: 1024 x 64 x 128 on 16 chunks
// 5.5, 5.3; 40 x 1152 x 256 on 2 5.7, 5.4; 16 x 15184 x 256 on 2 6.4, 6.1; long K 0 to 1 % less.  In the wide-tile kernel it is reading the
// words where they are wanted that counts, which lets the compiler keep none of them through the main loop; by scalar loads at the
// same places it is as fast (2136 x 3072 x 1000 on 8 29.4, 29.3; 1697 x 2304 x 1120 on 32 25.2, 25.3; 523 x 16064 x 752 on 16 39.9, 40.0; a
// ring step of 4096 x 1536 x 1536 28.6, 28.9; twelve shapes 0.1 % less).
struct PlanWords {
  static constexpr int kWords = sizeof(Plan) / 4;
  static_assert(sizeof(Plan) % 4 == 0 && kWords > 64 && kWords <= 128, "two registers");
  uint32_t lo, hi;
  // (the plan is the kernel's only argument)
  __device__ __forceinline__ void load(int lane) {
    const __attribute__((address_space(4))) uint32_t *words = (const __attribute__((address_space(4))) uint32_t *)__builtin_amdgcn_kernarg_segment_ptr();
    lo = words[lane];
    hi = words[lane + 64 < kWords ? lane + 64 : kWords - 1];
  }
  // The plan, to be read here: what is used of it is read out of the lanes now, not kept from before.
  __device__ __forceinline__ Plan now() {
    struct {
      uint32_t w[kWords];
    } d;
    asm volatile("" : "+v"(lo), "+v"(hi));
#pragma unroll
    for (int i = 0; i < kWords; ++i) d.w[i] = (uint32_t)__builtin_amdgcn_readlane((int)(i < 64 ? lo : hi), i & 63);
    return __builtin_bit_cast(Plan, d);
  }
};

// Tracker state (uint32 words): two banks of { counter[P] ready[P] queue[P] queue_len done },
// then the globals { gen, error }.  A launch works in bank gen & 1; the last workgroup of the
// launch to finish clears the other bank and increments gen, so the next launch starts from a
// clean bank without a reset kernel in between, and the caller finds the results of the launch
// that just ended in bank (gen - 1) & 1.
__device__ inline int trk_bank_words(int P) { return 3 * P + 2; }
struct Trk {
  uint32_t *counter, *ready, *queue, *queue_len, *done;   // this launch's bank
  uint32_t *other;                                         // the bank to clear at the end
  uint32_t *gen, *error;
};
// the pointers of the launch that finds generation `gen_now`
__device__ inline Trk trk_at(const Plan &p, uint32_t gen_now) {
  Trk t;
  t.gen = p.track + 2 * trk_bank_words(p.P);
  t.error = t.gen + 1;
  // (the same in every lane: made uniform so that the bank pointers live in scalar registers)
  const uint32_t g = __builtin_amdgcn_readfirstlane(gen_now);
  uint32_t *b = p.track + (g & 1u) * trk_bank_words(p.P);
  t.counter = b;
  t.ready = b + p.P;
  t.queue = b + 2 * p.P;
  t.queue_len = b + 3 * p.P;
  t.done = b + 3 * p.P + 1;
  t.other = p.track + ((g & 1u) ^ 1u) * trk_bank_words(p.P);
  return t;
}
// (an ordinary load: only the end of a launch changes the word, so the XCD's L2 may serve it)
__device__ inline uint32_t trk_gen(const Plan &p) { return p.track[2 * trk_bank_words(p.P)]; }
__device__ inline Trk trk_open(const Plan &p) { return trk_at(p, trk_gen(p)); }
// Who acts on the tracker's words: one thread, behind a branch of its own (an answer is waited for in there: where
// the paths meet again there is none on its way; gemm_tile_kernel's, which clears a bank word by word) ...
struct TrkThread {
  __device__ uint32_t add(uint32_t *w, uint32_t v) const {
    const uint32_t old = __hip_atomic_fetch_add(w, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_s_waitcnt(kWaitVm0);
    return old;
  }
  // two additions on their way together
  __device__ void add_both(uint32_t *w0, uint32_t &v0, uint32_t *w1, uint32_t &v1) const {
    v0 = __hip_atomic_fetch_add(w0, v0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    v1 = __hip_atomic_fetch_add(w1, v1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_s_waitcnt(kWaitVm0);
  }
  __device__ void clear_bank(uint32_t *b, int P) const {
    for (int i = 0; i < 3 * P + 2; ++i) put(&b[i], (i >= 2 * P && i < 3 * P) ? kEmpty : 0u);
  }
  __device__ void put(uint32_t *w, uint32_t v) const {
    __hip_atomic_store(w, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ void wait() const { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
};
// ... or a wavefront as one: every lane issues the access, lane 0's address alone lies inside the array.  Without
// a branch that differs between lanes the compiler keeps rare code out of the way of the loop it stands in (such
// branches have it lay out everything around them as one structured region, the loop's normal path last).
constexpr uint32_t kOob = 0x80000000u;  // an offset past every buffer
struct TrkWave {
  __amdgpu_buffer_rsrc_t words;
  uint32_t *base;
  uint32_t lane_at;                     // lane 0: 0, the others: kOob
  __device__ uint32_t ask(uint32_t *w, uint32_t v) const {       // (lane 0 has the answer)
    return (uint32_t)__builtin_amdgcn_raw_ptr_buffer_atomic_add_i32((int)v, words, (int)lane_at, (int)at(w), 0);
  }
  __device__ uint32_t add(uint32_t *w, uint32_t v) const { return __builtin_amdgcn_readfirstlane(ask(w, v)); }
  __device__ void add_both(uint32_t *w0, uint32_t &v0, uint32_t *w1, uint32_t &v1) const {
    const uint32_t old0 = ask(w0, v0), old1 = ask(w1, v1);
    v0 = __builtin_amdgcn_readfirstlane(old0);
    v1 = __builtin_amdgcn_readfirstlane(old1);
  }
  // (a word per lane: one thread's 3 P + 2 stores one after the other stand at the very end of a launch)
  __device__ void clear_bank(uint32_t *b, int P) const {
    const int lane = (int)(threadIdx.x & 63), n = 3 * P + 2;
    for (int i0 = 0; i0 < n; i0 += 64) {
      const int i = i0 + lane;
      __builtin_amdgcn_raw_buffer_store_b32((i >= 2 * P && i < 3 * P) ? kEmpty : 0u, words, i < n ? i * 4 : (int)kOob, (int)at(b),
                                            16 /* sc1 */);
    }
  }
  __device__ void put(uint32_t *w, uint32_t v) const {
    __builtin_amdgcn_raw_buffer_store_b32(v, words, (int)lane_at, (int)at(w), 16 /* sc1 */);
  }
  __device__ uint32_t get(uint32_t *w) const {
    asm volatile("" ::: "memory");               // (asked for anew every time)
    return __builtin_amdgcn_readfirstlane((uint32_t)__builtin_amdgcn_raw_buffer_load_b32(words, (int)lane_at, (int)at(w), 16 /* sc1 */));
  }
  __device__ void wait() const { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
  __device__ uint32_t at(uint32_t *w) const { return (uint32_t)(w - base) * 4u; }
};
// Called behind a workgroup's addition to `done`; d = what that made of it.
template <typename Who>
__host__ __device__ inline void trk_close_if_last(const Plan &p, const Trk &t, uint32_t d, const Who &who) {
  if (d == (uint32_t)p.expected_done) {
    who.clear_bank(t.other, p.P);
    who.add(t.gen, 1u);
  }
}

// Position j of a stage -> tile.  Workgroups are dealt round-robin to the 8 XCDs: grid position b
// runs on XCD b % 8.  If a stage's tiles split into 8 equal rectangles, XCD x gets a compact block of
// xcd_bmk x xcd_bnk tiles which share A rows and B columns in its L2.  Otherwise it gets a run of
// neighbouring tiles (down the columns), as long as the others' up to one tile.
__device__ inline bool decode_tile(const Plan &p, int s, int j, Tile &tl) {
  int mi, nj;
  if (p.xcd_nbm) {
    const int x = j & 7, i = j >> 3;
    const int bxm = x & (p.xcd_nbm - 1), bxn = x >> (31 - __builtin_clz(p.xcd_nbm));   // (a power of two)
    const int col = (int)div_by((uint32_t)i, p.by_column);
    mi = bxm * p.xcd_bmk + i - col * p.xcd_bmk;
    nj = bxn * p.xcd_bnk + col;
  } else {
    // the stage's positions are b0 .. n - 1 counted from the last multiple of 8 before them; in
    // front of XCD x's run come the positions of XCDs 0 .. x - 1
    const int b0 = ((s - p.stage0) * p.tpc) & 7, n = b0 + p.tpc, jj = j + b0, x = jj & 7;
    const int q = (n >> 3) * x + min(n & 7, x) - min(b0, x) + (jj >> 3) - (x < b0 ? 1 : 0);
    nj = (int)div_by((uint32_t)q, p.by_column);
    mi = q - nj * p.Mt;
  }
  const int64_t t = (int64_t)s * p.tpc + (int64_t)nj * p.Mt + mi;   // issue index
  int c = p.rank + s;
  if (c >= p.P) c -= p.P;
  tl.s = s;
  tl.c = c;
  tl.mi = mi;
  tl.nj = nj;
  return t >= p.begin && t < p.limit;
}

// Grid layout: the tiles of the range's stages in order.  False: a position outside the tile range.
__device__ inline bool decode_block(const Plan &p, int b, Tile &tl) {
  const int s = (int)div_by((uint32_t)b, p.by_tpc);
  return decode_tile(p, p.stage0 + s, b - s * p.tpc, tl);
}
// Whether this launch produces all of stage s's chunk: only then does the chunk get released.
__device__ inline bool chunk_is_whole(const Plan &p, int s) {
  return (int64_t)s * p.tpc >= p.begin && (int64_t)(s + 1) * p.tpc <= p.limit;
}

// The it-th piece of work of a persistent workgroup: grid position `blk`, part `part` of
// `nparts` parts of K.  Without a balanced tail, workgroup w of G takes positions w, w + G, ...
// (split-K: `split_k` consecutive positions share a tile).
//
// Balanced tail.  With T = q G + r positions, 0 < r <= G / 2, the last round would run r tiles on
// r workgroups while the others idle.  Instead each of those r tiles is cut into two halves of
// K.  Half the workgroups are "early": early workgroup number i < r computes the first half of
// tile q G + i BEFORE its q whole tiles, starting from the incoming partial as any tile does,
// and stores the partial sums where the tile's result belongs.  The others are "late": late
// workgroup number i < r computes the second half AFTER its q whole tiles, starting from those
// partial sums, and stores and counts the tile.  Each workgroup then has at most q + 1/2 tiles
// of work, and the first half is q tile times old when the second half asks for it (a flag per
// tile says it is there; see the wait in the kernel).
//
// Workgroups 0 .. r-1 are early, r .. 2r-1 late; the early workgroup of a tile has the lower
// index: it was dispatched first and waits for nothing, so the late one's wait ends.  Early and
// late workgroups run half a tile time apart for the whole launch, and every XCD has both kinds
// (r is normally a multiple of 8, so the two halves of a tile even run on the same XCD): that
// spread of phases measures 5 % faster than whole XCDs running early or late.
template <int TAIL>
__device__ inline bool work_item(const Plan &p, int it, int &blk, int &part, int &nparts) {
  // (workgroups of the grid, or more than there are positions: gridDim's hidden arguments cost the host 0.5 us a launch)
  const int G = p.resident, w = (int)blockIdx.x;
  if (TAIL && p.tail_r) {
    nparts = 1;
    part = 0;
    const bool early = w < p.tail_r;
    const int i = early ? w : w - p.tail_r;
    if (early) {
      if (it == 0) {
        blk = p.tail_q * G + i;
        nparts = 2;
        return true;
      }
      blk = w + (it - 1) * G;
      return it <= p.tail_q;
    }
    if (it < p.tail_q) {
      blk = w + it * G;
      return true;
    }
    if (it == p.tail_q && !early && i < p.tail_r) {
      blk = p.tail_q * G + i;
      part = 1;
      nparts = 2;
      return true;
    }
    return false;
  }
  // (positions fit 31 bits, the launch code sees to that)
  const uint32_t pos = (uint32_t)w + (uint32_t)it * (uint32_t)G;
  if (TAIL || p.split_k == 1) {                  // (a kernel with a balanced tail has no split-K)
    blk = (int)pos;
    part = 0;
    nparts = 1;
    return pos < (uint32_t)p.total_blocks;
  }
  if (pos >= (uint32_t)p.total_blocks * (uint32_t)p.split_k) return false;
  blk = (int)(pos / (uint32_t)p.split_k);
  part = (int)(pos - (uint32_t)blk * (uint32_t)p.split_k);
  nparts = p.split_k;
  return true;
}

// Phase offsets at start-up.  All workgroups of the first wave of tiles start together and would
// reach their reduction traffic (incoming tile in, sums out) together, an HBM-bound burst during
// which no matrix core works.  The first `stagger_blocks` workgroups are put into
// `stagger_groups` phase groups; group g starts g * stagger_ticks (100 MHz ticks) late.  A
// persistent workgroup keeps its offset through all its tiles (every tile takes the same time);
// with one workgroup per grid position, later ones are dispatched as earlier ones retire.
// width_log2: that of the bands of tiles in a line (wide-tile kernel).
__device__ inline void stagger_start(const Plan &p, uint32_t width_log2) {
  const int b = blockIdx.x;
  if (b >= p.stagger_blocks) return;
  // (In a line, workgroups of an XCD that share a row of tiles are in one group: 8689 x 840 x 1120 on 4 chunks 115.3 us with a
  // band's columns in groups, 113.1 with its rows.  In blocks, tiles down the columns, a row's are in one group where the groups divide the
  // block's rows, four groups on blocks of 4 x 3; eight groups on blocks of 4 x 6 have a row in two.)
  const int grp = (((b >> 3) >> width_log2) + (b >> 8)) % p.stagger_groups;
  if (!grp) return;
  const uint64_t t0 = wall_clock64(), wait = (uint64_t)grp * (uint64_t)p.stagger_ticks;
  while (wall_clock64() - t0 < wait) __builtin_amdgcn_s_sleep(8);
}

// Stores that are visible to every XCD once acknowledged: agent scope, i.e. the sc1 bit, which
// writes through the issuing XCD's L2.  (Plain and non-temporal stores stay in that L2 until a
// release fence writes the whole cache back.)
// Tile results and the incoming partial are accessed through buffer instructions: uniform
// descriptor, 32-bit byte offset of the lane, uniform offset of the block.  They are issued as
// compiler builtins, not inline assembly, so that the compiler keeps the required distance
// between an MFMA and a store that reads its result.
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
constexpr int kAuxNt = 2, kAuxSc1 = 16;     // cache-policy bits of the buffer builtins on gfx94x/gfx950
__device__ inline __amdgpu_buffer_rsrc_t make_rsrc(const void *base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)bytes, 0x00020000);
}
__device__ inline void store_agent(__amdgpu_buffer_rsrc_t r, uint32_t lane_off, uint32_t blk_off, f32x4 v) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), r, (int)lane_off, (int)blk_off, kAuxSc1);
}
// (NT: with the streaming hint as well: the lines do not stay in the XCD's L2, where slabs of A
// and B are better kept)
template <bool NT>
__device__ inline void store_agent_hint(__amdgpu_buffer_rsrc_t r, uint32_t lane_off, uint32_t blk_off, f32x4 v) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), r, (int)lane_off, (int)blk_off,
                                         NT ? (kAuxSc1 | kAuxNt) : kAuxSc1);
}
__device__ inline f32x4 load_stream(__amdgpu_buffer_rsrc_t r, uint32_t lane_off, uint32_t blk_off) {
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)lane_off, (int)blk_off, kAuxNt));
}

// fp32 -> bfloat16, round to nearest even (v_cvt_pk_bf16_f32): the 16-bit format a forward slot
// may hold (activations under mixed precision, Sec. 5.2).
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
__device__ inline u32x2 pack_bf16(f32x4 v) {
  return __builtin_bit_cast(u32x2, __builtin_convertvector(v, bf16x4));
}
__device__ inline u32x4 pack_bf16(f32x4 lo, f32x4 hi) {
  const u32x2 a = pack_bf16(lo), b = pack_bf16(hi);
  return u32x4{a[0], a[1], b[0], b[1]};
}

// Rows r0, r0 + step, ... < r_end of chunk c of R into forward slot `slot`, one wavefront per
// row, 16 bytes per lane: the copy a trigger starts (Sec. 4.2.2).  The slot holds fp32, or
// bfloat16 under kFlagFwdBf16.
__device__ inline f32x4 load_agent(__amdgpu_buffer_rsrc_t r, uint32_t lane_off, uint32_t row_off) {
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)lane_off, (int)row_off, kAuxSc1 | kAuxNt));
}
__device__ inline void copy_chunk_rows(const Plan &p, int slot, int c, int r0, int r_end, int step) {
  const int lane = threadIdx.x & 63;
  // R is read with agent-scope loads: they see the producers' write-through stores, so no cache
  // has to be invalidated first (which would cost every workgroup of the XCD its slabs in L2)
  const __amdgpu_buffer_rsrc_t rs = make_rsrc(p.R, (uint32_t)p.M * (uint32_t)p.ldr * 4u);
  const uint32_t col_off = (uint32_t)c * (uint32_t)p.W * 4u;
  if (p.flags & kFlagFwdBf16) {
    const int W8 = p.W >> 3;
    for (int r = r0; r < r_end; r += step) {
      const uint32_t row_off = (uint32_t)r * (uint32_t)p.ldr * 4u + col_off;
      u32x4 *dst = (u32x4 *)((uint16_t *)p.fwd + ((int64_t)slot * p.M + r) * p.W);
      for (int c0 = lane; c0 < W8; c0 += 2 * 64) {
        f32x4 v[4];
#pragma unroll
        for (int u = 0; u < 2; ++u)
          if (c0 + u * 64 < W8) {
            v[2 * u] = load_agent(rs, (uint32_t)(c0 + u * 64) * 32u, row_off);
            v[2 * u + 1] = load_agent(rs, (uint32_t)(c0 + u * 64) * 32u + 16u, row_off);
          }
#pragma unroll
        for (int u = 0; u < 2; ++u)
          if (c0 + u * 64 < W8)
            __builtin_nontemporal_store(pack_bf16(v[2 * u], v[2 * u + 1]), dst + c0 + u * 64);
      }
    }
    return;
  }
  const int W4 = p.W >> 2;
  for (int r = r0; r < r_end; r += step) {
    const uint32_t row_off = (uint32_t)r * (uint32_t)p.ldr * 4u + col_off;
    f32x4 *dst = (f32x4 *)(p.fwd + ((int64_t)slot * p.M + r) * p.W);
    for (int c0 = lane; c0 < W4; c0 += 4 * 64) {
      f32x4 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (c0 + u * 64 < W4) v[u] = load_agent(rs, (uint32_t)(c0 + u * 64) * 16u, row_off);
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (c0 + u * 64 < W4) __builtin_nontemporal_store(v[u], dst + c0 + u * 64);
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Track & trigger (Sec. 4.2).  Tile results are written with agent-scope stores; once they have been
// acknowledged (vmcnt == 0 in every wavefront, then a barrier) the tile is counted.  A device-scope
// release fence instead would write back the whole L2 for every tile and costs several times the
// reduction itself.
//
// Atomic adds to words of one line are done one after the other at the memory side, 20 to 30 ns
// each: with two of them per tile (the chunk's counter and `done`) a launch of 16000 small tiles
// took 1020 us for the counting alone.  So `done` grows by whole chunks, where the launch runs whole
// chunks, and the tiles of a chunk are counted in sub_groups groups first, each in a word of its
// own, eight lines apart in turn; the tile that completes a group counts the group.  (The words are those of
// the balanced tail, which such a launch does not have, and return to 0.)
__host__ __device__ inline uint32_t *trk_group_word(const Plan &p, int s, int g) {
  return p.tail_flags + (((g & 7) << 5) | ((s - p.stage0) << p.sub_shift) | (g >> 3));
}
// By thread 0, when the tile's results are visible: requests the count.
struct TrkCount {
  uint32_t old, done;
};
__host__ __device__ inline uint32_t *track_word(const Plan &p, const Trk &t, const Tile &tl) {     // what counts this tile
  return p.sub_groups > 1 ? trk_group_word(p, tl.s, (tl.nj * p.Mt + tl.mi) & (p.sub_groups - 1)) : &t.counter[tl.c];
}
__device__ inline TrkCount track_issue(const Plan &p, const Trk &t, const Tile &tl) {
  TrkCount k;
  k.old = __hip_atomic_fetch_add(track_word(p, t, tl), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  k.done = p.whole_chunks ? 0u : __hip_atomic_fetch_add(t.done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __builtin_amdgcn_s_waitcnt(kWaitVm0);          // (see TrkThread)
  return k;
}
// Acts on what the count returned.  whole: the launch runs whole chunks (p.whole_chunks; kernels that serve no others say
// so, and the chain at a launch's end has no more code than it needs: 64 x 18432 x 576 on 32 chunks 15.4 us asked, 14.9
// known).  (On the host too: a test plays launches through it.)
template <typename Who>
__host__ __device__ inline void track_finish(const Plan &p, const Trk &t, const Tile &tl, TrkCount k, bool whole, const Who &who) {
  const int c = tl.c;
  uint32_t parts = (uint32_t)p.tpc;
  if (p.sub_groups > 1) {
    const int g = (tl.nj * p.Mt + tl.mi) & (p.sub_groups - 1);
    if (k.old + 1u != (uint32_t)(p.tpc - g + p.sub_groups - 1) >> (31 - __builtin_clz(p.sub_groups))) return;
    who.put(trk_group_word(p, tl.s, g), 0u);
    k.old = who.add(&t.counter[c], 1u);
    parts = (uint32_t)p.sub_groups;
  }
  // threshold = regions of the chunk x updates expected per element (Sec. 4.2.1)
  const uint32_t upd = (uint32_t)(c == p.rank ? p.upd_first : p.upd_rest);
  if (k.old + 1u == parts * upd) {                // the landing that reaches the threshold triggers
    // Over whole chunks `done` and the place in the queue are asked for together: each answer is a round trip to the
    // memory side and back, at the end of the launch's last tile with nothing to cover it.  (One after the other on
    // one thread, which cleared the other bank as well, and this way, in us: 256 x 1024 x 256 on 4 chunks 6.7, 5.7;
    // 24 x 12288 x 1536 on 8 13.0, 11.4; 2048 x 18432 x 576 on 32, without start-up offsets, 94.1, 90.6.)
    // The kept chunk's addition of 0 to queue_len goes along.  Where every tile has asked for its part of `done` already,
    // an addition of nothing to it delays the others (300 x 792 x 320 on 3 chunks from the second tile on 11.8 us,
    // 12.4 with one).
    const bool forwarded = c != p.own;
    uint32_t at = forwarded ? 1u : 0u;
    if (whole) {
      k.done = (uint32_t)p.tpc;
      who.add_both(t.done, k.done, t.queue_len, at);
    } else if (forwarded) {
      at = who.add(t.queue_len, at);
    }
    if (p.tracked * upd != k.old + 1u)            // what the counter is read as: tracked tiles
      who.put(&t.counter[c], (uint32_t)p.tracked * upd);
    if (forwarded) who.put(&t.queue[at], (uint32_t)c);
    // The flag is what publishes.  Everything it stands for was written through the caches and has
    // been acknowledged: the tiles before they were counted, the queue entry by the wait here.  (A
    // release store would write back the L2 on top, in which nothing of this is left.)
    // (queue_len alone publishes nothing: it may run ahead of the entry it reserves.)
    who.wait();
    who.put(&t.ready[c], 1u);
  } else if (whole) {
    return;
  }
  trk_close_if_last(p, t, k.done + (whole ? (uint32_t)p.tpc : 1u), who);
}
__device__ inline TrkWave trk_wave(const Plan &p) {
  return TrkWave{make_rsrc(p.track, (uint32_t)(2 * trk_bank_words(p.P) + 2 + kTailSlots) * 4u), p.track, threadIdx.x == 0 ? 0u : kOob};
}
// The whole of it, by all threads of a workgroup, after the tile's stores have been issued.
__device__ inline void track_tile(const Plan &p, const Trk &t, const Tile &tl, bool whole) {
  __builtin_amdgcn_s_waitcnt(kWaitAll);
  __syncthreads();
  if (threadIdx.x >= 64) return;
  const TrkWave who = trk_wave(p);
  TrkCount k{who.ask(track_word(p, t, tl), 1u), 0u};
  if (!whole) k.done = who.ask(t.done, 1u);
  k.old = __builtin_amdgcn_readfirstlane(k.old);
  k.done = __builtin_amdgcn_readfirstlane(k.done);
  track_finish(p, t, tl, k, whole, who);
}

}  // namespace t3k
