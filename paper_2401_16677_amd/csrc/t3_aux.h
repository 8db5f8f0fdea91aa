// The kernels around the tile kernel: reduction, second writer, release, all-gather, tracker set-up.
// Included by t3_api.hip only.
#pragma once

#include "t3_device.h"

namespace t3k {

// ---------------------------------------------------------------------------------------------
// Unfused baseline, second kernel: the reduce-scatter's reduction (Sec. 2.3): out = C + incoming,
// tile by tile in the same issue order, driving the same tracker and release.
//
// Memory bound, and on problems that do not fill the chip bound by the round trips a wavefront makes
// one after the other.  So a lane requests four 16-byte pieces of C and of R each before it adds any,
// its row and column move on by a step instead of a division, and the tile (p.tile_m x p.tile_n,
// reduce_tile_shape in t3_choice.h) is cut to what there is to do.
// One piece at a time on tiles of 128 x 128 (before), two, four and eight in flight, in us: 1148 x 4096 23.6,
// 14.8, 15.2, 17.5; 2048 x 4096 40.5, 21.5, 22.3, 23.2; 2343 x 17664 131.7, 114.9, 115.9, 120.6.
// A range that cuts a ring step keeps the tracked tile, many batches per lane: the next batch is requested before
// the sums of this one leave, or it would wait, in order, for their acknowledgement (1024 x 4096 in 256 x 256 tiles,
// the range from the 7th to the 20th: 38.1 us where it waited, 13.2 now; 184 x 9672 19.8, 9.5; 4096 x 12288 125.6, 115.6).
// Sums leave with the streaming hint, or they push out of the memory-side cache what the next GEMM and
// reduction read there: GEMM and reduction of 4096 x 12288 x 1536 219 us with it, 229 without; of 16384 x 3072 x 1536
// 235 and 242; of 2343 x 17664 x 384 135 and 132.  (A reduction repeated on its own buffers, with no GEMM between,
// is the other way round: 4096 x 12288 109 and 95.)
static_assert(kReduceThreads == kThreads, "");
constexpr uint32_t kPastAll = 0xFFFFFFF0u;      // an offset past every array below 4 GiB
// The tile's sums, V x 4 columns per piece (V = 2: sums leave as bfloat16, 16 bytes of eight).  Pieces past the tile's end
// are addresses past the array: no access is conditional, and the compiler knows how many are in flight.  ONE: a
// batch per lane is all there is (50 registers a lane instead of 90: three wavefronts more per SIMD).
template <int V, bool TO_R, bool TO_SLOT, bool ONE>
__device__ inline void reduce_tile(const Plan &p, const Tile &tl, bool store_only) {
  constexpr int U = kReduceBatch / V, kStep = U * kThreads;
  const int m0 = tl.mi * p.tile_m, nc = tl.nj * p.tile_n;              // nc: column within the chunk
  const int rows = min(p.tile_m, p.M - m0), cols = min(p.tile_n, p.W - nc) / (4 * V);
  const int total = rows * cols, n0 = tl.c * p.W + nc;
  const uint32_t ldc = (uint32_t)p.ldc * 4u, ldr = (uint32_t)p.ldr * 4u, lds = (uint32_t)p.W * (V == 2 ? 2u : 4u);
  const __amdgpu_buffer_rsrc_t c_rsrc = make_rsrc(p.C, (uint32_t)p.M * ldc), r_rsrc = make_rsrc(p.R, (uint32_t)p.M * ldr);
  const __amdgpu_buffer_rsrc_t in_rsrc = make_rsrc(p.R, store_only ? 0u : (uint32_t)p.M * ldr);    // (no bytes: zeros)
  const __amdgpu_buffer_rsrc_t s_rsrc = make_rsrc((const char *)p.fwd + (TO_SLOT ? (int64_t)tl.s * p.M * lds : 0), (uint32_t)p.M * lds);
  int row = (int)threadIdx.x / cols, cc = (int)threadIdx.x - row * cols, e = (int)threadIdx.x;
  const int row_step = kThreads / cols, cc_step = kThreads - row_step * cols;
  struct Batch {
    uint32_t at_r[U], at_s[U];
    f32x4 c[U][V], r[U][V];
  };
  auto request = [&](Batch &b) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t m = (uint32_t)(m0 + row), col = (uint32_t)(n0 + cc * 4 * V) * 4u;
      const bool in = e < total;
      const uint32_t at_c = in ? m * ldc + col : kPastAll;
      b.at_r[u] = in ? m * ldr + col : kPastAll;
      b.at_s[u] = in ? m * lds + (uint32_t)(nc + cc * 4 * V) * (V == 2 ? 2u : 4u) : kPastAll;
#pragma unroll
      for (int v = 0; v < V; ++v) {
        b.c[u][v] = load_stream(c_rsrc, in ? at_c + 16u * v : kPastAll, 0u);
        b.r[u][v] = load_stream(in_rsrc, in ? b.at_r[u] + 16u * v : kPastAll, 0u);
      }
      e += kThreads;
      row += row_step;
      cc += cc_step;
      if (cc >= cols) {
        cc -= cols;
        ++row;
      }
    }
  };
  auto finish = [&](Batch &b) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int v = 0; v < V; ++v) {
        if (!store_only) b.c[u][v] += b.r[u][v];
        if (TO_R) store_agent_hint<true>(r_rsrc, b.at_r[u] == kPastAll ? kPastAll : b.at_r[u] + 16u * v, 0u, b.c[u][v]);
      }
      if constexpr (TO_SLOT && V == 2)
        __builtin_amdgcn_raw_buffer_store_b128(pack_bf16(b.c[u][0], b.c[u][1]), s_rsrc, (int)b.at_s[u], 0, kAuxSc1 | kAuxNt);
      else if constexpr (TO_SLOT)
        store_agent_hint<true>(s_rsrc, b.at_s[u], 0u, b.c[u][0]);
    }
  };
  Batch a, b;
  request(a);
  if constexpr (ONE) {
    finish(a);
    return;
  }
  for (int left = total - kStep; left > 0; left -= kStep) {
    request(b);
    finish(a);
    left -= kStep;
    if (left <= 0) {
      finish(b);
      return;
    }
    request(a);
    finish(b);
  }
  finish(a);
}
// WORDS: the plan by one vector request (PlanWords), for launches of a few workgroups per compute unit, all of which start on lines
// nobody has touched; where thousands follow, the scalar cache has them (GEMM and reduction, scalar and by vector: 39 x 632 x 664
// on 2 chunks 10.4 us, 10.1; 8 x 1124 x 3968 on 16 32.6, 32.1; 1000 x 1000 x 512 on 4, 976 workgroups, 24.3, 24.2; 2343 x 552 x 384 on 32,
// 10000, 152.5, 154.7; 16384 x 384 x 1536 on 8 241.7, 243.1).
template <bool ONE, bool WORDS>
__global__ __launch_bounds__(kThreads) void reduce_tile_kernel(const Plan arg) {
  PlanWords words;
  if (WORDS) words.load((int)(threadIdx.x & 63));
  Plan p = arg;
  if (WORDS) p = words.now();
  uint32_t gen = *(const __attribute__((address_space(4))) uint32_t *)(p.track + 2 * trk_bank_words(p.P));
  Tile tl;
  if (!decode_block(p, blockIdx.x, tl)) return;
  const bool store_only = (p.flags & kFlagStep0StoreOnly) && tl.s == 0;
  const bool direct = p.flags & kFlagFwdDirect, forwarded = tl.c != p.own, bf16 = p.flags & kFlagFwdBf16;
  const bool to_slot = forwarded && (direct || chunk_is_whole(p, tl.s)), to_r = !(forwarded && direct);
  if (to_slot && bf16) {
    if (to_r) reduce_tile<2, true, true, ONE>(p, tl, store_only);
    else reduce_tile<2, false, true, ONE>(p, tl, store_only);
  } else if (to_slot) {
    if (to_r) reduce_tile<1, true, true, ONE>(p, tl, store_only);
    else reduce_tile<1, false, true, ONE>(p, tl, store_only);
  } else {
    reduce_tile<1, true, false, ONE>(p, tl, store_only);
  }
  if (WORDS) p = words.now();
  // (Read as constant memory, which it is until this workgroup's tile is counted.  Behind that another workgroup may end the launch and
  // change it, in a range that cuts a ring step while this one still has a chunk to publish: the compiler may not read it again there.)
  asm volatile("" : "+s"(gen));
  track_tile(p, trk_at(p, gen), tl, p.whole_chunks != 0);
}

// The upstream neighbour's updates (the DMA updates of Sec. 4.1), stood in for on one GPU:
// `incoming` (p.C) is added into R tile by tile with the same op-and-store atomics as the local
// GEMM's tiles, in the same issue order, and every tile is counted in the same tracker.  With
// the first chunk stored only (Sec. 4.4) it has no upstream update: those tiles are skipped.
template <int BM, int BN>
__global__ __launch_bounds__(kThreads) void upstream_update_kernel(const Plan p) {
  const Trk trk = trk_open(p);
  // one workgroup per grid position, or fewer workgroups walking the positions in issue order
  for (int pos = blockIdx.x; pos < p.total_blocks; pos += gridDim.x) {
    Tile tl;
    if (!decode_block(p, pos, tl)) continue;
    if ((p.flags & kFlagStep0StoreOnly) && tl.s == 0) continue;
    const int m0 = tl.mi * BM;
    const int col_lo = tl.c * p.W;
    const int n0 = col_lo + tl.nj * BN;
    const int rows = min(BM, p.M - m0);
    const int cols = min(BN, col_lo + p.W - n0);
    const int total = rows * cols;
    // One word per lane, so that an atomic instruction covers whole 128-byte lines; eight loads
    // in flight per lane before their adds go out (a workgroup would otherwise move one word per
    // lane per memory round trip).
    constexpr int kBatch = 8;
    for (int e0 = threadIdx.x; e0 < total; e0 += kBatch * kThreads) {
      float v[kBatch];
      int64_t at[kBatch];
#pragma unroll
      for (int k = 0; k < kBatch; ++k) {
        const int e = e0 + k * kThreads;
        const int rr = e / cols, cc = e - rr * cols;
        at[k] = (int64_t)(m0 + rr);
        v[k] = 0.f;
        if (e < total) v[k] = __builtin_nontemporal_load(p.C + at[k] * p.ldc + n0 + cc);
        at[k] = at[k] * p.ldr + n0 + cc;
      }
#pragma unroll
      for (int k = 0; k < kBatch; ++k)
        if (e0 + k * kThreads < total)
          __hip_atomic_fetch_add(p.R + at[k], v[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    track_tile(p, trk, tl, p.whole_chunks != 0);
  }
}

// The triggered transfers, as a launch of their own (two-writer mode, where no launch can wait
// for the other writer): workgroup (slot, agent) copies its rows of chunk order[slot] into the
// forward slot if the chunk's ready flag is set in the bank of the launch that last completed.
__global__ __launch_bounds__(kThreads) void release_ready_kernel(const Plan p) {
  const int slot = blockIdx.x / p.agents, agent = blockIdx.x % p.agents;
  if (slot > p.P - 2) return;
  const uint32_t g = __builtin_amdgcn_readfirstlane(__hip_atomic_load(
      p.track + 2 * trk_bank_words(p.P), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  const uint32_t *bank = p.track + ((g + 1u) & 1u) * trk_bank_words(p.P);   // bank (g - 1) & 1
  int c = p.rank + slot;
  if (c >= p.P) c -= p.P;
  if (__hip_atomic_load(bank + p.P + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0u) return;
  copy_chunk_rows(p, slot, c, agent * p.rows_per_agent + (int)(threadIdx.x >> 6),
                  min(p.M, (agent + 1) * p.rows_per_agent), kThreads / 64);
}

// Clears tracker state: both banks (queue entries to empty, the rest to 0), gen, error and the
// flags of split tiles to 0.
__global__ void track_reset_kernel(uint32_t *track, int P) {
  const int bank = 3 * P + 2, n = 2 * bank + 2 + kTailSlots;
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    const int j = i < 2 * bank ? i % bank : -1;
    track[i] = (j >= 2 * P && j < 3 * P) ? kEmpty : 0u;
  }
}

// One step of the ring all-gather (Sec. 2.3): a chunk of M rows x W columns moves, unchanged,
// from the upstream neighbour's buffer into the same columns of this rank's.  Memory bound, and short (50 MB of traffic
// take 10 us).  A row is copied by a team of T lanes, U 16-byte pieces per lane and batch; copy_shape in
// t3_choice.h says which.  The loads of a batch and their stores stand behind the same conditions: behind others
// (a pointer that is null where there is nothing to store) the compiler carries the batch's registers through the
// loop and waits for each load before the next.  IN_FLIGHT < U: such a wait on purpose, see copy_shape.
// grid_rows: rows of all workgroups (asked of the launch, as gridDim, it costs the host 0.5 us a call for hidden arguments).
// (A wavefront per row in every shape; pieces numbered across a workgroup's rows, load by load; and now, in us, eight
// chunks: 100 x 1536 2.8, 2.8, 2.4; 1536 x 640 3.0, 3.8, 3.0; 2500 x 1024 5.2, 5.7, 5.2; 8192 x 640 10.3, 9.9, 9.3;
// 4096 x 1536 11.5, 10.5, 10.4; 4096 x 4100 31.6, 31.6, 29.3; 16384 x 12 4.2, 2.8, 2.8; 16384 x 1024 24.8, 27.7, 23.9;
// 16384 x 1536 43.4, 46.1, 43.6.  Over 448 shapes of 8 to 16384 rows and 4 to 5120 columns 6 % less time than the
// first and 8 % less than the second; at most 0.1 us or 4 % over the first; 6000 rows and more of 384 to 1024
// columns up to 10 % over the second on some.)
template <int T, int U, int IN_FLIGHT>
__global__ __launch_bounds__(kThreads) void ag_copy_kernel(const float *src, int64_t ld_src, float *dst,
                                                           int64_t ld_dst, int32_t M, int32_t W, int64_t grid_rows) {
  const int lane = (int)(threadIdx.x % T), W4 = W >> 2;
  for (int64_t r = (int64_t)blockIdx.x * (kThreads / T) + (int)(threadIdx.x / T); r < M; r += grid_rows) {
    const f32x4 *s4 = (const f32x4 *)(src + r * ld_src);
    f32x4 *d4 = (f32x4 *)(dst + r * ld_dst);
    for (int c0 = lane; c0 < W4; c0 += U * T) {
      f32x4 v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (c0 + u * T < W4) v[u] = __builtin_nontemporal_load(s4 + c0 + u * T);
        if (IN_FLIGHT < U) asm volatile("s_waitcnt vmcnt(%0)" : : "n"(IN_FLIGHT - 1) : "memory");
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (c0 + u * T < W4) __builtin_nontemporal_store(v[u], d4 + c0 + u * T);
    }
  }
}

// Copies n words of tracker state (for callers that want to read the state another array holds).
__global__ void track_copy_kernel(const uint32_t *src, uint32_t *dst, int n) {
  for (int i = threadIdx.x; i < n; i += blockDim.x)
    dst[i] = __hip_atomic_load(&src[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace t3k
