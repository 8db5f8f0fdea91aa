// The kernels around the tile kernel: reduction, second writer, release, all-gather, tracker set-up.
// Included by t3_api.hip only.
#pragma once

#include "t3_device.h"

namespace t3k {

// ---------------------------------------------------------------------------------------------
// Unfused baseline, second kernel: the reduce-scatter's reduction (Sec. 2.3): out = C + incoming,
// tile by tile in the same issue order, driving the same tracker and release.
template <int BM, int BN>
__global__ __launch_bounds__(kThreads) void reduce_tile_kernel(const Plan p) {
  Tile tl;
  if (!decode_block(p, blockIdx.x, tl)) return;
  const Trk trk = trk_open(p);
  const int tid = threadIdx.x;
  const int m0 = tl.mi * BM;
  const int col_lo = tl.c * p.W;
  const int n0 = col_lo + tl.nj * BN;
  const int rows = min(BM, p.M - m0);
  const int cols4 = min(BN, col_lo + p.W - n0) >> 2;
  const bool store_only = (p.flags & kFlagStep0StoreOnly) && tl.s == 0;
  const bool to_fwd = (p.flags & kFlagFwdDirect) && tl.c != p.own;
  const bool to_both = !(p.flags & kFlagFwdDirect) && tl.c != p.own && chunk_is_whole(p, tl.s);
  if ((to_fwd || to_both) && (p.flags & kFlagFwdBf16)) {
    // bfloat16 forward slot: eight sums = 16 bytes per lane
    const int cols8 = cols4 >> 1;
    uint16_t *out16 = (uint16_t *)p.fwd + (int64_t)tl.s * p.M * p.W + (n0 - col_lo);
    for (int e = tid; e < rows * cols8; e += kThreads) {
      const int rr = e / cols8, cc = e - rr * cols8;
      const int64_t row = m0 + rr;
      const f32x4 *c = (const f32x4 *)(p.C + row * p.ldc + n0) + 2 * cc;
      f32x4 *r = (f32x4 *)(p.R + row * p.ldr + n0) + 2 * cc;
      f32x4 lo = __builtin_nontemporal_load(c), hi = __builtin_nontemporal_load(c + 1);
      if (!store_only) {
        lo += __builtin_nontemporal_load(r);
        hi += __builtin_nontemporal_load(r + 1);
      }
      if (to_both) {
        store_agent(r, lo);
        store_agent(r + 1, hi);
      }
      const u32x4 v = pack_bf16(lo, hi);
      asm volatile("global_store_dwordx4 %0, %1, off sc1"
                   : : "v"((u32x4 *)(out16 + row * p.W) + cc), "v"(v) : "memory");
    }
    track_tile(p, trk, tl);
    return;
  }
  float *fwd_base = p.fwd + (int64_t)tl.s * p.M * p.W + (n0 - col_lo);
  const int total = rows * cols4;
  for (int e = tid; e < total; e += kThreads) {
    const int rr = e / cols4, cc = e - rr * cols4;
    const int64_t row = m0 + rr;
    f32x4 *r = (f32x4 *)(p.R + row * p.ldr + n0) + cc;
    f32x4 v = __builtin_nontemporal_load((const f32x4 *)(p.C + row * p.ldc + n0) + cc);
    if (!store_only) v += __builtin_nontemporal_load(r);
    if (!to_fwd) store_agent(r, v);
    if (to_fwd || to_both) store_agent((f32x4 *)(fwd_base + row * p.W) + cc, v);
  }
  track_tile(p, trk, tl);
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
    track_tile(p, trk, tl);
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
// from the upstream neighbour's buffer into the same columns of this rank's.  One wavefront per
// row and pass, 16 bytes per lane, four accesses in flight per lane.
__global__ __launch_bounds__(kThreads) void ag_copy_kernel(const float *src, int64_t ld_src, float *dst,
                                                           int64_t ld_dst, int32_t M, int32_t W) {
  const int lane = threadIdx.x & 63;
  const int W4 = W >> 2;
  const int waves = (int)(gridDim.x * (blockDim.x >> 6));
  for (int r = (int)(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)); r < M; r += waves) {
    const f32x4 *s4 = (const f32x4 *)(src + (int64_t)r * ld_src);
    f32x4 *d4 = (f32x4 *)(dst + (int64_t)r * ld_dst);
    for (int c0 = lane; c0 < W4; c0 += 4 * 64) {
      f32x4 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (c0 + u * 64 < W4) v[u] = __builtin_nontemporal_load(s4 + c0 + u * 64);
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (c0 + u * 64 < W4) __builtin_nontemporal_store(v[u], d4 + c0 + u * 64);
    }
  }
}

// Copies n words of tracker state (for callers that want to read the state another array holds).
__global__ void track_copy_kernel(const uint32_t *src, uint32_t *dst, int n) {
  for (int i = threadIdx.x; i < n; i += blockDim.x)
    dst[i] = __hip_atomic_load(&src[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace t3k
