// The tile kernel for problems too small to fill the chip with large tiles.
//
// What bounds such a launch is latency: a few thousand clocks from the first request to the first
// product, one memory round trip per K-slab unless many are in flight, and the tail of stores and
// counts.  So the tiles are small (32 or 64 on a side: many workgroups), K is split over the WK
// wavefronts of a workgroup (each computes the WHOLE tile over every WK-th K-slab of 64: the serial
// chain is WK times shorter, and a wavefront reads no operand byte another one reads too), and every
// wavefront has LDS stages of its own, so that the K loop has no barrier: as soon as a slab's
// operands are in registers its stage is requested again, NST slabs ahead.  The WK partial tiles
// are summed through LDS, together with the incoming partial, which was requested behind the first
// slabs; rows leave in whole.
//
// A 64 x 64 tile reads 64 KiB of LDS and copies 64 KiB through L1 for 512 clocks of products per
// WK = 4 slabs, half the matrix rate at best: where 128-wide tiles fill the chip, they win.
#pragma once

#include "t3_gemm.h"

namespace t3k {

// WORDS: the plan by one vector request (PlanWords), where all workgroups of the launch start on argument lines nobody has touched.  Those that
// take the place of finished ones find the lines in the scalar cache, and a request past it costs each of them 0.3 us (by scalar loads and
// by vector: 24 x 12288 x 1536 on 8 chunks, 384 tiles of 32 x 32, 10.9 us, 10.8; 33 x 16000 x 256 on 2, 250 of 64 x 64,
// 8.3, 8.1; 24 x 24576 x 1536 on 8, 768 of 32 x 32, 17.1, 17.7; 16 x 24576 x 4096 on 16 41.1, 42.4; 2097 x 1280 x 1472 on 32, 1056 of 64 x 64, 47.5, 48.1).
template <int BM, int BN, int WK, int NST, int MODE, int BKN, int AKM, bool WORDS>
__global__ __launch_bounds__(64 * WK) void small_tile_kernel(const Plan arg) {
  constexpr int FM = BM / 16, FN = BN / 16, KS = kBK / 32;
  constexpr int NA = BM / kRPC, NB = BN / kRPC, NL = NA + NB;     // 1-KiB copies per slab
  constexpr int kStageBytes = (BM + BN) * kRowBytes, kBOff = BM * kRowBytes;
  constexpr int kRowsPerWave = BM / WK, kChunks = BN / 4;
  constexpr int NIN = kRowsPerWave * kChunks / 64;                // 16-byte pieces of the result per lane
  constexpr int kLds = WK * (NST * kStageBytes > BM * BN * 4 ? NST * kStageBytes : BM * BN * 4);
  static_assert(NIN * 64 == kRowsPerWave * kChunks && (NST - 1) * NL < 64 && kLds <= 160 * 1024, "");
  __shared__ __attribute__((aligned(1024))) char lds[kLds];

  const int lane = threadIdx.x & 63;
  PlanWords words;
  if (WORDS) words.load(lane);
  Plan p = arg;
  if (WORDS) p = words.now();
  // The generation is needed only when the tile is counted.  By scalar loads it is asked for behind the last wait for the argument, or the
  // first copies would wait for its round trip to memory as well (9 x 16896 x 784 on 8 chunks 12.3 us, 12.7); with the argument by vector nothing
  // waits, and its address is out of the way.  (Constant for as long as this kernel reads it: the launch's end, which changes it, waits
  // for every workgroup's count.)
  uint32_t gen = 0;
  auto ask_generation = [&]() {
    if (MODE == kModeFused) gen = *(const __attribute__((address_space(4))) uint32_t *)(p.track + 2 * trk_bank_words(p.P));
  };
  if (WORDS) ask_generation();
  Tile tl;
  if (!decode_block(p, (int)blockIdx.x, tl)) return;
  if (!WORDS) ask_generation();

  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int m0 = tl.mi * BM, col_lo = tl.c * p.W, col_hi = col_lo + p.W, n0 = col_lo + tl.nj * BN;
  const int nkf = p.K / kBK, ktail = p.K - nkf * kBK;
  const int n = wave < nkf ? (nkf - wave + WK - 1) / WK : 0;      // full slabs of this wavefront

  // ---- global -> LDS copies (layouts and swizzles as in gemm_tile_kernel)
  char *const st0 = lds + wave * (NST * kStageBytes);
  const uint32_t lds_w = (uint32_t)(uintptr_t)(lds_void_ptr)st0;
  uint32_t offA[NA], offB[NB];
  constexpr int kARowBytes = BM * 2, kBRowBytes = BN * 2;         // one k-row of a transposed operand
  constexpr int kSwMaskA = (BM / 16 < 8 ? BM / 16 : 8) - 1, kSwMaskB = (BN / 16 < 8 ? BN / 16 : 8) - 1;
  auto k_chunk = [&](int q) { return (lane % kCPR) ^ swz(q * kRPC + lane / kCPR); };
  auto tr_at = [&](int q, int row_bytes, int mask, int &k, int &col) {
    const int L = q * 1024 + lane * 16, cp = (L % row_bytes) / 16;
    k = L / row_bytes;
    const int sw = ((k & 3) | (((k >> 3) & 1) << 2)) & mask;
    col = (((cp >> 1) ^ sw) * 2 + (cp & 1)) * 8;
  };
#pragma unroll
  for (int q = 0; q < NA; ++q) {
    if (AKM) {
      int k, col;
      tr_at(q, kARowBytes, kSwMaskA, k, col);
      offA[q] = (uint32_t)((k * p.lda + min(m0 + col, p.M - 8)) * 2);
    } else {
      offA[q] = (uint32_t)((min(m0 + q * kRPC + lane / kCPR, p.M - 1) * p.lda + k_chunk(q) * 8) * 2);
    }
  }
#pragma unroll
  for (int q = 0; q < NB; ++q) {
    if (BKN) {
      int k, col;
      tr_at(q, kBRowBytes, kSwMaskB, k, col);
      offB[q] = (uint32_t)((k * p.ldb + min(n0 + col, col_hi - 8)) * 2);
    } else {
      offB[q] = (uint32_t)((min(n0 + q * kRPC + lane / kCPR, col_hi - 1) * p.ldb + k_chunk(q) * 8) * 2);
    }
  }
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
  auto issue = [&](int i) {                       // this wavefront's i-th slab
    const int kt = wave + i * WK;
    const char *a = (const char *)p.A + (AKM ? (int64_t)kt * kBK * p.lda * 2 : (int64_t)kt * (kBK * 2));
    const char *b = (const char *)p.B + (BKN ? (int64_t)kt * kBK * p.ldb * 2 : (int64_t)kt * (kBK * 2));
    const uint32_t dst = lds_w + (uint32_t)(i % NST) * kStageBytes;
#pragma unroll
    for (int q = 0; q < NA; ++q)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                   : : "s"(dst + q * 1024), "v"(offA[q]), "s"(a) : "memory", "m0");
#pragma unroll
    for (int q = 0; q < NB; ++q)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                   : : "s"(dst + kBOff + q * 1024), "v"(offB[q]), "s"(b) : "memory", "m0");
  };
#pragma clang diagnostic pop
#pragma unroll
  for (int i = 0; i < NST; ++i)
    if (i < n) issue(i);

  // ---- this wavefront's rows of the tile: the incoming partial, behind the first slabs.  (The
  // waits for slabs below count the slabs' copies only: with these loads among them they wait for
  // a few copies more than they need, never fewer.)
  const bool store_only = MODE == kModeGemm || ((p.flags & kFlagStep0StoreOnly) && tl.s == 0);
  const bool direct = MODE == kModeFused && (p.flags & kFlagFwdDirect);
  const bool to_fwd = MODE == kModeFused && tl.c != p.own && (direct || chunk_is_whole(p, tl.s));
  const bool to_out = !direct || tl.c == p.own;
  const uint32_t ld_out = (uint32_t)(MODE == kModeGemm ? p.ldc : p.ldr);
  const __amdgpu_buffer_rsrc_t r_rsrc = make_rsrc(p.R, (uint32_t)p.M * ld_out * 4u);
  auto at_row = [&](int u) { return wave * kRowsPerWave + (u * 64 + lane) / kChunks; };
  const int chunk = lane % kChunks, col = n0 + chunk * 4;         // (64 is a multiple of kChunks)
  f32x4 in[NIN];
#pragma unroll
  for (int u = 0; u < NIN; ++u) {
    in[u] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int row = m0 + at_row(u);
    if (!store_only && row < p.M && col < col_hi)
      in[u] = load_stream(r_rsrc, ((uint32_t)row * ld_out + (uint32_t)col) * 4u, 0u);
  }

  // ---- K loop
  const int fr = lane & 15, fq = lane >> 4, fs = swz(fr);
  int frag[KS];
#pragma unroll
  for (int kk = 0; kk < KS; ++kk) frag[kk] = fr * kRowBytes + ((4 * kk + fq) ^ fs) * 16;
  const int tr_row = 8 * fq + (fr >> 2), tr_sw = (fr >> 2) | ((fq & 1) << 2);
  auto tr_read = [&](const char *at, int row_bytes) {             // see gemm_tile_kernel
    typedef __attribute__((ext_vector_type(4))) short s16x4;
    typedef __attribute__((ext_vector_type(8))) short s16x8;
    typedef __attribute__((address_space(3))) s16x4 *lds_s16x4_ptr;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(lds_void_ptr)at);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(lds_void_ptr)(at + 4 * row_bytes));
    const s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, both);
  };
  bf16x8 fa[2][KS][FM], fb[2][KS][FN];
  auto read_slab = [&](auto SET, const char *st) {
    constexpr int set = decltype(SET)::value;
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
#pragma unroll
      for (int i = 0; i < FM; ++i)
        fa[set][kk][i] = AKM ? tr_read(st + (32 * kk + tr_row) * kARowBytes + ((i ^ (tr_sw & kSwMaskA)) << 5) + (fr & 3) * 8,
                                       kARowBytes)
                             : *(const bf16x8 *)(st + frag[kk] + i * 16 * kRowBytes);
#pragma unroll
      for (int j = 0; j < FN; ++j)
        fb[set][kk][j] = BKN ? tr_read(st + kBOff + (32 * kk + tr_row) * kBRowBytes +
                                           ((j ^ (tr_sw & kSwMaskB)) << 5) + (fr & 3) * 8, kBRowBytes)
                             : *(const bf16x8 *)(st + kBOff + frag[kk] + j * 16 * kRowBytes);
    }
  };
  f32x4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto multiply = [&](auto SET) {
    constexpr int set = decltype(SET)::value;
#pragma unroll
    for (int kk = 0; kk < KS; ++kk)
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[set][kk][j], fa[set][kk][i], acc[i][j], 0, 0, 0);
  };
  auto wait_slabs = [&](int younger) {            // at most `younger` slabs still on their way
    if (NST >= 3 && younger >= 2) __builtin_amdgcn_s_waitcnt(wait_vm(2 * NL));
    else if (younger >= 1) __builtin_amdgcn_s_waitcnt(wait_vm(NL));
    else __builtin_amdgcn_s_waitcnt(kWaitVm0);
    asm volatile("" ::: "memory");
  };
  static_assert(NST == 2 || NST == 3, "waits are written for these");
  // slab i's operands are on their way from LDS into set SET; the next slab's follow, then its products
  auto step = [&](auto SET, int i) {
    constexpr int set = decltype(SET)::value;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");            // slab i is in registers: its stage is free
    if (i + NST < n) issue(i + NST);
    if (i + 1 < n) {
      wait_slabs(min(NST - 1, n - 2 - i));
      read_slab(std::integral_constant<int, set ^ 1>{}, st0 + ((i + 1) % NST) * kStageBytes);
    }
    multiply(SET);
  };
  constexpr std::integral_constant<int, 0> set0{};
  constexpr std::integral_constant<int, 1> set1{};
  if (n > 0) {
    wait_slabs(min(NST - 1, n - 1));
    read_slab(set0, st0);
    int i = 0;
    for (; i + 1 < n; i += 2) {
      step(set0, i);
      step(set1, i + 1);
    }
    if (i < n) step(set0, i);
  }
  if (ktail && wave == nkf % WK) {                // ragged end of K (K-contiguous operands only)
    if constexpr (!AKM && !BKN) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      const int64_t kb = (int64_t)nkf * (kBK * 2);
#pragma unroll
      for (int q = 0; q < NL; ++q) {
        const int r = q < NA ? q : q - NA;
        u32x4 v{0, 0, 0, 0};
        if (k_chunk(r) * 8 < ktail)
          v = *(const __attribute__((address_space(1))) u32x4 *)((q < NA ? (const char *)p.A + offA[q < NA ? q : 0] : (const char *)p.B + offB[q < NA ? 0 : r]) + kb);
        *(u32x4 *)(st0 + q * 1024 + lane * 16) = v;
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      read_slab(set0, st0);
      multiply(set0);
    }
  }

  // ---- the WK partial tiles through LDS: wavefront w's at w, rows of BN floats, 16-byte chunk k of
  // row r at k ^ (r & 7) (both sides free of bank conflicts)
  __syncthreads();                                // everyone is done with the stages
  {
    char *mine = lds + wave * (BM * BN * 4);
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
        *(f32x4 *)(mine + (16 * i + fr) * (BN * 4) + (((4 * j + fq) ^ (fr & 7)) << 4)) = acc[i][j];
  }
  __syncthreads();
  const float *slot = p.fwd + (int64_t)tl.s * p.M * p.W;
  const uint16_t *slot16 = (const uint16_t *)p.fwd + (int64_t)tl.s * p.M * p.W;
  const bool bf16 = MODE == kModeFused && (p.flags & kFlagFwdBf16);
  const __amdgpu_buffer_rsrc_t f_rsrc = bf16 ? make_rsrc(slot16, (uint32_t)p.M * (uint32_t)p.W * 2u)
                                             : make_rsrc(slot, (uint32_t)p.M * (uint32_t)p.W * 4u);
#pragma unroll
  for (int u = 0; u < NIN; ++u) {
    const int r = at_row(u), row = m0 + r;
    f32x4 v = in[u];
#pragma unroll
    for (int w = 0; w < WK; ++w)
      v += *(const f32x4 *)(lds + w * (BM * BN * 4) + r * (BN * 4) + ((chunk ^ (r & 7)) << 4));
    if (row < p.M && col < col_hi) {
      if (to_out) store_agent(r_rsrc, ((uint32_t)row * ld_out + (uint32_t)col) * 4u, 0u, v);
      const uint32_t at = (uint32_t)row * (uint32_t)p.W + (uint32_t)(col - col_lo);
      if (to_fwd && !bf16) store_agent(f_rsrc, at * 4u, 0u, v);
      if (to_fwd && bf16)
        __builtin_amdgcn_raw_buffer_store_b64(pack_bf16(v), f_rsrc, (int)(at * 2u), 0, kAuxSc1);
    }
  }
  if (MODE == kModeFused) {
    if (WORDS) p = words.now();
    track_tile(p, trk_at(p, gen), tl, true);
  }
}

}  // namespace t3k
