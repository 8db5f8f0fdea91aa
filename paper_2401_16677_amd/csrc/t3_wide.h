// The tile kernel for problems that fill the chip: persistent workgroups of four wavefronts (2 x 2),
// tiles of 32 FM x 32 FN, v_mfma_f32_16x16x32_bf16 with a hand-ordered main loop, any operand layout.
//
// What bounds it.  A 256 x 256 tile is 2048 clocks of products per K-slab of 64; its slab copies
// come at 64 bytes/clock out of the XCD's L2 and at whatever the memory gives where they miss, and
// the reduction adds 512 KiB of HBM traffic per tile (incoming partial in, sums out).  One wavefront
// per SIMD: nobody else fills the matrix pipe while it waits, so everything is arranged for it
// never to wait:
//
//  - The slabs of all the pieces of work of a workgroup are ONE stream of global -> LDS copies, NSTAGE
//    slabs ahead of the products, across the ends of tiles: while a tile's last slabs are multiplied
//    and its results leave, the next tile's first slabs arrive.  A tile costs no fill of the pipeline.
//  - Accumulators start from zero.  The incoming partial (Sec. 4.3) is requested PRE row blocks of it
//    during the tile's last NSTAGE slabs and the rest right behind them, into registers (operands'
//    and spare ones), in the layout the results leave in, and is added on the way out.
//  - Results go row block by row block through an LDS image of its own and leave in whole rows of
//    the tile.  (A chunk's rows start anywhere; every run of addresses that ends inside a 64-byte
//    granule costs the memory side a read-modify-write: 8192 x 4256 x 128, chunks of 532 columns,
//    stored to R and slots took 224 us in 128-byte runs, 134 us in rows, 88 us where 544 columns.)
//  - The plain GEMM is an instantiation of its own, whose whole tiles have nothing to add: requested or
//    cleared registers for it are known to the compiler as accesses to wait for where the way out begins.
//  - The count of a tile is asked for when its stores are known to be acknowledged, in the next
//    tile's main loop, and acted on a slab later.
//
// Copies, incoming partial and results are buffer accesses of buffers that start where the tile does: rows
// past M, columns past the chunk and K past its end are addresses past the buffer, read as zeros and not
// written; no access is conditional, so the number of accesses in flight is always known.  (Addresses past the
// buffer: behind its last row, or kOob = 2^31 plus anything, with buffers of at most 2^31 bytes: the host sees to that.)
//
// Included by the launch units only.
#pragma once

#include "t3_gemm.h"

namespace t3k {

__device__ __forceinline__ void asm_tie(u32x2 (&a)[8]) {
  asm volatile("" : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]), "+v"(a[6]), "+v"(a[7]));
}
__device__ __forceinline__ void asm_tie(u32x2 (&a)[6]) {
  asm volatile("" : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]));
}
__device__ __forceinline__ void asm_tie(u32x2 (&a)[4]) {
  asm volatile("" : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]));
}
__device__ __forceinline__ void asm_accumulator(f32x4 &v) { asm volatile("" : "+a"(v)); }
template <int OFF>
__device__ __forceinline__ void asm_ds_read_tr(u32x2 &dst, uint32_t addr) {
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(OFF));
}

// The operands of one side for a k-step of 32: F blocks of 16 rows, K-contiguous (one 16-byte read
// each) or transposed (TR: two transposing reads of 8 bytes each).
template <int F, bool TR>
struct Operands;
template <int F>
struct Operands<F, false> {
  static constexpr int kReads = F;
  bf16x8 v[F];
  __device__ __forceinline__ void tie() { asm_tie(v); }
  template <int I>
  __device__ __forceinline__ bf16x8 get() const { return v[I]; }
};
template <int F>
struct Operands<F, true> {
  static constexpr int kReads = 2 * F;
  u32x2 lo[F], hi[F];
  __device__ __forceinline__ void tie() {
    asm_tie(lo);
    asm_tie(hi);
  }
  template <int I>
  __device__ __forceinline__ bf16x8 get() const {
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo[I], hi[I], 0, 1, 2, 3));
  }
};

// A piece of work: a tile, or one half of K of it (balanced tail).
struct Piece {
  Tile tl;
  int k0, nf, ns;      // first K-slab, full slabs, slabs with a ragged last one
  int half, idx;       // 0: whole tile, 1 / 2: first / second half of split tile idx
};
// (each part of it reads of the plan what it needs: what is read is read, and kept, whether the branch is taken or not)
__device__ __forceinline__ bool get_piece(PlanWords &words, int it, Piece &w) {
  Plan p = words.now();
  int blk, part, nparts;
  if (!work_item<1>(p, it, blk, part, nparts)) return false;
  const int slabs = p.K / kBK, per = nparts == 2 ? slabs >> 1 : slabs;
  w.k0 = part ? per : 0;
  w.nf = part == nparts - 1 ? slabs - w.k0 : per;
  w.ns = w.nf + (part == nparts - 1 && p.K % kBK ? 1 : 0);
  w.half = nparts == 2 ? 1 + part : 0;
  w.idx = blk - p.tail_q * p.resident;
  if (p.order.rows) {
    p = words.now();
    const TilePlace at = tile_place(p.order, (uint32_t)blk);
    w.tl.s = p.stage0 + at.stage;
    w.tl.c = p.rank + w.tl.s >= p.P ? p.rank + w.tl.s - p.P : p.rank + w.tl.s;
    w.tl.mi = at.row;
    w.tl.nj = at.col;
  } else {
    p = words.now();
    decode_block(p, blk, w.tl);                  // (launches of whole ring steps: every position is a tile)
  }
  return true;
}

template <int FM, int FN, int NSTAGE, int NIMG, int PRE, int DEPTH, int MODE, int BKN, int AKM, int OVERLAP>
__global__ __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu((32 * (FM + FN) * 128 * NSTAGE + NIMG * 4096 * FN) <= 80 * 1024 ? 2 : 1)))
void wide_tile_kernel(const Plan) {
  constexpr int BM = 32 * FM, BN = 32 * FN, WM = 16 * FM, WN = 16 * FN;
  constexpr int NA = BM / kRPC / 4, NB = BN / kRPC / 4, NL = NA + NB;   // 1-KiB copies per wavefront and slab
  constexpr int kStageBytes = (BM + BN) * kRowBytes, kBOff = BM * kRowBytes;
  constexpr int kImgBytes = 2 * 16 * BN * 4, kImgOff = NSTAGE * kStageBytes;
  static_assert(kImgOff + NIMG * kImgBytes <= 160 * 1024 && (NSTAGE == 2 || NSTAGE == 3), "LDS");
  constexpr bool kOneWave = kImgOff + NIMG * kImgBytes > 80 * 1024;     // per SIMD: 512 registers
  static_assert(PRE > 0 && PRE <= DEPTH && DEPTH <= FM && NL + PRE * FN < 64, "");
  __shared__ __attribute__((aligned(1024))) char lds[kImgOff + NIMG * kImgBytes];

  constexpr bool tracked = MODE == kModeFused;
  const int lane = threadIdx.x & 63;
  PlanWords words;
  words.load(lane);
  Plan p = words.now();                          // (read anew where something rare begins)
  // The tracker's generation, a scalar load nothing waits for until a tile is counted.  (Waited for here it puts a round trip
  // to memory in front of the first slabs.)  It is read as constant memory, which it is while this workgroup reads it: the launch's
  // end, which changes it, waits for every workgroup's last count.
  uint32_t gen = 0u;
  if (tracked) gen = *(const __attribute__((address_space(4))) uint32_t *)(p.track + 2 * trk_bank_words(p.P));
  if (p.stagger_groups > 1) stagger_start(p, p.order.width_log2);

  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int ktail = __builtin_amdgcn_readfirstlane(p.K % kBK);
  // bytes from one slab to the next in each operand
  const uint32_t a_step = __builtin_amdgcn_readfirstlane(AKM ? (uint32_t)p.lda * (kBK * 2) : (uint32_t)kRowBytes);
  const uint32_t b_step = __builtin_amdgcn_readfirstlane(BKN ? (uint32_t)p.ldb * (kBK * 2) : (uint32_t)kRowBytes);
  const uint32_t lds_base = (uint32_t)(uintptr_t)(lds_void_ptr)lds;

  // ---- tracking, deferred into the next piece's main loop
  Tile pending{0, -1, 0, 0};
  int pending_half = -1;
  // The count is an atomic the compiler knows of: the register is its to keep, the wait its to make.  (Out of
  // inline assembly the value would be taken as there at once, and could be copied before it is.)
  const uint32_t lane_at = threadIdx.x == 0 ? 0u : kOob;
  auto tracker = [&]() {
    return TrkWave{make_rsrc(p.track, tracked ? (uint32_t)(2 * trk_bank_words(p.P) + 2 + kTailSlots) * 4u : 0u), p.track, lane_at};
  };
  uint32_t count_old = 0u;
  auto ask_count = [&]() {                       // behind a barrier, stores acknowledged
    p = words.now();
    if (pending_half >= 0) TrkWave{make_rsrc(p.tail_flags, kTailSlots * 4u), p.tail_flags, lane_at}.put(p.tail_flags + pending_half, 1u);
    pending_half = -1;
    count_old = pending.c >= 0 ? tracker().ask(track_word(p, trk_at(p, gen), pending), 1u) : 0u;
  };
  auto act_on_count = [&]() {
    if (pending.c >= 0 && wave == 0) {
      p = words.now();
      track_finish(p, trk_at(p, gen), pending, TrkCount{(uint32_t)__builtin_amdgcn_readfirstlane(count_old), 0u}, true, tracker());
    }
    pending.c = -1;
  };
  const bool timeline = __builtin_amdgcn_readfirstlane(p.timeline != nullptr);
  auto stamp = [&](int it, int k) {
    if (!timeline) return;
    p = words.now();
    if (wave == 0 && (int)blockIdx.x < p.timeline_wgs && it < kTimelineItems) {
      const uint64_t now = wall_clock64();
      __builtin_amdgcn_raw_buffer_store_b64(u32x2{(uint32_t)now, (uint32_t)(now >> 32)},
                                            make_rsrc(p.timeline + ((size_t)blockIdx.x * kTimelineItems + it) * 4 + k, 8u), (int)lane_at, 0, 0);
    }
  };

  // ---- the copy stream.  Copy q of a wavefront and operand fills 1 KiB of the operand's region of a
  // stage: eight rows of 64 K-contiguous bf16, or k-rows of a transposed operand (layouts and
  // swizzles as in gemm_tile_kernel).  off*: this lane's byte offsets from where the tile starts in the
  // operand, which is where the piece's descriptor points: from one piece to the next only the descriptors
  // change, in scalar registers (and, transposed, which columns lie outside), and a K-contiguous operand may be as large as the
  // host takes one: fewer than 2^31 elements, so that a tile's start is a 32-bit product.
  uint32_t offA[NA], offB[NB];
  constexpr int kARow = BM * 2, kBRow = BN * 2;  // bytes of a k-row of a transposed operand's region
  auto sw_mask = [](int blocks) { return (blocks % 8 == 0 ? 8 : 4) - 1; };
  auto k_chunk = [&](int q) { return (lane % kCPR) ^ swz(q * kRPC + lane / kCPR); };   // (K-contiguous) chunk of copy q
  auto tr_at = [&](int L, int row_bytes, int mask, int &k, int &col) {                 // (transposed) k-row, column
    const int cp = (L % row_bytes) / 16;
    k = L / row_bytes;
    const int sw = ((k & 3) | (((k >> 3) & 1) << 2)) & mask;
    col = (((cp >> 1) ^ sw) * 2 + (cp & 1)) * 8;
  };
#pragma unroll
  for (int q = 0; q < NA; ++q) {
    if (AKM) {
      int k, col;
      tr_at((wave * NA + q) * 1024 + lane * 16, kARow, sw_mask(BM / 16), k, col);
      offA[q] = (uint32_t)(k * (int)p.lda + col) * 2u;
    } else {
      offA[q] = (uint32_t)((wave * (BM / 4) + q * kRPC + lane / kCPR) * (int)p.lda + k_chunk(q) * 8) * 2u;
    }
  }
#pragma unroll
  for (int q = 0; q < NB; ++q) {
    if (BKN) {
      int k, col;
      tr_at((wave * NB + q) * 1024 + lane * 16, kBRow, sw_mask(BN / 16), k, col);
      offB[q] = (uint32_t)(k * (int)p.ldb + col) * 2u;
    } else {
      offB[q] = (uint32_t)((wave * (BN / 4) + q * kRPC + lane / kCPR) * (int)p.ldb + k_chunk(q) * 8) * 2u;
    }
  }
  auto descriptor = [](const void *base, uint32_t bytes) {       // what make_rsrc makes, for inline assembly
    const uint64_t a = (uint64_t)(uintptr_t)base;
    return u32x4{(uint32_t)a, (uint32_t)(a >> 32), bytes, 0x00020000u};
  };
  // A tile's first column in the chunk, and how many it has.  Where the grid has columns to spare, the chunk's tiles but the
  // first start up to 12 columns early (p.col_align), at a 64-byte granule of R's rows (see column_align), and the
  // first one has that many fewer.
  // OVERLAP: all of them overlap by p.overlap columns, which both compute, and every row is cut between them where its granule ends (see
  // column_overlap).  An instantiation of its own: in one with the others its arithmetic cost launches of one short tile 0.1 to 0.3 us.
  auto col_at = [&](const Tile &t) {
    if constexpr (OVERLAP) return t.nj * (BN - p.overlap);
    else return t.nj * BN - (t.nj ? (t.c * p.W) & p.col_align : 0);
  };
  auto cols_of = [&](const Tile &t, int at) {
    if constexpr (OVERLAP) return min(BN, p.W - at);
    else return t.nj ? min(BN, p.W - at) : min(BN - ((t.c * p.W) & p.col_align), p.W);
  };
  u32x4 descA, descB;
  // Which of a lane's copies lie outside in the piece's last slab (K-contiguous, ragged K) or throughout (transposed,
  // columns past the tile's end): their offsets get the top bit, the others lose it.
  auto mark = [](uint32_t off, bool outside) { return outside ? off | kOob : off & ~kOob; };
  bool markedA = false, markedB = false;         // some have it
  // The stream's piece in bytes from where the descriptors point, in A and in B (one value where both are K-contiguous): the next
  // slab copied, the piece's first, and behind its last full one.
  struct Walk {
    uint32_t at, begin, end;
  };
  Walk walkA, walkB;
  auto stream_to = [&](const Piece &w) {
    const int m0 = w.tl.mi * BM, at = col_at(w.tl), n0 = w.tl.c * p.W + at;
    const int rows = min(BM, p.M - m0), cols = cols_of(w.tl, at);
    // (arrays of less than 2^31 elements: offsets in them are 32-bit products)
    const uint32_t lda = (uint32_t)p.lda, ldb = (uint32_t)p.ldb;
    descA = AKM ? descriptor(p.A + m0, ((uint32_t)p.K * lda - m0) * 2u) : descriptor(p.A + (uint32_t)m0 * lda, (uint32_t)rows * lda * 2u);
    descB = BKN ? descriptor(p.B + n0, ((uint32_t)p.K * ldb - n0) * 2u) : descriptor(p.B + (uint32_t)n0 * ldb, (uint32_t)cols * ldb * 2u);
    const bool cutA = AKM && rows < BM, cutB = BKN && cols < BN;
    if (cutA || markedA) {
#pragma unroll
      for (int q = 0; q < NA; ++q) {
        int k, col = 0;
        if (AKM) tr_at((wave * NA + q) * 1024 + lane * 16, kARow, sw_mask(BM / 16), k, col);
        offA[q] = mark(offA[q], AKM && col >= rows);
      }
      markedA = cutA;
    }
    if (cutB || markedB) {
#pragma unroll
      for (int q = 0; q < NB; ++q) {
        int k, col = 0;
        if (BKN) tr_at((wave * NB + q) * 1024 + lane * 16, kBRow, sw_mask(BN / 16), k, col);
        offB[q] = mark(offB[q], BKN && col >= cols);
      }
      markedB = cutB;
    }
    // K walks start at another slab on every XCD (p.k_groups of them) and wrap around: the chip reads as many
    // K ranges at a time instead of one, which spreads the traffic over the memory channels
    const int off = p.k_groups > 1 ? (int)div_by((blockIdx.x - div_by(blockIdx.x, p.by_groups) * (uint32_t)p.k_groups) * (uint32_t)w.nf, p.by_groups) : 0;
    // (the same in every lane: said so, so that a slab's addresses are formed in scalar registers)
    auto walk = [&](uint32_t step) {
      return Walk{(uint32_t)__builtin_amdgcn_readfirstlane((w.k0 + off) * step), (uint32_t)__builtin_amdgcn_readfirstlane(w.k0 * step),
                  (uint32_t)__builtin_amdgcn_readfirstlane((w.k0 + w.nf) * step)};
    };
    walkA = walk(a_step);
    if (AKM || BKN) walkB = walk(b_step);
  };
  auto stream_ragged = [&]() {                   // the stream's last slab ends with K: nothing behind it
    if constexpr (!AKM && !BKN) {
      walkA.at = walkA.end;
#pragma unroll
      for (int q = 0; q < NA; ++q) offA[q] = mark(offA[q], k_chunk(q) * 8 >= ktail);
#pragma unroll
      for (int q = 0; q < NB; ++q) offB[q] = mark(offB[q], k_chunk(q) * 8 >= ktail);
      markedA = markedB = true;
    }
  };
  auto stream_end = [&]() { descA[2] = descB[2] = 0u; };          // (buffers of no bytes)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
  auto copy_one = [&](auto Q, uint32_t so) {     // of the slab the walks are at
    constexpr int q = decltype(Q)::value;
    constexpr bool a = q < NA;
    const uint32_t dst = lds_base + so + (a ? wave * (NA * 1024) + q * 1024 : kBOff + wave * (NB * 1024) + (q - NA) * 1024);
    const uint32_t off = a ? offA[a ? q : 0] : offB[a ? 0 : q - NA], soff = a || !(AKM || BKN) ? walkA.at : walkB.at;
    const u32x4 desc = a ? descA : descB;
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 : : "s"(dst), "v"(off), "s"(desc), "s"(soff) : "memory", "m0");
  };
#pragma clang diagnostic pop
  auto slab_next = [&]() {                       // on to the slab behind the one copied last
    auto next = [](Walk &w, uint32_t step) {
      uint32_t at = w.at + step;
      if (at == w.end) at = w.begin;
      asm volatile("" : "+s"(at));
      w.at = at;
    };
    next(walkA, a_step);
    if (AKM || BKN) next(walkB, b_step);
  };

  // ---- operand addresses (see gemm_tile_kernel)
  const int fr = lane & 15, fq = lane >> 4, fs = swz(fr);
  uint32_t adA[2], adB[2];                       // (K-contiguous) this lane's row of k-step kk
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) {
    const uint32_t pos = ((4 * kk + fq) ^ fs) * 16;
    adA[kk] = lds_base + (AKM ? (8 * fq + (fr >> 2)) * kARow + (fr & 3) * 8 : (wm * WM + fr) * kRowBytes + pos);
    adB[kk] = lds_base + kBOff + (BKN ? (8 * fq + (fr >> 2)) * kBRow + (fr & 3) * 8 : (wn * WN + fr) * kRowBytes + pos);
  }
  uint32_t colA[AKM ? FM : 1], colB[BKN ? FN : 1];     // (transposed) byte position of block i's 32-byte piece
  if constexpr (AKM) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
      colA[i] = ((wm * FM + i) ^ (((fr >> 2) | ((fq & 1) << 2)) & sw_mask(BM / 16))) << 5;
  }
  if constexpr (BKN) {
#pragma unroll
    for (int j = 0; j < FN; ++j)
      colB[j] = ((wn * FN + j) ^ (((fr >> 2) | ((fq & 1) << 2)) & sw_mask(BN / 16))) << 5;
  }

  using OpA = Operands<FM, AKM != 0>;
  using OpB = Operands<FN, BKN != 0>;
  OpA xa[2];
  OpB xb[2];
  constexpr int NR = OpA::kReads + OpB::kReads, RA = AKM ? 2 : 1, RB = BKN ? 2 : 1;
  constexpr int NP = FM * FN;                    // products of a k-step
  constexpr int kGap = NP - 6 >= 3 * NR ? 3 : (NP - 6 >= 2 * NR ? 2 : 1);       // one operand read per kGap products,
  constexpr int kGapC = NP >= 3 * NL ? 3 : (NP >= 2 * NL ? 2 : 1);              //   one copy per kGapC
  static_assert(kGap * NR <= NP && kGapC * NL <= NP, "reads and copies fit a k-step");
  // read r of a k-step, in the order the products need them: B block 0, A block 0, the other B
  // blocks, the other A blocks
  auto read_a = [&](auto I, auto H, auto SET, auto KK, uint32_t a_addr) {
    constexpr int i = decltype(I)::value, set = decltype(SET)::value, kk = decltype(KK)::value;
    if constexpr (!AKM) asm_ds_read_b128<i * 16 * kRowBytes>(xa[set].v[i], a_addr);
    else if constexpr (decltype(H)::value == 0) asm_ds_read_tr<32 * kk * kARow>(xa[set].lo[i], a_addr + colA[i]);
    else asm_ds_read_tr<(32 * kk + 4) * kARow>(xa[set].hi[i], a_addr + colA[i]);
  };
  auto read_b = [&](auto J, auto H, auto SET, auto KK, uint32_t b_addr) {
    constexpr int j = decltype(J)::value, set = decltype(SET)::value, kk = decltype(KK)::value;
    if constexpr (!BKN) asm_ds_read_b128<j * 16 * kRowBytes>(xb[set].v[j], b_addr);
    else if constexpr (decltype(H)::value == 0) asm_ds_read_tr<32 * kk * kBRow>(xb[set].lo[j], b_addr + colB[j]);
    else asm_ds_read_tr<(32 * kk + 4) * kBRow>(xb[set].hi[j], b_addr + colB[j]);
  };
  auto read_op = [&](auto R, auto SET, auto KK, uint32_t a_addr, uint32_t b_addr) {
    constexpr int r = decltype(R)::value;
    if constexpr (r < RB) read_b(std::integral_constant<int, 0>{}, std::integral_constant<int, r>{}, SET, KK, b_addr);
    else if constexpr (r < RB + RA) read_a(std::integral_constant<int, 0>{}, std::integral_constant<int, r - RB>{}, SET, KK, a_addr);
    else if constexpr (r < RA + RB * FN)
      read_b(std::integral_constant<int, (r - RA) / RB>{}, std::integral_constant<int, (r - RA) % RB>{}, SET, KK, b_addr);
    else
      read_a(std::integral_constant<int, (r - RB * FN) / RA>{}, std::integral_constant<int, (r - RB * FN) % RA>{}, SET, KK, a_addr);
  };
  f32x4 acc[FM][FN];
  // One k-step: the products of operand set CS, (READS) k-step KK's operands of the stage at `sr` into the
  // other set, and (COPIES) the stream's slab into the stage at `sc`.  `under`: what else is to be done under the products.
  auto kstep = [&](auto FIRST, auto CS, auto KK, auto READS, auto COPIES, uint32_t sr, uint32_t sc, auto under) {
    constexpr int cs = decltype(CS)::value, kk = decltype(KK)::value;
    uint32_t a_addr = 0, b_addr = 0;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");            // this k-step's operands have landed
    xa[cs].tie();
    xb[cs].tie();
    if constexpr (kOneWave && !decltype(FIRST)::value) {                    // (accumulators: the accumulation half of the register file)
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) asm_accumulator(acc[i][j]);
    }
    __builtin_amdgcn_sched_barrier(0);
    static_for<NP>([&](auto Mi) {
      constexpr int m = decltype(Mi)::value, i = m / FN, j = m % FN;
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xb[cs].template get<j>(), xa[cs].template get<i>(), decltype(FIRST)::value ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);                          // nothing moves across: the order is as written
      if constexpr (m == 0) {
        a_addr = adA[AKM ? 0 : kk] + sr;
        b_addr = adB[BKN ? 0 : kk] + sr;
      }
      if constexpr (m == 4) {
        under();
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (decltype(READS)::value && m % kGap == 0 && m / kGap < NR) {
        read_op(std::integral_constant<int, m / kGap>{}, std::integral_constant<int, cs ^ 1>{}, KK, a_addr, b_addr);
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (decltype(COPIES)::value && m % kGapC == (kGapC > 1 ? 1 : 0) && m / kGapC < NL) {
        copy_one(std::integral_constant<int, m / kGapC>{}, sc);
        __builtin_amdgcn_sched_barrier(0);
      }
    });
  };
  using std::false_type;
  using std::true_type;
  constexpr std::integral_constant<int, 0> c0{};
  constexpr std::integral_constant<int, 1> c1{};

  // ---- the way out.  Image of a row block: 2 strips (wm) x 16 rows x BN columns; chunk k (16 bytes) of
  // image row ir at k ^ (ir & 7) (both sides free of bank conflicts).  Wavefront w reads rows 8 w .. 8 w + 7
  // in FN accesses of 64 consecutive chunks; access u is at image row ir(u), column col(u) of the tile,
  // and the rows of access u + UB are those of access u plus RS.
  // (OVERLAP: four rows, over which the place of the granules in a row repeats)
  constexpr int kRowCh = BN / 4, UB = OVERLAP ? BN / 64 : (BN == 192 ? 3 : 1), RS = UB * 64 / kRowCh;
  static_assert(UB * 64 == RS * kRowCh && FN % UB == 0, "");
  auto strip_row = [](int ir) { return (ir >> 4) * WM + (ir & 15); };   // image row -> tile row, row block 0

  Piece cur;
  get_piece(words, 0, cur);                      // (the grid is no larger than the number of pieces)
  p = words.now();
  stream_to(cur);
#pragma unroll
  for (int j = 0; j < NSTAGE; ++j) {
    if (j) slab_next();
    if (ktail && j == cur.ns - 1 && cur.ns > cur.nf) stream_ragged();
    static_for<NL>([&](auto Q) { copy_one(Q, (uint32_t)(j * kStageBytes)); });
  }
  asm volatile("s_waitcnt vmcnt(%0)" : : "n"((NSTAGE - 1) * NL) : "memory");      // slab 0 landed
  uint32_t so = 0;                               // byte offset of the stage that holds the current slab
  auto flush = [&]() {                           // the pending count at once
    if (pending.c < 0 && pending_half < 0) return;
    __builtin_amdgcn_s_waitcnt(kWaitAll);
    __syncthreads();
    ask_count();
    __builtin_amdgcn_s_waitcnt(kWaitVm0);        // (in every wavefront: nothing is on its way where paths meet)
    act_on_count();
  };
  auto next_stage = [](uint32_t s) {
    s += (uint32_t)kStageBytes;
    return s == (uint32_t)(NSTAGE * kStageBytes) ? 0u : s;
  };

  for (int it = 0;; ++it) {
    stamp(it, 0);
    const Tile tl = cur.tl;
    p = words.now();
    const bool has_in = cur.half == 2 || (tracked && !((p.flags & kFlagStep0StoreOnly) && tl.s == 0));

    if (cur.ns <= NSTAGE) flush();               // (too short a K loop to put the count off into)
    if (cur.half == 2 && wave == 0) {
      p = words.now();
      // The first half was computed by a workgroup with a lower index as its first piece of work and
      // waits for nothing, so this wait ends (normally at once).
      const TrkWave flag{make_rsrc(p.tail_flags + cur.idx, 4u), p.tail_flags + cur.idx, lane_at};
      int spins = 0;
      while (flag.get(flag.base) == 0u && ++spins < kSpinLimit) __builtin_amdgcn_s_sleep(16);
      if (tracked && spins >= kSpinLimit) tracker().put(trk_at(p, gen).error, 1u);
      // (this workgroup is the flag's only reader: cleared for the next launch)
      flag.put(flag.base, 0u);
      __builtin_amdgcn_s_waitcnt(kWaitVm0);
    }
    // slab 0 of this piece is in LDS (every wavefront has seen its own copies land); the images are free
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    stamp(it, 1);
    static_for<NR>([&](auto R) { read_op(R, c0, c0, adA[0] + so, adB[0] + so); });

    f32x4 in[FM][FN];
    __amdgpu_buffer_rsrc_t in_rsrc;
    uint32_t in_at[UB], ld_in;
    auto load_in = [&](auto I) {                 // row block I of the incoming partial
      constexpr int i = decltype(I)::value;
      static_for<FN>([&](auto U) {
        constexpr int u = decltype(U)::value;
        in[i][u] = __builtin_bit_cast(
            f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                       in_rsrc, (int)(in_at[u % UB] + (uint32_t)(16 * i + (u / UB) * RS) * ld_in * 4u), 0, kAuxSc1 | kAuxNt));
      });
    };
    // Where this piece's results go, worked out where it is wanted rather than kept through the main loop.
    struct Place {
      int cols_in;                               // rows and columns of the tile inside the chunk
      uint32_t rows_in, ld_out, first, row;      // first, row: where its rows start in a granule (in R as if R's started at one)
      float *slot_at0, *r_at0, *out_base;        // the tile's first element in the slot, in R or C, where its fp32 sums go
      bool bf16, to_slot, to_r;
    };
    auto place = [&]() {
      Place o;
      const int m0 = tl.mi * BM, at = col_at(tl), n0 = tl.c * p.W + at;
      o.rows_in = (uint32_t)min(BM, p.M - m0);
      o.cols_in = cols_of(tl, at);
      const bool direct = (p.flags & kFlagFwdDirect) != 0;
      o.bf16 = (p.flags & kFlagFwdBf16) != 0;
      o.to_slot = tracked && tl.c != p.own && cur.half != 1 && (direct || chunk_is_whole(p, tl.s));
      o.to_r = !tracked || !direct || tl.c == p.own;
      // where a whole tile's fp32 sums go, or half a tile's (an fp32 slot if not R / C)
      const bool out_slot = tracked && direct && tl.c != p.own;
      o.slot_at0 = p.fwd + (((int64_t)tl.s * p.M + m0) * p.W + at);
      o.r_at0 = p.R + ((uint32_t)m0 * (uint32_t)p.ldr + (uint32_t)n0);
      o.out_base = out_slot ? o.slot_at0 : o.r_at0;
      o.ld_out = out_slot ? (uint32_t)p.W : (uint32_t)p.ldr;
      o.row = OVERLAP && out_slot ? (uint32_t)p.W : 0u;
      o.first = out_slot ? (uint32_t)(tl.s * p.M + m0) * (uint32_t)p.W + (uint32_t)at : (uint32_t)n0;
      return o;
    };
    // This lane's row and column in access u, and which of the UB accesses' columns are this tile's to write
    auto lane_row = [&](int l, int u) { return strip_row(wave * 8 + (u * 64 + l) / kRowCh); };
    auto lane_col = [&](int l, int u) { return ((u * 64 + l) % kRowCh) * 4; };
    auto inside = [&](const Place &o, int l, bool (&in)[UB]) {
#pragma unroll
      for (int u = 0; u < UB; ++u) in[u] = lane_col(l, u) < o.cols_in;
      if constexpr (OVERLAP) {
        const uint32_t next = (uint32_t)(BN - p.overlap), mask = (uint32_t)p.granule - 1u;
#pragma unroll
        for (int u = 0; u < UB; ++u) {
          const uint32_t e = o.first + (uint32_t)lane_row(l, u) * o.row;
          const int col = lane_col(l, u);
          if (tl.nj && col < (int)(-e & mask)) in[u] = false;
          if (tl.nj < p.Wt - 1 && col >= (int)(next + (-(e + next) & mask))) in[u] = false;
        }
      }
    };
    // Byte offsets of the UB accesses in rows of `ld` elements of `size` bytes (where 64 lanes are whole rows, access u is u * 64 / kRowCh rows behind access 0)
    auto offsets = [&](int l, uint32_t ld, uint32_t size, const bool (&in)[UB], uint32_t (&at)[UB]) {
      const uint32_t at0 = ((uint32_t)lane_row(l, 0) * ld + (uint32_t)lane_col(l, 0)) * size;
#pragma unroll
      for (int u = 0; u < UB; ++u) {
        const uint32_t here = 64 % kRowCh == 0 ? at0 + (uint32_t)(u * 64 / kRowCh) * ld * size
                                               : ((uint32_t)lane_row(l, u) * ld + (uint32_t)lane_col(l, u)) * size;
        at[u] = in[u] ? here : kOob;
      }
    };
    auto in_here = [&](const Place &o) {
      // the incoming partial, or the first half's partial sums where the result will go
      ld_in = cur.half == 2 ? o.ld_out : (uint32_t)p.ldr;
      in_rsrc = make_rsrc(cur.half == 2 ? o.out_base : o.r_at0, o.rows_in * ld_in * 4u);
      bool in[UB];
      inside(o, lane, in);
      offsets(lane, ld_in, 4u, in, in_at);
    };
    Piece nxt;
    bool more = false;
    // The K loop.  A slab is two k-steps with a barrier between them, behind which the slab's stage is free and
    // the next slab visible; the loop runs from barrier to barrier and is left where something has to be done behind
    // one (the count, the stream's last slab, its next piece) or a barrier waits for something else.  One wavefront per SIMD,
    // and it issues an instruction every four clocks at best: what stands between two products in the loop is time the matrix
    // cores idle, so a barrier is a wait and one test away from the last product, the next slab's place is worked out under the
    // products before it, everything rare is outside, and the first k-step, ahead of the loop, starts the sums from a constant
    // zero instead of 256 cleared registers.  (With all of it in the
    // loop, and one kernel for both modes: plain GEMM 4096 x 12288 x 1536 132.0 us, now 126.5; 16384 x 3072 x 1536
    // 141.6, 131.7; 4096 x 12288 x 6144 422.4, 415.1; fused 452.5, 444.6.)
    int kt = 0;                                  // slab multiplied; slab kt + NSTAGE, or as many of the next piece, is copied next
    const int last = cur.ns - 1, k_switch = cur.ns - NSTAGE;      // behind k_switch's barrier the stream goes on to the next piece
    const bool counting = pending.c >= 0 || pending_half >= 0;
    uint32_t sn;                                 // the next slab's stage
    auto first_half = [&](auto FIRST) {
      kstep(FIRST, c0, c1, true_type{}, false_type{}, so, 0u, [&]() {
        sn = next_stage(so);
        slab_next();
        asm volatile("" : "+s"(sn));
      });
    };
    auto barrier = [&]() {                       // this wavefront's own reads of the slab are done as well
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
    };
    // What it waits for beside them: the next slab's copies, with the incoming partial requested behind them or not; or nothing
    // (the first slabs of every piece but the first landed during the way out, and behind the last slab nothing is needed).
    auto next_landed = [&]() { asm volatile("s_waitcnt vmcnt(%0)" : : "n"((NSTAGE - 2) * NL) : "memory"); };
    auto next_landed_in = [&]() { asm volatile("s_waitcnt vmcnt(%0)" : : "n"((NSTAGE - 2) * NL + PRE * FN) : "memory"); };
    first_half(true_type{});
    if (it == 0 && last > 0) next_landed();
    barrier();
    for (;;) {                                   // behind the barrier of slab kt (left by equality: another test has the
                                                 //   compiler keep two sets of accumulators)
      if (counting && kt >= NSTAGE - 1) {        // (the previous piece's stores are older than copies that have been waited for)
        if (kt == NSTAGE - 1 && kt < last) ask_count();
        if (kt == NSTAGE) act_on_count();
      }
      if (kt == k_switch) {
        more = get_piece(words, it + 1, nxt);
        p = words.now();
        if (more) stream_to(nxt);
        else stream_end();
        if (tracked && has_in) {
          p = words.now();
          in_here(place());
          static_for<PRE>([&](auto I) { load_in(I); });
        }
      }
      // the slab copied next is the last one of the stream's piece, and ragged
      if (ktail && (kt == k_switch - 1 || (kt == last && more && nxt.ns == NSTAGE)) && (kt < k_switch ? cur.ns > cur.nf : nxt.ns > nxt.nf))
        stream_ragged();
      // the next barrier something is to be done behind, or whose wait is another one
      int stop = kt < k_switch ? (ktail && kt < k_switch - 1 ? k_switch - 1 : k_switch) : (NSTAGE > 2 && kt < last - 1 ? kt + 1 : last);
      if (kt < NSTAGE && (counting || (NSTAGE > 2 && it > 0))) stop = min(stop, kt + 1);
      const int kind = kt + 1 == last || (it > 0 && kt + 1 < NSTAGE - 1) ? 2 : (NSTAGE > 2 && kt >= k_switch && tracked && has_in ? 1 : 0);
      do {
        kstep(false_type{}, c1, c0, true_type{}, true_type{}, sn, so, []() {});     // (behind the last slab it reads what nobody uses)
        so = sn;
        ++kt;
        // (the first k-step's wait, ahead of the branch: whatever the compiler keeps in registers along the way out of
        // the loop is not in those that reads are on their way to)
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        xa[0].tie();
        xb[0].tie();
        if (kt == cur.ns) break;
        first_half(false_type{});
        if (kind == 0) next_landed();
        else if (kind == 1) next_landed_in();
        barrier();
      } while (kt < stop);
      if (kt == cur.ns) break;
    }
    stamp(it, 2);

    p = words.now();
    const Place to = place();
    const bool nt_out = p.nt_out != 0;
    auto zero_in = [&](auto I) {
#pragma unroll
      for (int u = 0; u < FN; ++u) in[decltype(I)::value][u] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    int lane_e = lane;                           // recomputed here rather than kept through the main loop
    asm volatile("" : "+v"(lane_e));
    const int e_row = lane_e & 15, e_q = lane_e >> 4;
    // TO: -1 = fp32 to C, kept in the caches; 0 = fp32 to R, C or a slot, streamed; 1 = R and the fp32 slot; 2 = the bfloat16 slot; 3 = R and the bfloat16 slot
    // ADD: there is something to add
    auto way_out = [&](auto TO, auto ADD) {
      constexpr int kTo = decltype(TO)::value;
      constexpr bool add = decltype(ADD)::value;
      const uint32_t ld_out = to.ld_out, W = (uint32_t)p.W;
      if constexpr (add && tracked) {
        if (has_in) static_for<DEPTH - PRE>([&](auto I) { load_in(std::integral_constant<int, decltype(I)::value + PRE>{}); });
        else static_for<DEPTH>(zero_in);
      } else if constexpr (add) {
        in_here(to);
        static_for<DEPTH>(load_in);
      }
      const __amdgpu_buffer_rsrc_t out_rsrc = make_rsrc(to.out_base, to.rows_in * ld_out * 4u);
      const void *slot = kTo >= 2 ? (const void *)((const uint16_t *)p.fwd + (to.slot_at0 - p.fwd)) : (const void *)to.slot_at0;
      const __amdgpu_buffer_rsrc_t slot_rsrc = make_rsrc(slot, to.rows_in * W * (kTo >= 2 ? 2u : 4u));
      uint32_t out_at[UB], slot_at[UB], img_at[FN];
      bool in_tile[UB];
      inside(to, lane_e, in_tile);
      if (kTo != 2) offsets(lane_e, ld_out, 4u, in_tile, out_at);
      if (kTo >= 1) offsets(lane_e, W, kTo >= 2 ? 2u : 4u, in_tile, slot_at);
#pragma unroll
      for (int u = 0; u < FN; ++u) {
        const int L = u * 64 + lane_e, ir = wave * 8 + L / kRowCh;
        img_at[u] = kImgOff + ir * (BN * 4) + (((L % kRowCh) ^ (ir & 7)) << 4);
      }
      static_for<FM>([&](auto I) {
        constexpr int i = decltype(I)::value;
        constexpr int img = (i % NIMG) * kImgBytes;
        if constexpr (NIMG == 1 && i > 0) {      // everyone has read the image
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
          __builtin_amdgcn_s_barrier();
          asm volatile("" ::: "memory");
        }
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          *(f32x4 *)(lds + kImgOff + img + (wm * 16 + e_row) * (BN * 4) + (((wn * (WN / 4) + 4 * j + e_q) ^ (e_row & 7)) << 4)) = acc[i][j];
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        static_for<FN>([&](auto U) {
          constexpr int u = decltype(U)::value;
          f32x4 v = *(const f32x4 *)(lds + img + img_at[u]);
          if constexpr (add) v += in[i][u];
          const uint32_t rows = (uint32_t)(16 * i + (u / UB) * RS);
          if constexpr (kTo != 2) store_agent_hint<(kTo >= 0)>(out_rsrc, out_at[u % UB] + rows * ld_out * 4u, 0u, v);
          if constexpr (kTo == 1) store_agent_hint<true>(slot_rsrc, slot_at[u % UB] + rows * W * 4u, 0u, v);
          if constexpr (kTo >= 2)
            __builtin_amdgcn_raw_buffer_store_b64(pack_bf16(v), slot_rsrc, (int)(slot_at[u % UB] + rows * W * 2u), 0,
                                                  kAuxSc1 | kAuxNt);
        });
        if constexpr (add && i + DEPTH < FM) {
          if (!tracked || has_in) load_in(std::integral_constant<int, i + DEPTH>{});
          else zero_in(std::integral_constant<int, i + DEPTH>{});
        }
        // The next piece's first NSTAGE slabs were requested before the last of the incoming partial,
        // so they have landed when that is used; where they were not, this wait makes sure of it.
        if constexpr (i == 1) {
          if (!add || !has_in || (PRE == DEPTH && DEPTH == FM)) asm volatile("s_waitcnt vmcnt(%0)" : : "n"(2 * FN * (kTo <= 0 || kTo == 2 ? 1 : 2)) : "memory");
        }
        __builtin_amdgcn_sched_barrier(0);
      });
    };
    constexpr std::integral_constant<int, -1> keep{};
    if constexpr (tracked) {
      if (to.to_slot && to.bf16) {
        if (to.to_r) way_out(std::integral_constant<int, 3>{}, true_type{});
        else way_out(std::integral_constant<int, 2>{}, true_type{});
      } else if (to.to_slot && to.to_r) {
        way_out(c1, true_type{});
      } else {
        way_out(c0, true_type{});
      }
    } else if (cur.half == 2) {
      way_out(keep, true_type{});
    } else {
      if (nt_out) way_out(c0, false_type{});
      else way_out(keep, false_type{});
    }
    stamp(it, 3);
    if (cur.half == 1) pending_half = cur.idx;
    else if (tracked) pending = tl;
    if (!more) break;
    cur = nxt;
  }
  flush();
}

}  // namespace t3k
