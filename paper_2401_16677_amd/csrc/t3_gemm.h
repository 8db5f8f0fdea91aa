// Device code of the fused sliced-GEMM + reduce-scatter-reduction path for gfx950 (CDNA4).
//
// A persistent workgroup produces BM x BN output tiles with v_mfma_f32_16x16x32_bf16.  K-slabs of
// 64 bf16 of A and B are copied global -> LDS without passing through registers
// (global_load_lds_dwordx4) into two or three stages, ahead of the slab being multiplied; LDS
// rows are XOR-swizzled so that the MFMA operand reads are bank-conflict free.
//
// This is the kernel of what the wide-tile and small-tile kernels (t3_wide.h, t3_small.h) do not
// take: two writers, split-K, tile ranges that cut a ring step, arrays past 2 GiB, and K of one slab.
// Eight wavefronts (128 x 128: four), compiler-scheduled.
//
// The reduction of Sec. 4.3 of the T3 paper (op-and-store into the buffer that also receives
// the upstream partial) is done by starting the accumulators from the incoming partial, so a
// tile is read once and written once; both moves use full 128-byte lines and are transposed to
// and from the accumulator layout through LDS.
#pragma once

#include "t3_device.h"

namespace t3k {

// ---------------------------------------------------------------------------------------------
// LDS layout of one stage: BM rows of A then BN rows of B; a row holds the 64 bf16 of one tile
// row of the K-slab (128 bytes = 8 chunks of 16).  Row r keeps chunk k at position k ^ swz(r),
// which makes both the 1-KiB linear writes of the global->LDS copies (8 rows each) and the MFMA
// operand reads (16 consecutive rows, one chunk) bank-conflict free.
__device__ inline int swz(int r) { return (r & 7) ^ ((r >> 3) & 1); }

constexpr int kBK = 64;               // bf16 elements of K per slab
constexpr int kRowBytes = kBK * 2;    // one LDS row
constexpr int kCPR = 8;               // 16-byte chunks per row
constexpr int kRPC = 8;               // rows filled by one 1-KiB copy

// sched_group_barrier masks
constexpr int kSchedMfma = 0x008, kSchedDsRead = 0x100;

// Instruction order of one MFMA k-step: the operand reads of each of its MH row passes (AREADS
// for the row blocks; FN + EXTRA more in the first), each followed by that pass's FMH * FN products.
template <int MH, int FMH, int FN, int EXTRA, int AREADS = FMH>
__device__ inline void sched_kstep() {
  __builtin_amdgcn_sched_group_barrier(kSchedDsRead, AREADS + FN + EXTRA, 0);
  __builtin_amdgcn_sched_group_barrier(kSchedMfma, FMH * FN, 0);
  if constexpr (MH >= 2) {
    __builtin_amdgcn_sched_group_barrier(kSchedDsRead, AREADS, 0);
    __builtin_amdgcn_sched_group_barrier(kSchedMfma, FMH * FN, 0);
  }
  if constexpr (MH == 4) {
    __builtin_amdgcn_sched_group_barrier(kSchedDsRead, AREADS, 0);
    __builtin_amdgcn_sched_group_barrier(kSchedMfma, FMH * FN, 0);
    __builtin_amdgcn_sched_group_barrier(kSchedDsRead, AREADS, 0);
    __builtin_amdgcn_sched_group_barrier(kSchedMfma, FMH * FN, 0);
  }
}

// Compile-time loop: f(integral_constant<int, 0>) ... f(integral_constant<int, N-1>), so that the
// index can be used where a constant is required (instruction offsets, which register).
template <int I, int N, typename F>
__device__ __forceinline__ void static_for_impl(F &f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for_impl<I + 1, N>(f);
  }
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F f) {
  static_for_impl<0, N>(f);
}

// The memory instructions of the hand-ordered main loop, one volatile statement each: they are
// emitted in exactly the order written, and the waits they need are written out as well.  The
// products stay compiler builtins (the compiler must know them to keep the distances the
// hardware requires around them) and are fenced into place with scheduling barriers.
template <int OFF>
__device__ __forceinline__ void asm_ds_read_b128(bf16x8 &dst, uint32_t addr) {
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(OFF));
}
// "The operands of a k-step have landed": the wait is followed by statements that carry them as
// in/out operands, so that no product that uses them can be moved above it.
__device__ __forceinline__ void asm_tie(bf16x8 (&a)[8]) {
  asm volatile("" : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]), "+v"(a[6]), "+v"(a[7]));
}
__device__ __forceinline__ void asm_tie(bf16x8 (&a)[6]) {
  asm volatile("" : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]));
}
__device__ __forceinline__ void asm_tie(bf16x8 (&a)[4]) {
  asm volatile("" : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]));
}
constexpr int kRingSlots = 4;         // 1-KiB LDS slots per wavefront for transposing pairs: two pairs

// WAVES_M x WAVES_N wavefronts per workgroup, each producing a (BM/WAVES_M) x (BN/WAVES_N)
// block of the tile out of 16 x 16 MFMA blocks; NSTAGE LDS stages, NSTAGE-1 slabs in flight.
//
// The products are formed transposed (the B rows go in as the MFMA's first operand, the A rows
// as its second), so that a lane ends up holding, per block, one output row and FOUR
// CONSECUTIVE COLUMNS: the incoming partial is read and the sum written with 16-byte accesses.
//
// BKN = 1: B is stored K x N with N contiguous (the layout of the backward-pass GEMMs).  Its
// stage region then holds 64 k-rows of BN values; the MFMA operand (8 consecutive k for one n
// per lane) is fetched with the transposing LDS read ds_read_b64_tr_b16: in each block of 16
// lanes, lane i supplies the address of 4 consecutive n of k-row i / 4 (n offset 4 (i % 4)) and
// receives, for n = i, the values of the block's 4 k-rows.  32-byte pieces of a k-row sit at
// position (piece ^ sw(k)), sw(k) = (k & 3) | ((k >> 3) & 1) << 2, which spreads the 8 k-rows
// that 32 lanes read together over all banks.  K must be a multiple of 64 in this layout.
//
// AKM = 1: A is stored K x M with M contiguous (the transposed operand of the backward-pass
// GEMMs, Sec. 5.2): the same arrangement on the A side -- its stage region holds 64 k-rows of BM
// values, pieces swizzled the same way, operands fetched with the transposing read.  K must be
// a multiple of 64 and M a multiple of 8.
template <int BM, int BN, int WAVES_M, int WAVES_N, int NSTAGE, int MODE, int BKN, int AKM>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N)
__attribute__((amdgpu_waves_per_eu(2)))
void gemm_tile_kernel(const Plan p) {
  constexpr int NW = WAVES_M * WAVES_N;
  constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;   // wavefront tile
  constexpr int FM = WM / 16, FN = WN / 16;     // 16x16 MFMA blocks per wavefront
  constexpr int MH = FM > 4 ? T3_MH : 1;        // a k-step is taken in MH passes over the rows,
  constexpr int FMH = FM / MH;                  //   FMH row blocks each, to bound operand registers
  constexpr int KS = kBK / 32;                  // MFMA k-steps per slab
  constexpr int US = KS * MH;                   // micro-steps (row pass of a k-step) per slab
  constexpr int NA = BM / kRPC / NW, NB = BN / kRPC / NW;   // copies per wavefront per slab
  constexpr int NL = NA + NB;
  constexpr int NBLK = FM * FN;
  constexpr int kStageBytes = (BM + BN) * kRowBytes;
  constexpr int kBOff = BM * kRowBytes;
  static_assert(NA * kRPC * NW == BM && NB * kRPC * NW == BN, "copies must tile the slab");
  static_assert(NSTAGE >= 2 && (NSTAGE - 2) * NL < 64, "vmcnt range");
  static_assert(KS == 2, "the loop body is written as two k-steps");
  static_assert(NL % MH == 0, "a slab's copies are split evenly over the first k-step's passes");
  static_assert(NSTAGE * kStageBytes <= 160 * 1024, "LDS");

  static_assert(NW * kRingSlots * 1024 <= kStageBytes, "scratch of the pair transpositions: the last stage");

  __shared__ __attribute__((aligned(1024))) char lds[NSTAGE * kStageBytes];

  // Persistent workgroups: workgroup w takes grid positions w, w + p.resident, ... in order (see work_item).  The tracking of a finished tile is
  // deferred into the next tile: by the first barrier of that tile's main loop every
  // wavefront has waited for its stores (they are older than the slab copies waited for
  // there), so the acknowledgement wait costs nothing.
  constexpr bool tracked = MODE == kModeFused;
  Trk trk;
  if (tracked) trk = trk_open(p);              // reads gen now; used when tiles are done
  if (p.stagger_groups > 1) stagger_start(p, 0u);

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;
  Tile pending{0, -1, 0, 0};                   // the tile whose stores are issued but not counted (c < 0: none)
  // To be called after a barrier that every wavefront reached with its stores acknowledged.  (The count's
  // request and its use behind ONE branch: as two, the compiler sees a way past the use and puts a wait for
  // every access in flight into the main loop, where the request's registers are used again.  4096 x 12288 x 1536
  // from the second tile on, tiles of 256 x 128: 191 us as two, 183 as one; of 128 x 256: 194 and 181.)
  auto settle_pending = [&]() {
    if (tracked && pending.c >= 0 && threadIdx.x == 0)
      track_finish(p, trk, pending, track_issue(p, trk, pending), p.whole_chunks != 0, TrkThread{});
    pending.c = -1;
  };
  auto flush_pending = [&]() {
    if (tracked && pending.c >= 0) {
      __builtin_amdgcn_s_waitcnt(kWaitAll);
      __syncthreads();
      settle_pending();
    }
  };

  // (not in the eight-wavefront 256 x 256 kernels: they have no register to spare)
  constexpr bool kTimeline = !(NW == 8 && FM == 8);
  auto stamp = [&](int it, int k) {
    if (kTimeline && p.timeline && threadIdx.x == 0 && (int)blockIdx.x < p.timeline_wgs && it < kTimelineItems)
      p.timeline[((size_t)blockIdx.x * kTimelineItems + it) * 4 + k] = wall_clock64();
  };

  f32x4 acc[FM][FN];
  for (int it = 0;; ++it) {
  // Parts of K (split-K in two-writer mode): part j
  // takes K-slabs [j q, (j+1) q) of the K / 64 full ones, the last part also what is left over
  int blk, part, nparts;
  if (!work_item<0>(p, it, blk, part, nparts)) break;
  stamp(it, 0);
  const int part_slabs = (p.K / kBK) / nparts;
  const int k0 = part * part_slabs * kBK;
  const int Kpart = (part == nparts - 1) ? p.K - k0 : part_slabs * kBK;
  const char *const Ap = (const char *)p.A + (AKM ? (int64_t)k0 * p.lda * 2 : (int64_t)k0 * 2);
  const char *const Bp = (const char *)p.B + (BKN ? (int64_t)k0 * p.ldb * 2 : (int64_t)k0 * 2);
  Tile tl;
  if (!decode_block(p, blk, tl)) continue;
  __syncthreads();                             // the previous tile's epilogue is done with the LDS

  const int m0 = tl.mi * BM;
  const int col_lo = tl.c * p.W;                 // chunk bounds in N
  const int col_hi = col_lo + p.W;
  const int n0 = col_lo + tl.nj * BN;

  const int nkf = Kpart / kBK;                   // full slabs
  const int ktail = Kpart - nkf * kBK;           // leftover elements of K (a multiple of 8)
  // Workgroups that run on different XCDs walk K from different starting slabs (and wrap
  // around): at any moment the chip then reads 8 different K ranges of A and B instead of one,
  // which spreads the traffic over the memory channels, and what one XCD misses in its L2
  // another has usually brought into the memory-side cache already.  Workgroups of one XCD
  // (same index modulo the group count) keep the same offset, so they still share slabs in L2.
  const int koff = p.k_groups > 1
                       ? (int)(((uint32_t)(blockIdx.x % (uint32_t)p.k_groups) * (uint32_t)nkf) / (uint32_t)p.k_groups)
                       : 0;
  // ---- global -> LDS copy addressing.  Copy q of this wavefront fills 8 LDS rows (1 KiB):
  // lane l lands in row l / 8, position l % 8, so it must fetch chunk (l % 8) ^ swz(row).
  const int cp_row = lane / kCPR;
  uint32_t offA[NA], offB[NB];                   // byte offsets, rows clamped into range
  auto chunk_of = [&](int rows_per_wave, int q) {  // the k-chunk copy q of this lane fetches
    return (lane % kCPR) ^ swz(wave * rows_per_wave + q * kRPC + cp_row);
  };
  constexpr int kARowBytes = BM * 2;             // (AKM) one k-row of the A region
  constexpr int kSwMaskA = (BM / 16 < 8 ? BM / 16 : 8) - 1;
#pragma unroll
  for (int q = 0; q < NA; ++q) {
    if (AKM) {
      // as for B stored K x N below: copy (wave * NA + q) fills 1 KiB of the A region, lane l
      // lands in k-row L / kARowBytes at 16-byte position cp = half (cp & 1) of piece (cp >> 1) ^ sw(k)
      const int L = (wave * NA + q) * 1024 + lane * 16;
      const int k = L / kARowBytes, cp = (L % kARowBytes) / 16;
      const int sw = ((k & 3) | (((k >> 3) & 1) << 2)) & kSwMaskA;
      const int mcol = (((cp >> 1) ^ sw) * 2 + (cp & 1)) * 8;
      offA[q] = (uint32_t)((k * p.lda + min(m0 + mcol, p.M - 8)) * 2);
    } else {
      const int r = wave * (BM / NW) + q * kRPC + cp_row;
      offA[q] = (uint32_t)((min(m0 + r, p.M - 1) * p.lda + chunk_of(BM / NW, q) * 8) * 2);
    }
  }
  constexpr int kBRowBytes = BN * 2;             // (BKN) one k-row of the B region
  constexpr int kSwMask = (BN / 16 < 8 ? BN / 16 : 8) - 1;
#pragma unroll
  for (int q = 0; q < NB; ++q) {
    if (BKN) {
      // copy (wave * NB + q) fills bytes [1024 (wave NB + q), +1024) of the B region: lane l
      // lands in k-row L / kBRowBytes at 16-byte position cp, which holds half (cp & 1) of
      // 32-byte piece (cp >> 1) ^ sw(k)
      const int L = (wave * NB + q) * 1024 + lane * 16;
      const int k = L / kBRowBytes, cp = (L % kBRowBytes) / 16;
      const int sw = ((k & 3) | (((k >> 3) & 1) << 2)) & kSwMask;
      const int ncol = (((cp >> 1) ^ sw) * 2 + (cp & 1)) * 8;
      offB[q] = (uint32_t)((k * p.ldb + min(n0 + ncol, col_hi - 8)) * 2);
    } else {
      const int r = wave * (BN / NW) + q * kRPC + cp_row;
      offB[q] = (uint32_t)((min(n0 + r, col_hi - 1) * p.ldb + chunk_of(BN / NW, q) * 8) * 2);
    }
  }
  const int ldsA_w = wave * (BM / NW) * kRowBytes;            // this wavefront's rows, stage 0
  const int ldsB_w = kBOff + wave * (BN / NW) * kRowBytes;

  // The copies are issued as inline assembly: the compiler would otherwise wait for every
  // outstanding global->LDS copy (vmcnt(0)) before any LDS read, which defeats the prefetch.
  // Waits for them are therefore explicit (s_waitcnt below).  Copies [q0, q1) of the slab's
  // NA + NB are issued by one call, so that a slab's copies can be spread over its micro-steps
  // (all eight wavefronts issuing all of theirs at once stalls them on the memory pipeline).
  // They write m0 (the LDS destination of the copy) and say so in their clobber lists, so the
  // compiler never assumes a value of its own survives them; it flags every clobber of that
  // register as "reserved", which is exactly what is meant here.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
  const uint32_t lds_base = (uint32_t)(uintptr_t)(lds_void_ptr)lds;
  auto issue_copies = [&](int kt, int stage, int q0, int q1) {
    kt += koff;                                   // slab kt of this workgroup's walk over K
    if (kt >= nkf) kt -= nkf;
    const char *a = Ap + (AKM ? (int64_t)kt * kBK * p.lda * 2 : (int64_t)kt * (kBK * 2));
    const char *b = Bp + (BKN ? (int64_t)kt * kBK * p.ldb * 2 : (int64_t)kt * (kBK * 2));
    const uint32_t dst = lds_base + stage * kStageBytes;
#pragma unroll
    for (int q = 0; q < NA; ++q)
      if (q >= q0 && q < q1)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                     :
                     : "s"(dst + ldsA_w + q * 1024), "v"(offA[q]), "s"(a)
                     : "memory", "m0");
#pragma unroll
    for (int q = 0; q < NB; ++q)
      if (NA + q >= q0 && NA + q < q1)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                     :
                     : "s"(dst + ldsB_w + q * 1024), "v"(offB[q]), "s"(b)
                     : "memory", "m0");
  };
#pragma clang diagnostic pop
  auto issue_slab = [&](int kt, int stage) { issue_copies(kt, stage, 0, NL); };

  // ---- MFMA operand addressing (v_mfma_f32_16x16x32_bf16): lane reads row (lane & 15) of a
  // 16-row block, k-chunk 4*kk + (lane >> 4) of k-step kk.
  const int fr = lane & 15, fq = lane >> 4, fs = swz(fr);
  int fragA[KS], fragB[KS];
#pragma unroll
  for (int kk = 0; kk < KS; ++kk) {
    const int pos = ((4 * kk + fq) ^ fs) * 16;
    fragA[kk] = (wm * WM + fr) * kRowBytes + pos;
    fragB[kk] = kBOff + (wn * WN + fr) * kRowBytes + pos;
  }
  // (BKN) this lane's address parts of the transposing reads: k-row 8 (lane >> 4) + (fr >> 2) of
  // a k-step's 32 (+ 4 for the second read), 8 bytes at n offset 4 (fr & 3) of 32-byte piece
  // (wn WN / 16 + j) ^ sw
  const int trB = kBOff + (8 * fq + (fr >> 2)) * kBRowBytes + (fr & 3) * 8;
  const int trSw = ((fr >> 2) | ((fq & 1) << 2)) & kSwMask;
  const int trA = (8 * fq + (fr >> 2)) * kARowBytes + (fr & 3) * 8;        // (AKM) the same for A
  const int trSwA = ((fr >> 2) | ((fq & 1) << 2)) & kSwMaskA;

  // NSTAGE-1 slabs are always in flight.  Past the last slab the copies are repeated into
  // stages nobody reads any more, so every wait below is for the same number of younger copies.
  if (nkf > 0) issue_slab(0, 0);

  // ---- accumulators start from the incoming partial (fused) or zero.
  // Block (i, j), element e of this lane: row 16*i + (lane & 15), column 16*j + 4*(lane >> 4) + e
  // of the wavefront tile.  Per 16-byte access 4 lanes cover 64 contiguous bytes of a row.
  const bool store_only = (MODE == kModeGemm) || ((p.flags & kFlagStep0StoreOnly) && tl.s == 0);
  const bool to_fwd = (MODE == kModeFused) && (p.flags & kFlagFwdDirect) && tl.c != p.own;
  // two writers (Sec. 4.1): the tile is ADDED into R with atomics, as the upstream update is
  const bool two_writers = (MODE == kModeFused) && (p.flags & kFlagTwoWriters);
  // Release by copy: the sums go to R AND into the chunk's forward slot, from the registers that
  // hold them, if this launch completes the chunk.  (A copy behind the chunk's trigger would read
  // R back: 4 M W bytes more per chunk, and it measured 30 to 60 % of the launch's time.)
  const bool to_both = (MODE == kModeFused) && !two_writers && !(p.flags & kFlagFwdDirect) &&
                       tl.c != p.own && chunk_is_whole(p, tl.s);
  const bool slot_bf16 = (MODE == kModeFused) && (p.flags & kFlagFwdBf16) && (to_fwd || to_both);
  const int rw0 = m0 + wm * WM, cw0 = n0 + wn * WN;          // wavefront tile origin (uniform)
  const bool full = (rw0 + WM <= p.M) && (cw0 + WN <= col_hi);
  // where the tile's result goes (uniform): R, C, or the chunk's forward slot
  const float *out_base;
  uint32_t ld_out;
  int col_org;            // column the base's rows start at
  if (to_fwd) {
    ld_out = (uint32_t)p.W;
    out_base = p.fwd + (int64_t)tl.s * p.M * p.W;
    col_org = col_lo;
  } else {
    ld_out = (uint32_t)((MODE == kModeGemm) ? p.ldc : p.ldr);
    out_base = p.R;
    col_org = 0;
  }
  // ---- "pairs".  Global accesses that touch half a 128-byte line per row (what one 16 x 16
  // block in the accumulator layout amounts to) run at a third of the rate of full lines, so
  // the incoming partial and the results move in units of one PAIR = two neighbouring blocks =
  // 16 rows x 32 columns = two instructions of 8 rows x 128 bytes each, and are transposed to
  // and from the accumulator layout in LDS.  A pair occupies two 1-KiB slots (rows 0-7, rows
  // 8-15); in a slot, the lane that a linear access maps to position (rp, pp) = (lane / 8,
  // lane % 8) holds row r = rp (first slot) or rp ^ 1 (second slot), 16-byte chunk pp ^ r: with
  // that swizzle both the linear side and the accumulator side are bank-conflict free.
  constexpr int UJ = FN / 2;                     // pairs per row of blocks
  struct PairLane {
    int row[2], col[2];   // row / column (in the pair) of the linear side's two instructions
    int acc[2];           // byte offset (in the pair's two slots) of the lane's 16 bytes of block 0 / 1
  };
  auto pair_lane = [](int ln) {
    PairLane u;
    const int rp = ln >> 3, pp = ln & 7;
    u.row[0] = rp;
    u.row[1] = 8 + (rp ^ 1);
    u.col[0] = 4 * (pp ^ rp);
    u.col[1] = 4 * (pp ^ rp ^ 1);
    const int m = ln & 15, q = ln >> 4, h = m >> 3, r = m & 7, rq = h ? (r ^ 1) : r;
    u.acc[0] = h * 1024 + rq * 128 + (q ^ r) * 16;
    u.acc[1] = h * 1024 + rq * 128 + ((4 + q) ^ r) * 16;
    return u;
  };
  const PairLane ul = pair_lane(lane);

  constexpr int NPAIR = NBLK / 2;
  static_assert(FN % 2 == 0, "pairs");
  // Every access to R, C or a forward slot is (uniform base) + (32-bit byte offset of the lane),
  // the offset formed per block when it is needed: byte sizes of these arrays stay below 4 GiB.
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  // The incoming partial: every pair as two full-line accesses (8 rows x 128 bytes), all in
  // flight together, landing in the pair's accumulator registers; then pair by pair through LDS
  // into the accumulator layout, so that the products accumulate on top of it.  (The scratch is
  // the last stage, which no copy touches before the main loop's first barrier.)
  if (MODE == kModeFused && !store_only && !two_writers) {
    const __amdgpu_buffer_rsrc_t in_rsrc = make_rsrc(p.R, (uint32_t)p.M * (uint32_t)p.ldr * 4u);
    uint32_t in_l[2];
#pragma unroll
    for (int h = 0; h < 2; ++h)
      in_l[h] = ((uint32_t)(rw0 + ul.row[h]) * (uint32_t)p.ldr + (uint32_t)(cw0 + ul.col[h])) * 4u;
#pragma unroll
    for (int t = 0; t < NPAIR; ++t) {
      const int i = t / UJ, jj = t % UJ;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
        if (full || (rw0 + 16 * i + ul.row[h] < p.M && cw0 + 32 * jj + ul.col[h] < col_hi))
          v = load_stream(in_rsrc, in_l[h], ((uint32_t)(16 * i) * (uint32_t)p.ldr + (uint32_t)(32 * jj)) * 4u);
        acc[i][2 * jj + h] = v;
      }
    }
    char *scr = lds + (NSTAGE - 1) * kStageBytes + wave * (kRingSlots * 1024);
#pragma unroll
    for (int t = 0; t < NPAIR; ++t) {
      const int i = t / UJ, jj = t % UJ;
      char *slot = scr + ((2 * t) & (kRingSlots - 1)) * 1024;
      *(f32x4 *)(slot + lane * 16) = acc[i][2 * jj];
      *(f32x4 *)(slot + 1024 + lane * 16) = acc[i][2 * jj + 1];
      acc[i][2 * jj] = *(const f32x4 *)(slot + ul.acc[0]);
      acc[i][2 * jj + 1] = *(const f32x4 *)(slot + ul.acc[1]);
      if (t % 2 == 1) __builtin_amdgcn_sched_barrier(0);
    }
  }
  stamp(it, 1);

  if (nkf > 0) {
#pragma unroll
    for (int st = 1; st < NSTAGE - 1; ++st) issue_slab(min(st, nkf - 1), st);
  }

  // Two sets of operand registers.  Micro-step u = (k-step kk, row pass h) reads FMH row blocks
  // of A (set u & 1) and, on the first pass of a k-step, the FN column blocks of B (set kk & 1),
  // while the products of micro-step u-1 are issued.
  bf16x8 fa[2][FMH], fb[2][FN];
  auto read_u = [&](int u, int stage_off) {
    const int kk = u / MH, h = u % MH;
#pragma unroll
    for (int i = 0; i < FMH; ++i) {
      if (AKM) {
        typedef __attribute__((ext_vector_type(4))) short s16x4;
        typedef __attribute__((address_space(3))) s16x4 *lds_s16x4_ptr;
        const char *a0 = lds + stage_off + trA + 32 * kk * kARowBytes +
                         (((wm * (WM / 16) + h * FMH + i) ^ trSwA) << 5);
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(lds_void_ptr)a0);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(lds_void_ptr)(a0 + 4 * kARowBytes));
        typedef __attribute__((ext_vector_type(8))) short s16x8;
        const s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        fa[u & 1][i] = __builtin_bit_cast(bf16x8, both);
      } else {
        fa[u & 1][i] = *(const bf16x8 *)(lds + stage_off + fragA[kk] + (h * FMH + i) * 16 * kRowBytes);
      }
    }
    if (h == 0) {
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        if (BKN) {
          typedef __attribute__((ext_vector_type(4))) short s16x4;
          typedef __attribute__((address_space(3))) s16x4 *lds_s16x4_ptr;
          const char *a0 = lds + stage_off + trB + 32 * kk * kBRowBytes + (((wn * (WN / 16) + j) ^ trSw) << 5);
          const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(lds_void_ptr)a0);
          const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(lds_void_ptr)(a0 + 4 * kBRowBytes));
          typedef __attribute__((ext_vector_type(8))) short s16x8;
          const s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
          fb[kk & 1][j] = __builtin_bit_cast(bf16x8, both);
        } else {
          fb[kk & 1][j] = *(const bf16x8 *)(lds + stage_off + fragB[kk] + j * 16 * kRowBytes);
        }
      }
    }
  };
  auto mfma_u = [&](int u) {
    const int kk = u / MH, h = u % MH;
#pragma unroll
    for (int i = 0; i < FMH; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
        acc[h * FMH + i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[kk & 1][j], fa[u & 1][i],
                                                                      acc[h * FMH + i][j], 0, 0, 0);
  };

  // ---- main loop: slab kt is multiplied while the next NSTAGE-1 slabs are in flight.  The
  // products of a slab's last micro-step are issued after the next barrier, under the next
  // slab's first LDS reads.  An iteration is: wait + barrier; k-step 0, with the next slab's
  // copies spread over its row passes; k-step 1.
  constexpr int kWaitSlab = wait_vm((NSTAGE - 2) * NL);
  if (nkf > 0) {
    // Slab 0 (and the incoming partial) landed -- and this wavefront's LDS accesses are done: the
    // transposition of the incoming partial used the last stage as scratch, and the copies issued
    // right after this barrier refill that stage.  A copy that finds its line in L1 can land
    // within a hundred clocks, before a read or write still waiting in a busy LDS queue (two
    // workgroups share the unit): the read then returns slab data, the late write ruins the slab.
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(kWaitSlab & kWaitLgkm0);
    __builtin_amdgcn_s_barrier();
    settle_pending();                              // (also older: the previous tile's stores)
    issue_slab(min(NSTAGE - 1, nkf - 1), NSTAGE - 1);
    read_u(0, 0);
#pragma unroll
    for (int u = 1; u < US; ++u) {
      read_u(u, 0);
      mfma_u(u - 1);
    }
    int stage = 1;
    for (int kt = 1; kt < nkf; ++kt) {
      const int so = stage * kStageBytes;
      const int kt_next = min(kt + NSTAGE - 1, nkf - 1);
      const int st_next = stage >= 1 ? stage - 1 : NSTAGE - 1;
      asm volatile("" ::: "memory");               // LDS reads above stay above the barrier
      __builtin_amdgcn_s_waitcnt(kWaitSlab & kWaitLgkm0);   // own copies of slab kt landed, own LDS reads done
      __builtin_amdgcn_s_barrier();                // everyone's; all are done with the stage refilled next
#pragma unroll
      for (int u = 0; u < MH; ++u) {               // k-step 0
        read_u(u, so);
        issue_copies(kt_next, st_next, u * NL / MH, (u + 1) * NL / MH);
        mfma_u((u + US - 1) % US);                 // u == 0: last micro-step of slab kt-1
      }
      sched_kstep<MH, FMH, FN, BKN ? FN : 0, AKM ? 2 * FMH : FMH>();   // (the transposing reads are two per block)
#pragma unroll
      for (int u = MH; u < US; ++u) {              // k-step 1
        read_u(u, so);
        mfma_u(u - 1);
      }
      sched_kstep<MH, FMH, FN, BKN ? FN : 0, AKM ? 2 * FMH : FMH>();   // (the transposing reads are two per block)
      stage = stage == NSTAGE - 1 ? 0 : stage + 1;
    }
    mfma_u(US - 1);
    __builtin_amdgcn_s_waitcnt(kWaitVm0);          // drain the repeated copies
  }
  asm volatile("" ::: "memory");

  if (ktail) {
    // ragged end of K: through registers, chunks past K zeroed, into stage 0
    __syncthreads();
    const int64_t kb = (int64_t)nkf * (kBK * 2);
    const uint4 zero = make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int q = 0; q < NA; ++q) {
      if (AKM) break;                              // (no ragged K in this layout)
      uint4 v = zero;
      if (chunk_of(BM / NW, q) * 8 < ktail) v = *(const uint4 *)(Ap + kb + offA[q]);
      *(uint4 *)(lds + ldsA_w + q * 1024 + lane * 16) = v;
      if (q % 2 == 1) __builtin_amdgcn_sched_barrier(0);   // two loads in flight, not all: registers
    }
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      if (BKN) break;                              // (no ragged K in this layout)
      uint4 v = zero;
      if (chunk_of(BN / NW, q) * 8 < ktail) v = *(const uint4 *)(Bp + kb + offB[q]);
      *(uint4 *)(lds + ldsB_w + q * 1024 + lane * 16) = v;
      if (q % 2 == 1) __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    // both k-steps, whatever ktail is: the zeroed chunks add nothing
#pragma unroll
    for (int u = 0; u < US; ++u) {
      read_u(u, 0);
      mfma_u(u);
    }
  }

  stamp(it, 2);
  // ---- epilogue: agent-scope (write-through) stores of whole rows of the WORKGROUP tile.  Row
  // block by row block, all wavefronts write their 16-row strips in the accumulator layout into
  // one LDS image (WAVES_M strips x 16 rows x BN columns) and read it back along the rows, so that
  // a store instruction covers 1 KiB of consecutive addresses.  What that is for: a chunk's rows start anywhere
  // (W * 4 bytes need not be a multiple of 64), and every end of a contiguous run that falls
  // inside a 64-byte granule costs the memory side a read-modify-write.  With 128-byte runs
  // (8 rows per instruction) an 8192 x 4256 x 2128 problem, W = 532, took 1.5 x the time of W = 544.
  // Two images: one barrier per row block.  Chunk k (16 bytes) of a row sits at k ^ (row & 7),
  // which keeps both sides free of bank conflicts.
  constexpr int kRowsPerWave = 16 / WAVES_N;
  constexpr int kImgBytes = WAVES_M * 16 * BN * 4;
  static_assert(2 * kImgBytes <= NSTAGE * kStageBytes, "images");
  __syncthreads();
  int lane_e = lane;                             // recomputed here rather than kept through the main loop
  asm volatile("" : "+v"(lane_e));
  const int e_row = lane_e & 15, e_q = lane_e >> 4;
  const int w_base = (wm * 16 + e_row) * (BN * 4);     // this lane's image row
  const bool whole = (m0 + BM <= p.M) && (n0 + BN <= col_hi);
  // Piece u of this wavefront's share of an image: G columns at image row ir, column col.
  auto piece = [&](int u, int G, int &ir, int &col) {
    const int L = u * 64 + lane_e, per_row = BN / G;
    ir = wave * kRowsPerWave + L / per_row;
    col = (L % per_row) * G;
  };
  auto img_chunk = [&](const char *img, int ir, int k) {   // 16-byte chunk k of image row ir
    return *(const f32x4 *)(img + ir * (BN * 4) + ((k ^ (ir & 7)) << 4));
  };
  // TO: 0 = R / C / fp32 slot (out_base), 1 = R and the fp32 slot, 2 = the bfloat16 slot,
  // 3 = R and the bfloat16 slot, 4 = atomic adds into R (two writers)
  auto store_tile = [&](auto NT, auto TO) {
    constexpr int to = decltype(TO)::value;
    const __amdgpu_buffer_rsrc_t out_rsrc = make_rsrc(out_base, (uint32_t)p.M * ld_out * 4u);
    const float *slot_base = p.fwd + (int64_t)tl.s * p.M * p.W;
    const __amdgpu_buffer_rsrc_t fwd_rsrc = make_rsrc(slot_base, (uint32_t)p.M * (uint32_t)p.W * 4u);
    const __amdgpu_buffer_rsrc_t f16_rsrc =
        make_rsrc((const uint16_t *)p.fwd + (int64_t)tl.s * p.M * p.W, (uint32_t)p.M * (uint32_t)p.W * 2u);
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      char *img = lds + (i & 1) * kImgBytes;
#pragma unroll
      for (int j = 0; j < FN; ++j)
        *(f32x4 *)(img + w_base + (((wn * (WN / 4) + 4 * j + e_q) ^ (e_row & 7)) << 4)) = acc[i][j];
      // the strips are complete (and everyone's reads of the other image, an iteration ago, done)
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      if constexpr (to == 0 || to == 1 || to == 3) {
#pragma unroll
        for (int u = 0; u < FN; ++u) {
          int ir, col;
          piece(u, 4, ir, col);
          const f32x4 v = img_chunk(img, ir, col >> 2);
          const int row = m0 + (ir >> 4) * WM + 16 * i + (ir & 15);
          if (whole || (row < p.M && n0 + col < col_hi)) {
            store_agent_hint<decltype(NT)::value>(out_rsrc, ((uint32_t)row * ld_out + (uint32_t)(n0 - col_org + col)) * 4u,
                                                  0u, v);
            if constexpr (to == 1)
              store_agent_hint<decltype(NT)::value>(fwd_rsrc, ((uint32_t)row * (uint32_t)p.W + (uint32_t)(n0 - col_lo + col)) * 4u,
                                                    0u, v);
          }
        }
      }
      if constexpr (to == 2 || to == 3) {
#pragma unroll
        for (int u = 0; u < FN / 2; ++u) {
          int ir, col;
          piece(u, 8, ir, col);
          const u32x4 v = pack_bf16(img_chunk(img, ir, col >> 2), img_chunk(img, ir, (col >> 2) + 1));
          const int row = m0 + (ir >> 4) * WM + 16 * i + (ir & 15);
          if (whole || (row < p.M && n0 + col < col_hi))
            __builtin_amdgcn_raw_buffer_store_b128(
                v, f16_rsrc, (int)(((uint32_t)row * (uint32_t)p.W + (uint32_t)(n0 - col_lo + col)) * 2u), 0, kAuxSc1);
        }
      }
      if constexpr (to == 4) {
        // op-and-store (Sec. 4.3): the other writer adds into the same words.  One word per lane
        // and instruction: an instruction covers 256 consecutive bytes.
#pragma unroll
        for (int u = 0; u < 4 * FN; ++u) {
          int ir, col;
          piece(u, 1, ir, col);
          const float v = *(const float *)(img + ir * (BN * 4) + (((col >> 2) ^ (ir & 7)) << 4) + (col & 3) * 4);
          const int row = m0 + (ir >> 4) * WM + 16 * i + (ir & 15);
          if (whole || (row < p.M && n0 + col < col_hi))
            __hip_atomic_fetch_add(const_cast<float *>(out_base) + (int64_t)row * ld_out + (n0 - col_org + col), v,
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  using std::false_type;
  using std::true_type;
  constexpr std::integral_constant<int, 0> to_one{};
  constexpr std::integral_constant<int, 1> to_r_and_slot{};
  constexpr std::integral_constant<int, 2> to_slot16{};
  constexpr std::integral_constant<int, 3> to_r_and_slot16{};
  constexpr std::integral_constant<int, 4> to_atomic{};
  if (two_writers) {
    if constexpr (MODE == kModeFused) store_tile(false_type{}, to_atomic);
  } else if (slot_bf16) {
    if (to_fwd) store_tile(false_type{}, to_slot16);
    else store_tile(false_type{}, to_r_and_slot16);
  } else if (to_both) {
    store_tile(true_type{}, to_r_and_slot);
  } else if (p.nt_out) {
    store_tile(true_type{}, to_one);
  } else {
    store_tile(false_type{}, to_one);
  }
  stamp(it, 3);
  if (nkf == 0) flush_pending();                 // (no main loop ran: nothing was settled on the way)
  if (tracked) pending = tl;
  }  // pieces of work
  flush_pending();
}

}  // namespace t3k
