// Which kernel serves a launch, on which workgroup tile, and how the tiles fall to the workgroups.  Plain
// C++ without HIP: the library's host side and the tests share it.
#pragma once

#include <stdint.h>

#include "t3.h"
#include "t3_div.h"

namespace t3k {

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

struct TileShape {
  int32_t m, n;
};

enum Call { kCallFused, kCallGemm, kCallReduce, kCallOther };
enum Kernel { kGeneralTile, kWideTile, kSmallTile, kReduction };   // t3_gemm.h, t3_wide.h, t3_small.h, t3_aux.h

constexpr int kNumXcd = 8;            // the XCD grouping of decode_tile is written for 8 XCDs
constexpr int kTailMinSlabs = 8;      // K-slabs of 64 a tile needs before a balanced tail splits it
constexpr int kTailSlots = 256;       // tiles a balanced tail can split (flag words behind the tracker state)
constexpr int kReduceThreads = 256;   // threads of a reduction workgroup
constexpr int kReduceBatch = 4;       // 16-byte pieces of each operand such a thread has in flight

struct Choice {
  Kernel kernel;
  TileShape tile;
};

// For `steps` whole ring steps of a problem: the tile with the least time by rounds of workgroups x
// time of a tile.  The times are fitted to problems of 8 to 16384 tokens, K 128 to 10240, all layouts,
// TP 2 to 32, run on every tile.  On 60 such problems (profiles/workgroup_tiles.txt) what is picked takes 1.013 of
// the best tile's time on average and within 2 % on 51 of them; the worst, 2048 x 10240 x 512 with A transposed,
// 59 us where the best takes 48.  The times carry what the problems had in common (traffic past the L2s, clocks); release
// mode, incoming partial and the plain GEMM's shorter way out are not told apart.
// wide_ok: the wide-tile kernel may be used (sizes, see wide_fits).  Where it may not, or K has fewer slabs than
// its LDS stages, gemm_tile_kernel takes its place on the shapes it has: the same main loop rate (12288 x 4096 x 6144,
// B stored K x N: 493 us, 495 wide), but the incoming partial is waited for at the start of every tile
// (12288 x 4096 x 1536: 19 us per tile outside the main loop, 14 wide).
inline Choice workgroup_tile(const t3_problem *p, int cus, int64_t steps, bool wide_ok) {
  struct Cand {
    TileShape t;
    int stages, per_cu;          // LDS stages of the wide-tile kernel (0: small-tile kernel); workgroups per compute unit
    double slab_us, ends_us;     // a K-slab of 64 / the rest of a tile
  };
  static const Cand kCand[] = {{{256, 256}, 2, 1, 1.22, 14.3}, {{256, 192}, 2, 1, 0.90, 13.3},
                               {{256, 128}, 3, 1, 0.75, 10.9}, {{128, 192}, 3, 1, 0.59, 8.2},
                               {{128, 128}, 2, 2, 0.81, 7.4},  {{64, 64}, 0, 1, 0.166, 6.55},
                               {{32, 64}, 0, 1, 0.113, 6.9},   {{32, 32}, 0, 2, 0.115, 5.3}};
  const bool km = p->a_layout == T3_A_KM, kn = p->b_layout == T3_B_KN;
  const int64_t W = p->N / p->tp;
  const int64_t slabs = ceil_div(p->K, 64);
  double best = -1.0;
  Choice pick{kSmallTile, kCand[5].t};
  for (const Cand &c : kCand) {
    const bool general = c.stages && (!wide_ok || slabs < c.stages);
    if (general && c.t.n == 192) continue;
    // (32 x 64 is for k-rows of B of a whole 128-byte line; with B K-contiguous two 32 x 32 workgroups take its place
    // at the same time per slab, and start and end sooner)
    if (c.t.m == 32 && c.t.n == 64 && !kn) continue;
    const int64_t T = ceil_div(p->M, c.t.m) * ceil_div(W, c.t.n) * steps, slots = (int64_t)cus * c.per_cu;
    double rounds = (double)ceil_div(T, slots);
    const bool tail = c.stages && !general && c.per_cu == 1 && T > slots && T % slots && 2 * (T % slots) <= slots &&
                      p->K / 64 >= kTailMinSlabs && !(p->flags & T3_FLAG_FWD_BF16);
    if (tail) rounds -= 0.5;
    // (a compute unit with one tile instead of two has it done in 0.8 of the time)
    const double alone = c.per_cu == 2 && T <= cus ? 0.8 : 1.0;
    // (k-rows of a transposed operand are half a 128-byte line long in a 32 wide tile)
    const double slab_us = c.slab_us * (km && c.t.m == 32 ? 1.34 : 1.0) * (kn && c.t.n == 32 ? 1.34 : 1.0);
    const double us = rounds * alone * ((general ? 1.4 : 1.0) * c.ends_us + slab_us * (double)slabs);
    if (best < 0 || us < best * 0.999) {
      best = us;
      pick = {!c.stages ? kSmallTile : (general ? kGeneralTile : kWideTile), c.t};
    }
  }
  return pick;
}

// Workgroup tile of the reduction over whole ring steps: columns of a chunk in equal parts of at most
// 256 (1 KiB runs), cut at whole 128-byte lines; rows so that a workgroup of 256 lanes has one batch of
// four 16-byte pieces per lane, or half and a quarter of one where that leaves compute units idle.  (Two, four
// and eight batches per workgroup, GEMM and reduction of 2343 x 17664 x 384: 191, 200 and 197 us, one 188;
// of 2048 x 4096 x 512: 42, 47 and 47, one 40.)
inline TileShape reduce_tile_shape(const t3_problem *p, int cus, int64_t steps) {
  const int64_t W = p->N / p->tp, parts = ceil_div(W, 256);
  const int64_t tn = ceil_div(ceil_div(W, parts), 32) * 32, width = tn < W ? tn : W;
  int64_t tm = 1;
  for (int64_t batch = kReduceBatch; batch >= kReduceBatch / 4; batch /= 2) {
    tm = batch * kReduceThreads * 4 / width;
    if (ceil_div(p->M, tm) * ceil_div(W, tn) * steps >= 2 * cus) break;
  }
  return {(int32_t)tm, (int32_t)tn};
}

// How the all-gather step copies a chunk: `team` lanes of a workgroup of 256 per row, `batch` 16-byte pieces
// per lane at a time, in_flight of them at once.  In us, chunk of rows x columns,
// N of eight chunks:
//  - Two rows per compute unit or fewer: a workgroup per row (500 x 1536 by wavefronts 2.9, by workgroups 2.8; 24 x 4100 3.8, 2.5).
//  - Otherwise a wavefront per row while that is a batch of four or eight; a workgroup for longer rows, whose pieces
//    would follow each other through a loop (2048 x 4100: 17.0 by wavefronts, 15.3), and for rows of 256 pieces (if they
//    are many) and 512, which leave it no idle lane (8192 x 1024 13.8 by wavefronts, 13.0, 8192 x 2048 26.4 and 24.3); part of a wavefront for rows that do not fill it (16384 x 12: 4.2, 2.8).
//  - Fewer loads in flight than a batch where the chunk is on the compute units at once, eight workgroups of four rows
//    each at most, and they are well filled: all loads together, then all stores together, is slower there than a mixture of
//    both (all, two and one in flight: 4096 x 1536 11.4, 10.4, 10.4 to 11.3; 4096 x 1152 8.5, 8.0, 8.4; 8192 x 1536 21.9, 22.2, 20.2;
//    8192 x 640 10.1, 9.6, 8.6; with fewer workgroups, 2900 x 1536, 7.0, 7.3, 8.9; 4096 x 640 5.1, 5.3, 5.7).
//  - Beyond that a workgroup per row, one piece at a time (by wavefronts and that way: 12000 x 512 12.1 and 11.2, 16384 x 1152
//    31.4 and 29.3, 16384 x 2048 49.6 and 46.8; 16384 x 1536 43.4 both).
struct CopyShape {
  int32_t team, batch, in_flight;
  int64_t workgroups;
};
inline CopyShape copy_shape(int64_t M, int64_t W, int cus) {
  const int64_t pieces = W / 4, fours = ceil_div(M, 4);          // (workgroups of a wavefront per row)
  const int32_t batch = pieces <= 256 ? 4 : 8;
  CopyShape s{64, batch, batch, 0};
  if (M <= 2 * (int64_t)cus || pieces > 512)
    s = pieces <= 256 ? CopyShape{256, 1, 1, 0} : CopyShape{256, 8, 8, 0};
  else if (pieces <= 4)
    s = {4, 4, 4, 0};
  else if (pieces <= 16 && fours > 4 * (int64_t)cus)
    s = {16, 4, 4, 0};
  else if (pieces == 512 || (pieces == 256 && fours >= 5 * (int64_t)cus) || (pieces > 96 && fours > 8 * (int64_t)cus))
    s = {256, 1, 1, 0};
  else if (pieces > 64 && fours <= 8 * (int64_t)cus)
    s.in_flight = batch == 8 ? (fours < 4 * (int64_t)cus ? 8 : (fours < 6 * (int64_t)cus ? 2 : 1)) : (fours < 5 * (int64_t)cus ? 4 : 1);
  s.workgroups = ceil_div(M, 256 / s.team);
  return s;
}

// The wide-tile kernel's offsets count from where a tile starts, and what lies outside is marked by their top
// bit: the rows of a tile (256 at most) have to fit 2 GiB, of a transposed operand the whole array.  (65536 x 12288
// x 1536, R of 3 GiB: 2518 us here, 2744 by gemm_tile_kernel.)
inline bool wide_fits(const t3_problem *p, int64_t ld_out) {
  const int64_t kMost = 1ll << 31, rows = 256;
  return (p->a_layout == T3_A_KM ? p->K : rows) * p->lda * 2 <= kMost &&
         (p->b_layout == T3_B_KN ? p->K : rows) * p->ldb * 2 <= kMost && rows * ld_out * 4 <= kMost;
}

// Where a launch of the wide-tile kernel lets a chunk's tile columns start so that R's (the plain GEMM's C's) rows are cut at
// 64-byte granules: chunk c starts (c W) mod 16 columns into a granule, and its tiles but the first start as many columns
// early.  15, or 0: they start at multiples of the tile.  Only where that costs no further tile (the last tile has the columns
// to spare) and where something is written there for more than one chunk (with the direct release only the
// own chunk's sums are).  A granule written in two parts costs the memory side a
// read-modify-write each.  8192 x 4256 x 2128, chunks of 532 columns, sums to R and slots: 228 us at multiples of the
// tile, 218 at granules (chunks of 544 columns, where all edges are, 194).
// By sizes alone, whether rows and buffer start at granules or not: which tile, and so which workgroup, has a column decides
// the order its products are added in, and where a buffer lies shall not change results.  Buffers off granules pay
// for it: over 20 problems 0.3 to 0.7 %, at most 3 (8192 x 4256 x 200 by copy, 137 us at multiples of the tile, 142).
inline int32_t column_align(const t3_problem *p, Call call, TileShape tile, int64_t Wt) {
  const int64_t W = p->N / p->tp;
  const bool written = call == kCallGemm || (call == kCallFused && !(p->flags & T3_FLAG_FWD_DIRECT));
  if (!written || Wt < 2 || W % 16 == 0 || W % 4) return 0;
  const int64_t most = 16 - (W & -W);            // (W is a multiple of 4, of 8 with k-rows of B: so are all c W mod 16)
  return Wt * tile.n - W >= most ? 15 : 0;
}

// With the direct release: by how many columns neighbouring tile columns of a chunk overlap, or 0.  A slot's rows are W elements apart, so where W is
// no whole number of 64-byte granules, rows start at another place in one each, and no column is a granule's end in all of them.
// Where the grid has the columns to spare, both neighbours compute the columns around the cut, and every row is cut
// between them where its own granule ends; each element is still written once.  (What is left are the ends of the rows
// themselves.)  By sizes alone, as column_align, and whatever R's leading dimension.  In us, cut at multiples of the tile and this way: 4293 x 1612 x
// 208 on 4 chunks 70.0, 63.5; 8192 x 532 x 512 on 8 96.8, 91.2 (x 544, whole granules, 74.5); 6000 x 700 x 800 on 8 112.0, 106.8 (x 704 92.0);
// 16384 x 396 x 256 on 8 121.0, 115.7; 1071 x 1460 x 640 on 8 41.1, 39.2; 2048 x 404 x 640 on 16 43.3, 41.3; long K hides it, 8192 x 532 x 2128 on 8
// 189.5, 188.6.  Over 160 drawn problems 4.6 % less below K of 512, 2.9 below 1024, 1.0 below 2048, 0.5 beyond, with bfloat16 slots (10125 x 696 x 168
// on 8 99.5, 92.2; 620 x 2056 x 2352 on 8 67.1, 67.0) and transposed operands (1387 x 1288 x 192 on 2 13.9, 12.6; 3735 x 2472 x 640 on 4 109.7, 97.2)
// as with fp32 and K-contiguous ones; at worst 1756 x 1796 x 2520 on 8 168.9, 174.4, and 0.2 us on short launches of one round.  Not with the release by copy, where R and the slot would want different cuts of the same sums.
inline int32_t column_overlap(const t3_problem *p, Call call, TileShape tile, int64_t Wt) {
  const int64_t W = p->N / p->tp, granule = p->flags & T3_FLAG_FWD_BF16 ? 32 : 16;
  if (call != kCallFused || !(p->flags & T3_FLAG_FWD_DIRECT) || Wt < 2 || W % granule == 0) return 0;
  const int64_t most = granule - (W & -W);       // (rows start at multiples of W's power of two)
  return Wt * tile.n - W >= most * (Wt - 1) ? (int32_t)most : 0;
}

// What a call over a tile range launches.  `tracked`: the problem's tile, which the range is counted in.
struct LaunchShape {
  Kernel kernel;
  TileShape tile;                // the workgroup tile
  int64_t tracked_tpc;           // tracked tiles of a chunk
  int64_t Mt, Wt, tpc;           // workgroup tiles: rows, columns, tiles of a chunk
  int64_t begin, limit;          // the range in workgroup tiles
  int64_t stage0, total_blocks;  // the ring steps it touches: the first, grid positions from there
  int64_t resident;              // workgroups of this tile the device holds at once
  int64_t tail_r, tail_q;        // balanced tail: tiles split, full rounds before them (0: none)
};
inline LaunchShape launch_shape(const t3_problem *p, Call call, TileShape tracked, int cus) {
  LaunchShape s{};
  const bool two_writers = (call == kCallFused || call == kCallOther) && (p->flags & T3_FLAG_TWO_WRITERS);
  const int64_t W = p->N / p->tp;
  s.tracked_tpc = ceil_div(p->M, tracked.m) * ceil_div(W, tracked.n);
  const int64_t T = s.tracked_tpc * p->tp;
  s.limit = (p->tile_limit < 0 || p->tile_limit > T) ? T : p->tile_limit;
  s.begin = p->tile_begin < 0 ? 0 : (p->tile_begin > s.limit ? s.limit : p->tile_begin);
  s.kernel = call == kCallReduce ? kReduction : kGeneralTile;
  s.tile = tracked;
  // Over whole ring steps nothing but the counters' final values depends on the tracked tile, so a
  // chunk is cut as suits the chip; a range that cuts a step is in units of tracked tiles, and so are the
  // two-writer calls' counts.
  if (T && !two_writers && call != kCallOther && s.begin % s.tracked_tpc == 0 && s.limit % s.tracked_tpc == 0) {
    const int64_t steps = (s.limit - s.begin) / s.tracked_tpc;
    if (call == kCallReduce) {
      s.tile = reduce_tile_shape(p, cus, steps);
    } else {
      const Choice c = workgroup_tile(p, cus, steps, wide_fits(p, call == kCallGemm ? p->ldc : p->ldr));
      s.kernel = c.kernel;
      s.tile = c.tile;
    }
  }
  s.Mt = ceil_div(p->M, s.tile.m);
  s.Wt = ceil_div(W, s.tile.n);
  s.tpc = s.Mt * s.Wt;
  // (where workgroup tiles are not the tracked ones the range is whole steps)
  if (s.tpc != s.tracked_tpc && s.tracked_tpc) {
    s.limit = s.limit / s.tracked_tpc * s.tpc;
    s.begin = s.begin / s.tracked_tpc * s.tpc;
  }
  s.stage0 = s.tpc > 0 ? s.begin / s.tpc : 0;
  s.total_blocks = s.tpc > 0 && s.begin < s.limit ? (ceil_div(s.limit, s.tpc) - s.stage0) * s.tpc : 0;
  // one workgroup per compute unit, two of the smallest of the large tiles
  s.resident = (int64_t)cus * (s.tile.m == 128 && s.tile.n == 128 ? 2 : 1);
  // Balanced tail (see the kernels' work_item): launches of the wide-tile kernel whose last round of
  // grid positions would fill at most half the chip; every half needs a few K-slabs, and the partial sums pass
  // through the fp32 destination (so not with bfloat16 forward slots), each element with one writer at a time.
  const bool slot_bf16 = call == kCallFused && (p->flags & T3_FLAG_FWD_BF16);
  if (s.kernel == kWideTile && s.resident == cus && !slot_bf16 && s.total_blocks > s.resident && p->K / 64 >= kTailMinSlabs) {
    const int64_t r = s.total_blocks % s.resident;
    if (r > 0 && 2 * r <= s.resident && r <= kTailSlots) {
      s.tail_r = r;
      s.tail_q = s.total_blocks / s.resident;
    }
  }
  return s;
}

// XCD grouping: a stage's Mt x Wt tiles in 8 equal blocks, one per XCD, or, where they do
// not split or that is better, in 8 runs down the tile columns (see decode_tile).  What counts is
// how many A rows and B columns an XCD's L2 pulls; the A rows are the same ones in every stage, so
// if they stay in that L2 (half of its 4 MiB) they count once for all stages.  That is for small
// tiles, which are in flight for several stages at a time: with large ones the slabs of B push A
// out.  (A device with another number of XCDs takes the runs: order inside a stage is free.)
struct XcdBlocks {
  int32_t by_rows, rows, columns;      // blocks a tile column is cut into (0: runs), tiles of a block
};
inline XcdBlocks xcd_blocks(const t3_problem *p, const LaunchShape &s, int xcds) {
  XcdBlocks b{0, 0, 0};
  if (s.tpc <= 0) return b;
  const int64_t steps = ceil_div(s.limit, s.tpc) - s.begin / s.tpc;
  auto footprint = [&](double rows, double cols) {
    const bool stays = s.tile.m < 128 && rows * (double)p->K * 2.0 <= 2.0 * (1 << 20);
    return (stays && steps > 1 ? rows / (double)steps : rows) + cols;
  };
  double best = -1.0;
  if (s.tile.m < 128) {
    const double run = (double)ceil_div(s.tpc, kNumXcd);
    best = run >= (double)s.Mt ? footprint((double)p->M, (run / (double)s.Mt + 0.5) * s.tile.n) : footprint(run * s.tile.m, 1.5 * s.tile.n);
  }
  for (int nbm = 1; nbm <= kNumXcd && xcds == kNumXcd; nbm *= 2) {
    const int nbn = kNumXcd / nbm;
    if (s.Mt % nbm || s.Wt % nbn) continue;
    const double foot = footprint((double)(s.Mt / nbm) * s.tile.m, (double)(s.Wt / nbn) * s.tile.n);
    if (best < 0 || foot < best) {
      best = foot;
      b = {nbm, (int32_t)(s.Mt / nbm), (int32_t)(s.Wt / nbn)};
    }
  }
  return b;
}

// Tiles an XCD works on in step: an eighth of a round, or half of that with a balanced tail, whose two halves of the workgroups are
// half a tile apart.
inline int64_t xcd_run(const LaunchShape &s) {
  const int64_t round = s.total_blocks < s.resident ? s.total_blocks : s.resident, run = s.tail_r ? round / 16 : round / 8;
  return run < 1 ? 1 : run;
}
// The rows of A and of B it pulls for them stage by stage.  An XCD's A rows are the same ones in every stage of blocks; the plain GEMM,
// which pulls and stores little else, keeps them in its L2 of 4 MiB where they fit.  With a balanced tail, whose two halves of the
// workgroups would each pull their own in a line, they are counted once for the launch: stage by stage and in a line, 2048 x 20480 x K on 8 chunks,
// blocks of 2 x 5, K of 1536 134.7, 138.7; 3072 218.9, 225.7; 4096 273.6, 275.3; 10240, where they do not fit, 694, 681 (fused 144.6, 142.7;
// 235.1, 231.7; 283.9, 287.1; 708, 694); 3920 x 13248 x 560 on 8 93.7, 103.3; 4096 x 10752 x 1168 on 4 135.0, 144.1; over 20 shapes 1.2 %,
// with the reduction 0.8.  (Without a tail the line is 2.5 % ahead over 20 shapes, 0.4 behind with the reduction.)
constexpr int64_t kXcdCacheBytes = 4ll << 20;
inline double xcd_rows(const t3_problem *p, Call call, const LaunchShape &s, const XcdBlocks &blocks) {
  const double stages = 8.0 * (double)xcd_run(s) / (double)s.tpc;
  double rows = (double)blocks.rows, columns = (double)blocks.columns;
  if (!blocks.by_rows) {
    const double run = (double)s.tpc / 8.0, all = (double)s.Mt;
    rows = run < all ? (run < 1.0 ? 1.0 : run) : all;
    columns = run / all + 0.5 > 1.0 ? run / all + 0.5 : 1.0;
  } else if (call == kCallGemm && s.tail_r && (int64_t)blocks.rows * s.tile.m * p->K * 2 <= kXcdCacheBytes) {
    rows *= (double)s.resident / (double)s.total_blocks;
  }
  return rows * s.tile.m + columns * (stages > 1.0 ? stages : 1.0) * s.tile.n;
}

// The order in which the persistent workgroups of the wide-tile kernel take the tiles of whole ring steps.  Workgroups are
// dealt round-robin to the 8 XCDs, so of a round of grid positions every eighth runs on the same one and pulls its slabs
// through the same L2.  Cutting every stage into 8 blocks (or runs down its columns) of its own is good where a round is about a stage;
// where it is several, the stages' blocks lie on top of one another: 2048 x 20480 x 10240 on 8 chunks, 8 x 10 tiles a stage,
// gives an XCD 2 rows and 16 columns at a time, 18 slabs to pull for 32 tiles, where 8 rows and 4 columns are 12.
// So, here, the tiles are put in a line, an XCD takes a run of it in every round, and the line is laid so that a run is a compact
// block: tile columns, counted through the stages, are taken `width` (a power of two) at a time, and such a band
// is walked row by row, every other one from the bottom up, so that a run that goes on in the next band keeps its rows.
// A round's tiles run at the same time whatever their order, so a band may hold columns of several stages as long as it is
// no larger than a round; a larger one has to lie inside a stage.
struct TileOrder {
  uint32_t round, total, rows, bands, width_log2;    // positions of a round, of the launch; tile rows (0: not in a line); whole bands
  FastDiv by_round, by_band, by_last, by_stage;      // by `round`; rows << width_log2; columns behind the bands; Wt
};
struct TilePlace {
  int stage, row, col;                               // stage counted from the range's first
};
T3_HOST_DEVICE inline TilePlace tile_place(const TileOrder &o, uint32_t position) {
  const uint32_t r = div_by(position, o.by_round), base = r * o.round, j = position - base, x = j & 7;
  const uint32_t left = o.total - base, n = left < o.round ? left : o.round, odd = n & 7;
  const uint32_t t = base + (n >> 3) * x + (odd < x ? odd : x) + (j >> 3);
  const uint32_t band = div_by(t, o.by_band), in = t - ((band * o.rows) << o.width_log2);
  const bool last = band == o.bands;
  uint32_t row = last ? div_by(in, o.by_last) : in >> o.width_log2;
  const uint32_t col = (band << o.width_log2) + in - (last ? row * o.by_last.d : row << o.width_log2);
  if (band & 1) row = o.rows - 1 - row;
  const uint32_t stage = div_by(col, o.by_stage);
  return {(int)stage, (int)row, (int)(col - stage * o.by_stage.d)};
}
// now: xcd_rows of the blocks or runs stage by stage.  In us, stage by stage and in a line: 8689 x 840 x 1120 on 4 chunks, bfloat16 slots
// 131.0, 113.1; 11434 x 820 x 7200 on 2, GEMM and reduction 353.5, 328.0; 700 x 128 x 392 on 16 11.8, 11.0; 2048 x 18432 x 576 on
// 32 74.4, 71.2; 2048 x 20480 x 10240 on 8 663, 648; 2048 x 22528 x 4096 on 8 348, 325; 2506 x 944 x 2064 on 2 45.4, 44.5.  Over 660 drawn launches
// 4.8 % less; 18 are more than 2 % slower, the worst 1472 x 9968 x 6136 on 2 with the reduction, 200, 216.  Not taken
//  - where it needs 85 % of the rows or more: the A rows of a stage's blocks are the same ones in every stage, and an
//    XCD's L2 partly keeps them (4096 x 12288 x 1536 on 8, 12 bands either way: 160.8, 167.3);
//  - with fewer than four K-slabs, where there is little to pull (534 x 1048 x 128 on 2: 9.8, 9.9);
//  - with the release by copy of chunks whose rows start in the middle of a 128-byte line: the tiles either side of the line would
//    write it at the same time (2131 x 464 x 640 on 16 71.9, 77.4; x 432 68.6, 75.5; x 448, whole lines, 69.3, 68.1).
inline TileOrder tile_order(const t3_problem *p, Call call, const LaunchShape &s, double now) {
  TileOrder o{};
  if (s.total_blocks <= 0 || p->K < 256) return o;
  if (call == kCallFused && !(p->flags & T3_FLAG_FWD_DIRECT) && (p->N / p->tp) % 32) return o;
  const int64_t columns = s.total_blocks / s.Mt, round = s.total_blocks < s.resident ? s.total_blocks : s.resident;
  const int64_t run = xcd_run(s);
  double best = -1.0, best_foot = 0.0;
  auto foot = [&](int64_t tiles, int64_t width) {    // rows of A and of B of a run of so many tiles
    const int64_t in_rows = ceil_div(tiles, width), rows = in_rows < s.Mt ? in_rows : s.Mt;
    return (double)(rows * s.tile.m + ceil_div(in_rows, s.Mt) * width * s.tile.n);
  };
  for (uint32_t log2 = 0; log2 <= 3; ++log2) {       // (runs are of 64 tiles at most: no wider band needs fewer rows)
    const int64_t width = 1ll << log2;
    if (log2 && (width > columns || (s.Mt * width > round && s.Wt % width))) continue;
    // (of equal ones the one whose halves are small too: workgroups drift)
    const double cost = foot(run, width) + 0.25 * foot(ceil_div(run, 2), width);
    if (best < 0 || cost < best) {
      best = cost;
      best_foot = foot(run, width);
      o.width_log2 = log2;
    }
  }
  if (best_foot > 0.85 * now) return TileOrder{};
  o.round = (uint32_t)round;
  o.total = (uint32_t)s.total_blocks;
  o.rows = (uint32_t)s.Mt;
  o.bands = (uint32_t)(columns >> o.width_log2);
  const uint32_t rest = (uint32_t)columns & ((1u << o.width_log2) - 1);
  o.by_round = fast_div(o.round);
  o.by_band = fast_div(o.rows << o.width_log2);
  o.by_last = fast_div(rest ? rest : 1);
  o.by_stage = fast_div((uint32_t)s.Wt);
  return o;
}

// Start-up offsets: the first wave of persistent workgroups starts in `groups` phase groups over window_ns (see
// stagger_start; 0: all at once), from two rounds of tiles on.  The last group ends 3/4 of the window late; what is won is a
// part of every round's way out.  So the window is half an estimated tile time, at most 12 us, and on the large tiles, their
// columns and rows whole, what was measured to be better.  In us with half a tile time, 4 groups over 4 us, over 12 us,
// 8 over 16 us (rounds in brackets):
//   fused, 256 x 256   4096 x 12288 x 256     98.2  96.1  93.5  94.1  (3)    16384 x 8192 x 512, copy     331 336 314 301  (8)
//                      8192 x 4096 x 192, copy 82.3 82.4  86.5  80.6  (2)    8192 x 4096 x 448           74.3  -  70.5  -  (2)
//                      16384 x 4096 x 128, copy 155.6 153.9 163.1 -  (4)    eleven such with K of 128   1   .981 .987  -
//   fused, 256 x 192   4096 x 9216 x 256      74.6  72.2  74.0  75.2  (3)    8192 x 18432 x 1152         403 399 400 390  (12)
//                      14748 x 2304 x 1152   114.1 110.8 116.9 115.0  (2.7; over 6 us 110.7)
//                      4460 x 18432 x 1024   234.6 226.4 235.3 241.4  (6.8: not whole rounds)
//   rows off 64-byte granules, copy   12288 x 3072 x 640, ldr 3076    149 147 160 149  (3; ldr 3072   115 114 111 108)
//                                     4096 x 24576 x 512, ldr 24580   313  -  300  -   (6)
//   plain GEMM         8192 x 4576 x 200      50.5  49.9  64.8  63.5  (3)    16384 x 9216 x 384          167 167 153 161  (12)
//                      7144 x 6144 x 512      69.2  69.2  73.0  79.4  (3.5)  16384 x 6144 x 256           94  92  85  91  (6)
//                      4096 x 20480 x 192     73.7   -    75.7   -    (5)    16384 x 8192 x 192          121   -  108   -  (8)
// K of 4096 and more: none, four groups and eight differ by less than 1 % on eleven shapes of whole rounds; 9819 x 4608 x 4096
// (3.7), copy: none 356, over 12 us 372.
struct StartOffsets {
  int32_t groups;
  double window_ns;
};
// Matrix rate of one compute unit: 4096 flop/clock at a sustained ~1.5 GHz under load, in flop per nanosecond.
constexpr double kCuFlopPerNs = 6.25e3;
inline StartOffsets start_offsets(const t3_problem *p, Call call, const LaunchShape &s) {
  if (s.tile.m < 128 || s.total_blocks < 2 * s.resident) return {0, 0.0};
  const int64_t rounds = s.total_blocks / s.resident, slabs = p->K / 64, W = p->N / p->tp;
  const double half_tile = (double)s.tile.m * s.tile.n * (double)p->K / kCuFlopPerNs;
  const StartOffsets plain{4, half_tile < 12000.0 ? half_tile : 12000.0}, wide{4, 12000.0};
  const bool fused = call != kCallGemm, direct = p->flags & T3_FLAG_FWD_DIRECT;
  // (columns past the chunk's end, an eighth of a tile or more, have no way out)
  if (s.kernel != kWideTile || s.tile.m < 256 || s.tile.n < 192 || 8 * W < 7 * s.Wt * s.tile.n) return plain;
  if (slabs >= 64) return {0, 0.0};
  if ((fused ? p->ldr : p->ldc) % 16 && rounds < (fused && direct ? 3 : 6)) return plain;
  if (rounds >= 6 && slabs >= 12 && (s.total_blocks % s.resident == 0 || s.tail_r)) return {8, 16000.0};
  if (!fused) return rounds >= (slabs >= 8 ? 4 : (slabs >= 4 ? 5 : 8)) ? wide : plain;
  if (s.tile.n == 256) return slabs >= 8 || (rounds >= 3 && slabs >= 3) || direct ? wide : StartOffsets{4, 4000.0};
  if (slabs >= 8) return rounds >= 3 ? wide : StartOffsets{4, 6000.0};
  return rounds >= 6 && slabs >= 4 ? wide : StartOffsets{4, 4000.0};
}

}  // namespace t3k
