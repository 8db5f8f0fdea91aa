// t3_choice.h and t3_div.h for the tests: what a call launches on a device of so many compute units; n / d.
#include "t3_choice.h"
#include "t3_div.h"

extern "C" void launch_shape(const t3_problem *p, int call, int tracked_m, int tracked_n, int cus, int64_t *out) {
  const t3k::LaunchShape s = t3k::launch_shape(p, static_cast<t3k::Call>(call), {tracked_m, tracked_n}, cus);
  const int64_t v[] = {s.kernel, s.tile.m, s.tile.n, s.tpc, s.begin, s.limit, s.total_blocks, s.resident, s.tail_r, s.tail_q};
  for (int i = 0; i < 10; ++i) out[i] = v[i];
}

extern "C" void start_offsets(const t3_problem *p, int call, int tracked_m, int tracked_n, int cus, double *out) {
  const t3k::Call c = static_cast<t3k::Call>(call);
  const t3k::StartOffsets o = t3k::start_offsets(p, c, t3k::launch_shape(p, c, {tracked_m, tracked_n}, cus));
  out[0] = o.groups;
  out[1] = o.window_ns;
}

extern "C" int column_align(const t3_problem *p, int call, int tile_n) {
  return t3k::column_align(p, static_cast<t3k::Call>(call), {256, tile_n}, t3k::ceil_div(p->N / p->tp, tile_n));
}

extern "C" int column_overlap(const t3_problem *p, int call, int tracked_m, int tracked_n, int cus) {
  const t3k::Call c = static_cast<t3k::Call>(call);
  const t3k::LaunchShape s = t3k::launch_shape(p, c, {tracked_m, tracked_n}, cus);
  return s.kernel == t3k::kWideTile ? t3k::column_overlap(p, c, s.tile, s.Wt) : 0;
}

extern "C" void copy_shape(int64_t M, int64_t W, int cus, int64_t *out) {
  const t3k::CopyShape s = t3k::copy_shape(M, W, cus);
  const int64_t v[] = {s.team, s.batch, s.in_flight, s.workgroups};
  for (int i = 0; i < 4; ++i) out[i] = v[i];
}

// The order of a launch's tiles if they are put in a line (0 otherwise): position -> stage, row, column.
extern "C" int tile_places(const t3_problem *p, int call, int tracked_m, int tracked_n, int cus, double now, int32_t *out) {
  const t3k::Call c = static_cast<t3k::Call>(call);
  const t3k::LaunchShape s = t3k::launch_shape(p, c, {tracked_m, tracked_n}, cus);
  const t3k::TileOrder o = t3k::tile_order(p, c, s, now);
  for (int64_t i = 0; o.rows && i < s.total_blocks; ++i) {
    const t3k::TilePlace t = t3k::tile_place(o, (uint32_t)i);
    out[3 * i] = t.stage;
    out[3 * i + 1] = t.row;
    out[3 * i + 2] = t.col;
  }
  return (int)o.width_log2 + (o.rows ? 1 : 0);
}

// The order the library takes: columns of a band, or 0 stage by stage; and of blocks (0: runs), tile rows and columns of one.
extern "C" int tile_order(const t3_problem *p, int call, int tracked_m, int tracked_n, int cus, int xcds, int32_t *blocks) {
  const t3k::Call c = static_cast<t3k::Call>(call);
  const t3k::LaunchShape s = t3k::launch_shape(p, c, {tracked_m, tracked_n}, cus);
  const t3k::XcdBlocks b = t3k::xcd_blocks(p, s, xcds);
  blocks[0] = b.by_rows;
  blocks[1] = b.rows;
  blocks[2] = b.columns;
  if (s.kernel != t3k::kWideTile) return 0;
  const t3k::TileOrder o = t3k::tile_order(p, c, s, t3k::xcd_rows(p, c, s, b));
  return o.rows ? 1 << o.width_log2 : 0;
}

extern "C" void divide(const uint32_t *n, const uint32_t *d, uint32_t *out, int count) {
  for (int i = 0; i < count; ++i) out[i] = t3k::div_by(n[i], t3k::fast_div(d[i]));
}
