// The tracker's chain (t3_device.h) played on the host: the tiles of a launch land one by one.
#include "t3_device.h"

using namespace t3k;

namespace {
struct Counting {
  int64_t *zeros, *round_trips;        // additions of nothing; answers waited for
  uint32_t add(uint32_t *w, uint32_t v) const {
    *zeros += v == 0u;
    ++*round_trips;
    const uint32_t old = *w;
    *w += v;
    return old;
  }
  void add_both(uint32_t *w0, uint32_t &v0, uint32_t *w1, uint32_t &v1) const {
    v0 = add(w0, v0);
    v1 = add(w1, v1);
    --*round_trips;
  }
  void put(uint32_t *w, uint32_t v) const { *w = v; }
  void wait() const {}
  void clear_bank(uint32_t *b, int P) const {
    for (int i = 0; i < 3 * P + 2; ++i) b[i] = i >= 2 * P && i < 3 * P ? kEmpty : 0u;
  }
};
}  // namespace

// tiles: stage, row, column of each in the order they land (`updates` of them).  words: tracker state, in and out.  seen: zeros,
// round trips.
extern "C" void play(int P, int rank, int Mt, int Wt, int whole, int sub_groups, int sub_shift, int stage0, int upd_first,
                     int upd_rest, int expected_done, int tracked, const int32_t *tiles, int updates, uint32_t *words,
                     int64_t *seen) {
  Plan p{};
  p.P = P;
  p.rank = rank;
  p.own = (rank + P - 1) % P;
  p.Mt = Mt;
  p.Wt = Wt;
  p.tpc = Mt * Wt;
  p.tracked = tracked;
  p.whole_chunks = whole;
  p.sub_groups = sub_groups;
  p.sub_shift = sub_shift;
  p.stage0 = stage0;
  p.upd_first = upd_first;
  p.upd_rest = upd_rest;
  p.expected_done = expected_done;
  p.track = words;
  const int bank = 3 * P + 2;
  p.tail_flags = words + 2 * bank + 2;
  Trk t;
  t.gen = words + 2 * bank;
  t.error = t.gen + 1;
  uint32_t *b = words + (*t.gen & 1u) * bank;
  t.counter = b;
  t.ready = b + P;
  t.queue = b + 2 * P;
  t.queue_len = b + 3 * P;
  t.done = b + 3 * P + 1;
  t.other = words + ((*t.gen & 1u) ^ 1u) * bank;
  const Counting who{&seen[0], &seen[1]};
  for (int i = 0; i < updates; ++i) {
    Tile tl{tiles[3 * i], (rank + tiles[3 * i]) % P, tiles[3 * i + 1], tiles[3 * i + 2]};
    TrkCount k{who.add(track_word(p, t, tl), 1u), 0u};
    if (!whole) k.done = who.add(t.done, 1u);
    track_finish(p, t, tl, k, whole != 0, who);
  }
}
