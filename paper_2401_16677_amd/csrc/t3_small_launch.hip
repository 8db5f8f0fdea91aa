// Launches of the small-tile kernel for one mode (T3_LAUNCHER names the function, T3_MODE says which;
// compiled once for each).
#include "t3_small.h"
#include "t3_launch.h"

namespace t3k {
namespace {

template <int BM, int BN, int NST, bool WORDS, bool NK>
t3_status launch_small(const Plan &q, bool b_kn, bool a_km, hipStream_t s) {
  const dim3 grid((unsigned)q.total_blocks), block(256);
  if (b_kn)
    return a_km ? launch(small_tile_kernel<BM, BN, 4, NST, T3_MODE, 1, 1, WORDS>, grid, block, s, q)
                : launch(small_tile_kernel<BM, BN, 4, NST, T3_MODE, 1, 0, WORDS>, grid, block, s, q);
  if constexpr (NK)
    return a_km ? launch(small_tile_kernel<BM, BN, 4, NST, T3_MODE, 0, 1, WORDS>, grid, block, s, q)
                : launch(small_tile_kernel<BM, BN, 4, NST, T3_MODE, 0, 0, WORDS>, grid, block, s, q);
  return T3_ERR_UNSUPPORTED;
}
// (the plan by one vector request while all workgroups are on the chip at once: see small_tile_kernel)
template <int BM, int BN, int NST, bool NK = true>
t3_status launch_small(const Plan &q, bool b_kn, bool a_km, hipStream_t s) {
  const int32_t at_once = q.resident * (BM == 32 && BN == 32 ? 2 : 1);
  return q.total_blocks <= at_once ? launch_small<BM, BN, NST, true, NK>(q, b_kn, a_km, s)
                                   : launch_small<BM, BN, NST, false, NK>(q, b_kn, a_km, s);
}

}  // namespace

t3_status T3_LAUNCHER(const Plan &q, int32_t tm, int32_t tn, bool b_kn, bool a_km, hipStream_t s) {
  // 64 x 64: two 16-KiB stages per wavefront, one workgroup per compute unit; 32 x 64 (only
  // chosen with B stored K x N): three of 12 KiB; 32 x 32: two of 8 KiB, two workgroups
  if (tm == 64) return launch_small<64, 64, 2>(q, b_kn, a_km, s);
  return tn == 64 ? launch_small<32, 64, 3, false>(q, b_kn, a_km, s) : launch_small<32, 32, 2>(q, b_kn, a_km, s);
}

}  // namespace t3k
