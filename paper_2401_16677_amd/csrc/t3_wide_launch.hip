// Launches of the wide-tile kernel for one mode and operand layout (T3_LAUNCHER names the function, T3_MODE,
// T3_BKN, T3_AKM and T3_OVERLAP say which; compiled once for each).
#include "t3_wide.h"
#include "t3_launch.h"

namespace t3k {

// FM, FN, LDS stages, images; row blocks of the incoming partial requested during the last slabs, and at
// most in registers at a time (what the register file leaves)
#define T3_WIDE(...) launch(wide_tile_kernel<__VA_ARGS__, T3_MODE, T3_BKN, T3_AKM, T3_OVERLAP>, grid, dim3(256), s, q)

t3_status T3_LAUNCHER(const Plan &q, int32_t tm, int32_t tn, hipStream_t s) {
  // persistent workgroups: as many as the chip holds at once (work_item strides by q.resident: a smaller grid would leave
  // positions out, and with a balanced tail the halves of its tiles)
  const dim3 grid((unsigned)(q.total_blocks > q.resident ? q.resident : q.total_blocks));
  if (tm == 256 && tn == 256) return T3_WIDE(8, 8, 2, 1, 1, 2);
  if (tm == 256 && tn == 192) return T3_WIDE(8, 6, 2, 2, 2, 5);
  if (tm == 256) return T3_WIDE(8, 4, 3, 1, 4, 8);
  if (tn == 192) return T3_WIDE(4, 6, 3, 1, 4, 4);
  return T3_WIDE(4, 4, 2, 1, 2, 4);
}

}  // namespace t3k
