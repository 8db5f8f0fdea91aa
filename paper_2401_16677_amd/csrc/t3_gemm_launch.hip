// Launches of the tile kernel for one mode and operand layout.  Compiled once for each of the
// eight (T3_LAUNCHER names the function, T3_MODE, T3_BKN and T3_AKM say what it launches): the
// instantiations are most of the library's compile time, and they compile side by side.
#include "t3_gemm.h"
#include "t3_launch.h"

namespace t3k {
namespace {

template <int MODE, int BKN, int AKM>
t3_status launch_gemm_layout(const Plan &q, int32_t tm, int32_t tn, hipStream_t s) {
  // Persistent workgroups: as many as the chip holds at once, each walking the grid positions.  (work_item strides by
  // q.resident: a smaller grid would leave positions out)
  const int64_t positions = (int64_t)q.total_blocks * (MODE == kModeFused ? q.split_k : 1);
  const dim3 grid((unsigned)(positions > q.resident ? q.resident : positions));
  // K-slabs of 64 everywhere.  256 x 256: 8 wavefronts of 128 x 64, two 64-KiB stages; 256 x 128 and
  // 128 x 256: 8 wavefronts of 64 x 64, three 48-KiB stages; one workgroup per compute unit.
  // 128 x 128: 4 wavefronts of 64 x 64, two 32-KiB stages, two workgroups.
  if (tm == 256 && tn == 256)
    return launch(gemm_tile_kernel<256, 256, 2, 4, 2, MODE, BKN, AKM>, grid, dim3(512), s, q);
  if (tm == 256 && tn == 128)
    return launch(gemm_tile_kernel<256, 128, 4, 2, 3, MODE, BKN, AKM>, grid, dim3(512), s, q);
  if (tm == 128 && tn == 256)
    return launch(gemm_tile_kernel<128, 256, 2, 4, 3, MODE, BKN, AKM>, grid, dim3(512), s, q);
  return launch(gemm_tile_kernel<128, 128, 2, 2, 2, MODE, BKN, AKM>, grid, dim3(256), s, q);
}

}  // namespace

t3_status T3_LAUNCHER(const Plan &q, int32_t tm, int32_t tn, hipStream_t s) {
  return launch_gemm_layout<T3_MODE, T3_BKN, T3_AKM>(q, tm, tn, s);
}

}  // namespace t3k
