// Launches of the tile kernel for one mode and operand layout.  Compiled once for each of the
// eight (T3_LAUNCHER names the function, T3_MODE, T3_BKN and T3_AKM say what it launches): the
// instantiations are most of the library's compile time, and they compile side by side.
#include "t3_gemm.h"
#include "t3_launch.h"

namespace t3k {
namespace {

// The hand-ordered kernel (four wavefronts, operands K-contiguous).
template <int BM, int BN, int NSTAGE, int MODE, int TAIL>
t3_status launch_hand_ordered(const Plan &q, dim3 grid, hipStream_t s) {
  if constexpr (MODE == kModeFused && TAIL != 2) {
    if constexpr (TAIL == 0)
      if (q.flags & kFlagFwdBf16)
        return launch(gemm_tile_kernel<BM, BN, 2, 2, NSTAGE, MODE, 0, 0, TAIL, 2, 1>, grid, dim3(256), s, q);
    if (!(q.flags & kFlagFwdDirect) && q.P > 1)
      return launch(gemm_tile_kernel<BM, BN, 2, 2, NSTAGE, MODE, 0, 0, TAIL, 1, 1>, grid, dim3(256), s, q);
  }
  return launch(gemm_tile_kernel<BM, BN, 2, 2, NSTAGE, MODE, 0, 0, TAIL, 0, 1>, grid, dim3(256), s, q);
}
// With a balanced tail: the kernels' TAIL variants.  The plain GEMM's is cut from the fused kernel.
template <int BM, int BN, int NSTAGE, int MODE>
t3_status launch_hand_ordered_tile(const Plan &q, dim3 grid, hipStream_t s) {
  if (!q.tail_r) return launch_hand_ordered<BM, BN, NSTAGE, MODE, 0>(q, grid, s);
  if constexpr (MODE == kModeFused) {
    return launch_hand_ordered<BM, BN, NSTAGE, MODE, 1>(q, grid, s);
  } else {
    Plan g = q;
    g.flags = 0;
    g.ldr = q.ldc;                      // (R already is the output pointer)
    return launch_hand_ordered<BM, BN, NSTAGE, kModeFused, 2>(g, grid, s);
  }
}

template <int MODE, int BKN, int AKM>
t3_status launch_gemm_layout(const Plan &q, int32_t tm, int32_t tn, hipStream_t s) {
  // Persistent workgroups: as many as the chip holds at once, each walking the grid positions.
  const int64_t positions = (int64_t)q.total_blocks * (MODE == kModeFused ? q.split_k : 1);
  const dim3 grid((unsigned)(positions > q.resident ? q.resident : positions));
  if constexpr (!BKN && !AKM) {
    if (q.hand) {
      if (tm == 256)
        return tn == 256 ? launch_hand_ordered_tile<256, 256, 2, MODE>(q, grid, s)
               : tn == 192 ? launch_hand_ordered_tile<256, 192, 2, MODE>(q, grid, s)
                           : launch_hand_ordered_tile<256, 128, 3, MODE>(q, grid, s);
      return tn == 192 ? launch_hand_ordered_tile<128, 192, 3, MODE>(q, grid, s)
                       : launch_hand_ordered_tile<128, 128, 2, MODE>(q, grid, s);
    }
  }
  // The compiler-scheduled kernels: the other layouts, two writers, and tile ranges that cut a ring
  // step.  K-slabs of 64 everywhere.  256 x 256: 8 wavefronts of 128 x 64,
  // two 64-KiB stages; 256 x 128 and 128 x 256: 8 wavefronts of 64 x 64, three 48-KiB stages; one
  // workgroup per compute unit.  128 x 128: 4 wavefronts of 64 x 64, two 32-KiB stages, two workgroups.
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
