// How the host side launches kernels, and the tile-kernel launchers of the other translation units.
#pragma once

#include "t3.h"
#include "t3_device.h"

namespace t3k {

extern thread_local int32_t last_hip_error;      // t3_last_hip_error() (t3_api.hip)

// Launches `kernel` and returns what THIS launch returned: an error some earlier call left in
// the runtime is not taken for ours.
template <typename... KArgs>
t3_status launch(void (*kernel)(KArgs...), dim3 grid, dim3 block, hipStream_t s, KArgs... a) {
  void *args[] = {static_cast<void *>(&a)...};
  const hipError_t e = hipLaunchKernel(reinterpret_cast<const void *>(kernel), grid, block, args, 0, s);
  if (e != hipSuccess) {
    last_hip_error = (int32_t)e;
    return T3_ERR_HIP;
  }
  return T3_OK;
}

// The tile kernel of tile ranges that cut a ring step, of two writers, and of what the others do not take, by
// mode (fused / plain GEMM) and operand layout; defined in t3_gemm_launch.hip, which is compiled
// once for each.  tm x tn: the workgroup tile.
t3_status launch_fused(const Plan &q, int32_t tm, int32_t tn, hipStream_t s);
t3_status launch_fused_kn(const Plan &q, int32_t tm, int32_t tn, hipStream_t s);
t3_status launch_fused_km(const Plan &q, int32_t tm, int32_t tn, hipStream_t s);
t3_status launch_fused_km_kn(const Plan &q, int32_t tm, int32_t tn, hipStream_t s);
t3_status launch_gemm_nk(const Plan &q, int32_t tm, int32_t tn, hipStream_t s);
t3_status launch_gemm_kn(const Plan &q, int32_t tm, int32_t tn, hipStream_t s);
t3_status launch_gemm_km(const Plan &q, int32_t tm, int32_t tn, hipStream_t s);
t3_status launch_gemm_km_kn(const Plan &q, int32_t tm, int32_t tn, hipStream_t s);

// The wide-tile kernel by mode and operand layout (t3_wide_launch.hip).  The plain GEMM's C goes through q.R, q.ldr.
t3_status launch_wide_fused(const Plan &q, int32_t tm, int32_t tn, hipStream_t s);
t3_status launch_wide_fused_kn(const Plan &q, int32_t tm, int32_t tn, hipStream_t s);
t3_status launch_wide_fused_km(const Plan &q, int32_t tm, int32_t tn, hipStream_t s);
t3_status launch_wide_fused_km_kn(const Plan &q, int32_t tm, int32_t tn, hipStream_t s);
t3_status launch_wide_overlap(const Plan &q, int32_t tm, int32_t tn, hipStream_t s);      // (tile columns overlap, fused)
t3_status launch_wide_overlap_kn(const Plan &q, int32_t tm, int32_t tn, hipStream_t s);
t3_status launch_wide_overlap_km(const Plan &q, int32_t tm, int32_t tn, hipStream_t s);
t3_status launch_wide_overlap_km_kn(const Plan &q, int32_t tm, int32_t tn, hipStream_t s);
t3_status launch_wide_gemm_nk(const Plan &q, int32_t tm, int32_t tn, hipStream_t s);
t3_status launch_wide_gemm_kn(const Plan &q, int32_t tm, int32_t tn, hipStream_t s);
t3_status launch_wide_gemm_km(const Plan &q, int32_t tm, int32_t tn, hipStream_t s);
t3_status launch_wide_gemm_km_kn(const Plan &q, int32_t tm, int32_t tn, hipStream_t s);

// The small-tile kernel (64 x 64, 32 x 64, 32 x 32), any layout (t3_small_launch.hip).
t3_status launch_small_fused(const Plan &q, int32_t tm, int32_t tn, bool b_kn, bool a_km, hipStream_t s);
t3_status launch_small_gemm(const Plan &q, int32_t tm, int32_t tn, bool b_kn, bool a_km, hipStream_t s);

}  // namespace t3k
