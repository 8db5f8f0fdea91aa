// The launch plan of a call, made without a GPU: t3_api.hip as it is, on a device of 256 compute units and 8 XCDs that answers from here.
#include <hip/hip_runtime.h>
#include <string.h>

namespace {
hipError_t this_device(int *device) {
  *device = 0;
  return hipSuccess;
}
hipError_t attribute_of(int *value, hipDeviceAttribute_t attribute, int) {
  *value = attribute == hipDeviceAttributeMultiprocessorCount ? 256 : 8;
  return hipSuccess;
}
}  // namespace
#define hipGetDevice this_device
#define hipDeviceGetAttribute attribute_of

#include "t3_api.hip"

extern "C" int plan_bytes() { return (int)sizeof(t3k::Plan); }

// The plan of a fused call (0), a plain GEMM (1) or a reduction (2), every byte of it `before` until it is made.  (Nothing is read
// through the pointers.)
extern "C" int make(const t3_problem *p, int call, int before, void *plan) {
  static const t3k::Call calls[] = {t3k::kCallFused, t3k::kCallGemm, t3k::kCallReduce};
  static const int needs[] = {kNeedAB | kNeedR | kNeedFwd | kNeedTrack, kNeedAB | kNeedC, kNeedC | kNeedR | kNeedFwd | kNeedTrack};
  float *at = (float *)4096;
  int32_t tm, tn;
  bool empty;
  memset(plan, before, sizeof(t3k::Plan));
  return make_plan(p, calls[call], needs[call], at, at, call ? at : nullptr, at, at, call == 1 ? nullptr : (uint32_t *)at,
                   static_cast<t3k::Plan *>(plan), &tm, &tn, &empty);
}
