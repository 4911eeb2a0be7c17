// attend_kernel over the per-token fp8 cache, QK on the fp8 pipe, listed positions.
#include "attend.hpp"

namespace splash {

void launch_attend_fp8_topk(const AttendLaunch& a, int32_t workers, hipStream_t s) {
  launch_attend_heads<true, true, false, true>(a, workers, s);
}

}  // namespace splash
