// attend_kernel over the bf16 cache, listed positions.
#include "attend.hpp"

namespace splash {

void launch_attend_bf16_topk(const AttendLaunch& a, int32_t workers, hipStream_t s) {
  launch_attend_heads<false, true, false, false>(a, workers, s);
}

}  // namespace splash
