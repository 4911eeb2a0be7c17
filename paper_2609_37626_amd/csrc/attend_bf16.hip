// attend_kernel over the bf16 cache.
#include "attend.hpp"

namespace splash {

void launch_attend_bf16(const AttendLaunch& a, int32_t workers, hipStream_t s) {
  launch_attend_heads<false, false, false, false>(a, workers, s);
}

}  // namespace splash
