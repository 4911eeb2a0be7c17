// attend_kernel over the per-token fp8 cache, QK on the fp8 pipe.
#include "attend.hpp"

namespace splash {

void launch_attend_fp8(const AttendLaunch& a, int32_t workers, hipStream_t s) {
  launch_attend_heads<true, false, false, true>(a, workers, s);
}

}  // namespace splash
