// attend_kernel over the fp8 latent-row cache, QK on the fp8 pipe.
#include "attend.hpp"

namespace splash {

void launch_attend_latent(const AttendLaunch& a, int32_t workers, hipStream_t s) {
  launch_attend_heads<true, false, true, true>(a, workers, s);
}

}  // namespace splash
