// attend_kernel over the fp8 latent-row cache with the exact QK (K converted to bf16).
#include "attend.hpp"

namespace splash {

void launch_attend_exact_latent(const AttendLaunch& a, int32_t workers, hipStream_t s) {
  launch_attend_heads<true, false, true, false>(a, workers, s);
}

}  // namespace splash
