// attend_kernel over the per-token fp8 cache with the exact QK (K converted to bf16).
#include "attend.hpp"

namespace splash {

void launch_attend_exact_fp8(const AttendLaunch& a, int32_t workers, hipStream_t s) {
  launch_attend_heads<true, false, false, false>(a, workers, s);
}

}  // namespace splash
