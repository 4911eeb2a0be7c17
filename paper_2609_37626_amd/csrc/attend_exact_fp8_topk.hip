// attend_kernel over the per-token fp8 cache with the exact QK (K converted to bf16), listed positions.
#include "attend.hpp"

namespace splash {

void launch_attend_exact_fp8_topk(const AttendLaunch& a, int32_t workers, hipStream_t s) {
  launch_attend_heads<true, true, false, false>(a, workers, s);
}

}  // namespace splash
