// attend_kernel over the fp8 caches with the exact QK (K converted to bf16).
#include "attend.hpp"

namespace splash {

void launch_attend_exact_qk(const AttendLaunch& a, int32_t workers, hipStream_t s) {
  const bool topk = a.topk_idx != nullptr;
  if (a.kv_dtype == 2) {
    if (topk) launch_attend_heads<true, true, true, false>(a, workers, s);
    else launch_attend_heads<true, false, true, false>(a, workers, s);
  } else {
    if (topk) launch_attend_heads<true, true, false, false>(a, workers, s);
    else launch_attend_heads<true, false, false, false>(a, workers, s);
  }
}

}  // namespace splash
