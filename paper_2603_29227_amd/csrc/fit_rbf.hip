// Launches of the FP32 fits, RBF kernel.
#include "fit_launch.h"

namespace ksdf {

void launch_fit_small_rbf(const FitArgs& A, int mb, const FitList& l, hipStream_t s) {
  if (mb == 4) launch_small<4, false>(A, l, s);
  else if (mb == 8) launch_small<8, false>(A, l, s);
  else if (mb == 16) launch_small<16, false>(A, l, s);
  else launch_small<32, false>(A, l, s);
}
void launch_fit_large_rbf(const FitArgs& A, const FitList& q, const FitList& w, hipStream_t s) {
  launch_large<false>(A, q, w, s);
}

}  // namespace ksdf
