// Launches of the FP32 fits, Matern 3/2 kernel.
#include "fit_launch.h"

namespace ksdf {

void launch_fit_small_matern(const FitArgs& A, int mb, const FitList& l, hipStream_t s) {
  if (mb == 4) launch_small<4, true>(A, l, s);
  else if (mb == 8) launch_small<8, true>(A, l, s);
  else if (mb == 16) launch_small<16, true>(A, l, s);
  else launch_small<32, true>(A, l, s);
}
void launch_fit_large_matern(const FitArgs& A, const FitList& q, const FitList& w, hipStream_t s) {
  launch_large<true>(A, q, w, s);
}

}  // namespace ksdf
