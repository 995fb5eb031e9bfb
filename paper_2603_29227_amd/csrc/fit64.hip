// FP64 fits: launches of fit64_cell (fit64_dev.h), one workgroup per cell.
#include "fit64_dev.h"

namespace ksdf {
namespace {

// MB: the largest m of the launch, which sizes the factor in LDS
template <int MB>
__global__ void __launch_bounds__(FIT64_THREADS) fit64_kernel(FitArgs A, int n) {
  __shared__ double smem[fit64_smem_doubles(MB)];
  const int count = A.list_count ? *A.list_count : n;
  for (int t = blockIdx.x; t < count; t += gridDim.x) fit64_cell<MB>(A, A.list[t], smem);
}

}  // namespace

void launch_fit64(const ksdf_model* m, const FitArgs& A, int grid, hipStream_t s) {
  if (grid <= 0) return;
  if (m->max_m <= 64)
    hipLaunchKernelGGL(fit64_kernel<64>, dim3((unsigned)grid), dim3(FIT64_THREADS), 0, s, A, 0);
  else
    hipLaunchKernelGGL(fit64_kernel<128>, dim3((unsigned)grid), dim3(FIT64_THREADS), 0, s, A, 0);
}

// The cells of more than 64 samples first (the longest), then the rest with a quarter of the
// LDS and so more cells per CU.
void launch_fit64_all(const ksdf_model* m, FitArgs A, hipStream_t s) {
  const int small = m->bucket_start[3], large = m->bucket_start[4] - small;
  A.list_count = nullptr;
  A.list = m->bucket_cells + small;
  if (large > 0)
    hipLaunchKernelGGL(fit64_kernel<128>, dim3((unsigned)large), dim3(FIT64_THREADS), 0, s, A, large);
  A.list = m->bucket_cells;
  if (small > 0)
    hipLaunchKernelGGL(fit64_kernel<64>, dim3((unsigned)small), dim3(FIT64_THREADS), 0, s, A, small);
}

}  // namespace ksdf
