// Kernels and launches of the FP32 fits; included by one translation unit per kernel function,
// so that these compile in parallel.
#pragma once

#include "fit_quad.h"
#include "fit_wave.h"

namespace ksdf {
namespace {

// queues a cell for the FP64 fit
__device__ __forceinline__ void queue_fp64(const FitArgs& A, int c) {
  const int slot = atomicAdd(A.fb_count, 1);
  A.fb_list[slot] = c;
}

// block i's four cells of a list, one wave each
template <int MB, bool MATERN>
__device__ __forceinline__ void fit_four(const FitArgs& A, const FitList& l, int i,
                                         WaveFitLds<MB>* lds) {
  const int w = threadIdx.x / 64;
  const int t = i * (FIT_THREADS / 64) + w;
  if (t >= (l.count ? *l.count : l.n)) return;
  const int c = l.cells[t];
  if (fit32_wave<MB, MATERN>(A, c, lds[w]) && (threadIdx.x & 63) == 0) queue_fp64(A, c);
}

template <int MB, bool MATERN>
__global__ void __launch_bounds__(FIT_THREADS) __attribute__((amdgpu_waves_per_eu(2)))
fit_small_kernel(FitArgs A, FitList l) {
  __shared__ WaveFitLds<MB> lds[FIT_THREADS / 64];
  fit_four<MB, MATERN>(A, l, blockIdx.x, lds);
}

// The cells of 65 to 128 samples (q), one workgroup each, and behind them those of 33 to 64
// (w), four to a workgroup: both need the registers of two waves per SIMD, and the second kind
// fills the chip while the last of the first (a chain of 250 us each) drain.
template <bool MATERN>
__global__ void __launch_bounds__(FIT_THREADS) __attribute__((amdgpu_waves_per_eu(2)))
fit_large_kernel(FitArgs A, FitList q, FitList w) {
  __shared__ union Lds {
    QuadFitLds quad;
    WaveFitLds<64> wave[FIT_THREADS / 64];
    __device__ Lds() {}
  } lds;
  if ((int)blockIdx.x >= q.n) {
    fit_four<64, MATERN>(A, w, blockIdx.x - q.n, lds.wave);
    return;
  }
  if (q.count && (int)blockIdx.x >= *q.count) return;
  const int c = q.cells[blockIdx.x];
  if (fit32_quad<MATERN>(A, c, lds.quad) && threadIdx.x == 0) queue_fp64(A, c);
}

constexpr unsigned fours(int n) { return (unsigned)((n + FIT_THREADS / 64 - 1) / (FIT_THREADS / 64)); }

template <int MB, bool MATERN>
void launch_small(const FitArgs& A, const FitList& l, hipStream_t s) {
  if (l.n > 0)
    hipLaunchKernelGGL((fit_small_kernel<MB, MATERN>), dim3(fours(l.n)), dim3(FIT_THREADS), 0, s, A, l);
}

template <bool MATERN>
void launch_large(const FitArgs& A, const FitList& q, const FitList& w, hipStream_t s) {
  const unsigned g = (unsigned)q.n + fours(w.n);
  if (g > 0) hipLaunchKernelGGL(fit_large_kernel<MATERN>, dim3(g), dim3(FIT_THREADS), 0, s, A, q, w);
}

}  // namespace
}  // namespace ksdf
