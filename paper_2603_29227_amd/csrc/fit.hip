// Per-cell log-GP fit (Sec. IV-B.1, eq. log_gp_posterior_mean; RBF of Table I).
//
// Cells with m <= 64 are fitted by one wave each (fit_wave.h: rows in registers, four
// cells per workgroup, no workgroup barriers); larger cells by one workgroup each
// (fit_quad.h: four waves, 64 x 64 blocks in registers); fit_launch.h has their kernels.
// Both write the per-cell store: (p_i, a_i), sigma_i^2, the packed factor with the
// reciprocal diagonal, the sample bounding box and A+ = sum of positive a_i.
//
// Both bound cond_2(A) by A's row sums and, where that does not decide, estimate it by
// power and inverse iteration; a cell above the threshold or with a non-positive pivot is
// queued for the FP64 kernel (the plain FP64 path uses that kernel for every cell).
#include <algorithm>

#include "fit_dev.h"

namespace ksdf {
namespace {

// dA/dl of the FP32-fitted cells, packed as the factor (adjoint_var_f models), from the stored
// coordinates: dA_ik/dl = A_ik r_ik^2 / l^3 (RBF) or c^2 r_ik^2 exp(-c r_ik) / l (Matern 3/2).
// Its own kernel, one thread an entry: inside the fit its rows were 4-byte stores 64 rows
// apart, and their branches split the adjoint's sum and spilled its terms.  43 us for the
// room's 5516 cells of 64 samples.  first: the launch's first cell of the list.
__global__ void __launch_bounds__(FIT_THREADS) fit_dA_kernel(FitArgs A, FitList l, int first) {
  const int t = first + (int)blockIdx.x;
  if (l.count && t >= *l.count) return;
  const int c = l.cells[t];
  const int b = A.offsets[c], m = A.offsets[c + 1] - b;
  __shared__ float4 xh[MAXM], xl[MAXM];
  for (int i = threadIdx.x; i < m; i += FIT_THREADS) {
    xh[i] = reinterpret_cast<const float4*>(A.ps32)[b + i];
    xl[i] = reinterpret_cast<const float4*>(A.plo32)[b + i];
  }
  __syncthreads();
  const ff inv2l2{A.inv2l2_ff[0], A.inv2l2_ff[1]};
  float* D = A.D32 + A.loff[c];
  for (int e = threadIdx.x; e < m * (m + 1) / 2; e += FIT_THREADS) {
    int i = (int)((sqrtf(8.f * (float)e + 1.f) - 1.f) * 0.5f);
    while (i * (i + 1) / 2 > e) --i;
    while ((i + 1) * (i + 2) / 2 <= e) ++i;
    const int k = e - i * (i + 1) / 2;
    const float4 h = xh[i], l = xl[i], g = xh[k], f = xl[k];
    const ff r2 = ff_norm2_lean(ff_sub_lean(h.x, l.x, g.x, f.x), ff_sub_lean(h.y, l.y, g.y, f.y),
                                ff_sub_lean(h.z, l.z, g.z, f.z));
    float d;
    if (A.kernel == KSDF_KERNEL_MATERN32)
      d = A.mc2_ff[0] * r2.hi * expf(-A.mc_ff[0] * sqrtf(r2.hi)) * A.inv_l_ff[0];
    else
      d = ff_exp_neg_lean(ff_mul(r2, inv2l2)).hi * r2.hi * A.inv_l3_ff[0];
    D[e] = i == k ? 0.f : d;
  }
}

// The FP32 fits of the cells of up to 16, 32, 64 and 128 samples, and their packed dA/dl where
// the model keeps it.  le4, le8: where the first list is known to the host, how many at its
// start have up to 4 and up to 8 samples.  Those get launches of their own (a fit in a matrix of
// 16 rows does the work of 16 samples: 5456 cells of one sample, Matern 3/2 with adjoint, took
// 37 us with loops that ended at the samples and 78 us so) where they are too many for the next
// launch to take them along: fewer would cost more for the launch than they save.
constexpr int SMALL_CELLS_MIN = 1024;
void launch_fit32(const FitArgs& A, const FitList (&l)[4], int le4, int le8, hipStream_t s) {
  const bool matern = A.kernel == KSDF_KERNEL_MATERN32;
  const auto large = matern ? launch_fit_large_matern : launch_fit_large_rbf;
  const auto small = matern ? launch_fit_small_matern : launch_fit_small_rbf;
  large(A, l[3], l[2], s);
  small(A, 32, l[1], s);
  const int n = l[0].n;
  // [0, a) in matrices of 4 rows, [a, b) of 8, the rest of 16
  const int a = le4 >= SMALL_CELLS_MIN || le4 == n ? le4 : 0;
  const int b = le8 - a >= SMALL_CELLS_MIN || le8 == n ? le8 : a;
  small(A, 16, FitList{l[0].cells + b, l[0].count, n - b}, s);
  small(A, 8, FitList{l[0].cells + a, nullptr, b - a}, s);
  small(A, 4, FitList{l[0].cells, nullptr, a}, s);
  if (!A.adjoint || !A.D32) return;
  constexpr int MOST = 1 << 23;   // a launch holds fewer than 2^32 threads
  for (const FitList& k : l)
    for (int first = 0; first < k.n; first += MOST)
      hipLaunchKernelGGL(fit_dA_kernel, dim3((unsigned)std::min(k.n - first, MOST)), dim3(FIT_THREADS), 0, s,
                         A, k, first);
}

__global__ void set_int_kernel(int* p, int v) { *p = v; }

// ---- streaming refit (Sec. IV-C, App. G) ----

// Training-queue score of App. G, s = c2 (1 + eta c0), in FP32 with every rounding
// explicit (no contraction), so that a host computation in the same order agrees.
__device__ __forceinline__ float refit_score(const float* dirty, const float* qcount, float eta,
                                             int c) {
  return __fmul_rn(dirty[c], __fadd_rn(1.f, __fmul_rn(eta, qcount[c])));
}

// The dirty cells (c2 > 0) and their scores, appended in any order (wave-aggregated
// slots); n_dirty counts them.  The ranking below does not depend on the order.
__global__ void __launch_bounds__(256) refit_compact_kernel(const float* dirty, const float* qcount,
                                                            float eta, int n, int* dlist,
                                                            float* dscore, int* n_dirty) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  const bool mine = i < n && dirty[i] > 0.f;
  const unsigned long long live = __ballot(mine);
  if (!live) return;
  const int lane = threadIdx.x & 63;
  const int leader = __ffsll((long long)live) - 1;
  int base = 0;
  if (lane == leader) base = atomicAdd(n_dirty, __popcll(live));
  base = __shfl(base, leader, 64);
  if (mine) {
    const int slot = base + __popcll(live & ((1ull << lane) - 1ull));
    dlist[slot] = i;
    dscore[slot] = refit_score(dirty, qcount, eta, i);
  }
}

// Rank of every dirty cell by descending score, ties to the lower id, by comparison
// with the other dirty cells through LDS tiles (work grows with the square of the
// dirty count, not of the cell count); the first `budget` ranks name the cells to
// refit.  Launched with one thread per cell: blocks past the dirty count exit.
__global__ void __launch_bounds__(256) refit_rank_kernel(const int* dlist, const float* dscore,
                                                         const int* n_dirty, int budget, int* sel) {
  __shared__ float ts[256];
  __shared__ int tid_[256];
  const int d = *n_dirty;
  if ((int)blockIdx.x * 256 >= d) return;   // uniform over the block
  const int t = blockIdx.x * 256 + threadIdx.x;
  const bool mine = t < d;
  const float si = mine ? dscore[t] : 0.f;
  const int ci = mine ? dlist[t] : 0;
  int rank = 0;
  for (int base = 0; base < d; base += 256) {
    __syncthreads();
    const int j = base + threadIdx.x;
    ts[threadIdx.x] = j < d ? dscore[j] : 0.f;
    tid_[threadIdx.x] = j < d ? dlist[j] : 0;
    __syncthreads();
    const int lim = min(256, d - base);
    for (int k = 0; k < lim; ++k) {
      const float sj = ts[k];
      rank += (sj > si || (sj == si && tid_[k] < ci)) ? 1 : 0;
    }
  }
  if (mine && rank < budget) sel[rank] = ci;
}

// n_sel = min(budget, n_dirty); clears the per-bucket counts
__global__ void refit_count_kernel(const int* n_dirty, int budget, int* n_sel, int* bcount) {
  if (threadIdx.x == 0) *n_sel = min(budget, *n_dirty);
  if (threadIdx.x < 4) bcount[threadIdx.x] = 0;
}

// the selected cells into per-m-bucket lists (the bucket sizing of the full fit)
__global__ void __launch_bounds__(256) refit_bucket_kernel(const int* sel, const int* n_sel,
                                                           const int* offsets, int minb, int budget,
                                                           int* blist, int* bcount) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= *n_sel) return;
  const int c = sel[i];
  const int mc = offsets[c + 1] - offsets[c];
  int bk = mc <= 16 ? 0 : mc <= 32 ? 1 : mc <= 64 ? 2 : 3;
  if (minb >= 32 && bk < 1) bk = 1;
  if (minb >= 64 && bk < 2) bk = 2;
  const int pos = atomicAdd(&bcount[bk], 1);
  blist[(long)bk * budget + pos] = c;
}

// after the refit: c2 = 0 and c0 halved for the refitted cells (App. G)
__global__ void __launch_bounds__(256) refit_reset_kernel(const int* sel, const int* n_sel,
                                                          float* dirty, float* qcount) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= *n_sel) return;
  const int c = sel[i];
  dirty[c] = 0.f;
  qcount[c] = 0.5f * qcount[c];
}

// Query counters of App. G in two steps, so that the result does not depend on the
// order of the atomics: an integer histogram of the argmin cells (one atomic per
// distinct cell of a wave; queries that arrive spatially ordered mostly share their
// argmin cell within a wave), then one addition per cell, c0 = min(c0 + count, cap),
// rounded once.  (Halving on refit leaves c0 fractional, so float atomics adding
// counts to it directly would round differently in different orders.)  Argmins
// outside [0, n_cells) are not counted.
__global__ void __launch_bounds__(256) zero_kernel(unsigned* h, int n) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c < n) h[c] = 0u;
}

__global__ void __launch_bounds__(256) count_queries_kernel(const int* argmin, long Q, int n_cells,
                                                            unsigned* hist) {
  const long q = (long)blockIdx.x * 256 + threadIdx.x;
  int c = q < Q ? argmin[q] : -1;
  if (c >= n_cells) c = -1;
  const int lane = threadIdx.x & 63;
  unsigned long long todo = __ballot(c >= 0);
  while (todo) {
    const int leader = __ffsll((long long)todo) - 1;
    const int key = __shfl(c, leader, 64);
    const unsigned long long same = __ballot(c == key) & todo;
    if (lane == leader) atomicAdd(hist + key, (unsigned)__popcll(same));
    todo &= ~same;
  }
}

// The same counts through a histogram in LDS when the cells fit there: each block
// counts one contiguous range of the queries (neighbouring queries mostly share their
// argmin cell) and adds its non-zero bins to the global histogram, so the global
// atomics fall from one per run of equal argmins to one per (block, cell).
constexpr int CQ_T = 1024;
constexpr int CQ_LDS_CELLS = 16384;
__global__ void __launch_bounds__(CQ_T) count_queries_lds_kernel(const int* argmin, long Q,
                                                                int n_cells, unsigned* hist) {
  __shared__ unsigned h[CQ_LDS_CELLS];
  for (int c = threadIdx.x; c < n_cells; c += CQ_T) h[c] = 0u;
  __syncthreads();
  const long per = (Q + gridDim.x - 1) / gridDim.x;
  const long q0 = (long)blockIdx.x * per;
  const long q1 = q0 + per < Q ? q0 + per : Q;
  for (long q = q0 + threadIdx.x; q < q1; q += CQ_T) {
    const int c = argmin[q];
    if (c >= 0 && c < n_cells) atomicAdd(h + c, 1u);
  }
  __syncthreads();
  for (int c = threadIdx.x; c < n_cells; c += CQ_T)
    if (h[c]) atomicAdd(hist + c, h[c]);
}

__global__ void __launch_bounds__(256) count_apply_kernel(const unsigned* hist, float* qcount, int n,
                                                          float cap) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c < n) qcount[c] = fminf(qcount[c] + (float)hist[c], cap);
}

// Dense L^{-1} of each cell (64 x 64, column-major, zero beyond m) from the packed
// factor rows with reciprocal diagonal: lane j solves L x = e_j by forward
// substitution, x_i = -(sum_{k<i} L_ik x_k) / L_ii (x_k = 0 for k < j), x_j = 1 / L_jj,
// with its column in registers and the factor rows read once per wave (uniform
// loads); each lane stores its column as 16-byte pieces (no LDS, so that occupancy
// is set by the registers alone).
__global__ void __launch_bounds__(64) linv_kernel(const int* offsets, const long* loff,
                                                  const float* L, float* Linv) {
  const int c = blockIdx.x, j = threadIdx.x;
  const int m = offsets[c + 1] - offsets[c];
  const float* Lc = L + loff[c];
  float x[64];
#pragma unroll
  for (int i = 0; i < 64; ++i) {
    float xi = 0.f;
    if (i < m) {
      const float* row = Lc + i * (i + 1) / 2;
      float a0 = 0.f, a1 = 0.f, a2 = 0.f, a3 = 0.f;
#pragma unroll
      for (int k = 0; k + 3 < i; k += 4) {
        a0 = fmaf(row[k], x[k], a0);
        a1 = fmaf(row[k + 1], x[k + 1], a1);
        a2 = fmaf(row[k + 2], x[k + 2], a2);
        a3 = fmaf(row[k + 3], x[k + 3], a3);
      }
#pragma unroll
      for (int k = i & ~3; k < i; ++k) a0 = fmaf(row[k], x[k], a0);
      const float r = row[i];
      xi = j == i ? r : (j < i ? -((a0 + a1) + (a2 + a3)) * r : 0.f);
    }
    x[i] = xi;
  }
  float4* out = reinterpret_cast<float4*>(Linv + (long)c * 4096 + (long)j * 64);
#pragma unroll
  for (int i = 0; i < 16; ++i) out[i] = make_float4(x[4 * i], x[4 * i + 1], x[4 * i + 2], x[4 * i + 3]);
}

}  // namespace

void launch_linv(const ksdf_model* m, hipStream_t s) {
  m->linv_ok = false;
  if (!m->Linv32 || !m->tuning.query_mfma || m->n_cells == 0) return;
  hipLaunchKernelGGL(linv_kernel, dim3((unsigned)m->n_cells), dim3(64), 0, s, m->offsets, m->loff,
                     m->L32, m->Linv32);
  m->linv_ok = true;
}

size_t refit_workspace_bytes(const ksdf_model* m, int budget) {
  const long b = std::min(budget, m->n_cells);
  // bucket lists, bucket counts + n_dirty, then the dirty cells' ids and scores
  return 4 * b * sizeof(int) + 8 * sizeof(int) + 2 * (long)m->n_cells * sizeof(int);
}

int launch_refit(ksdf_model* m, const void* pts, int dtype, const void* svar, float* dirty,
                 float* qcount, double eta, int budget, int* sel, int* n_sel, uint8_t* user_status,
                 void* ws, hipStream_t s) {
  if (m->n_cells == 0) {
    hipLaunchKernelGGL(set_int_kernel, dim3(1), dim3(1), 0, s, n_sel, 0);
    KSDF_HIP_TRY(hipGetLastError());
    return KSDF_OK;
  }
  budget = std::min(budget, m->n_cells);
  int* blist = static_cast<int*>(ws);
  int* bcount = blist + 4L * budget;
  int* n_dirty = bcount + 4;
  int* dlist = bcount + 8;
  float* dscore = reinterpret_cast<float*>(dlist + m->n_cells);
  const unsigned gc = (unsigned)((m->n_cells + 255) / 256);
  const unsigned gb = (unsigned)((budget + 255) / 256);
  hipLaunchKernelGGL(set_int_kernel, dim3(1), dim3(1), 0, s, n_dirty, 0);
  hipLaunchKernelGGL(refit_compact_kernel, dim3(gc), dim3(256), 0, s, dirty, qcount, (float)eta,
                     m->n_cells, dlist, dscore, n_dirty);
  hipLaunchKernelGGL(refit_rank_kernel, dim3(gc), dim3(256), 0, s, dlist, dscore, n_dirty, budget, sel);
  hipLaunchKernelGGL(refit_count_kernel, dim3(1), dim3(64), 0, s, n_dirty, budget, n_sel, bcount);
  FitArgs A = make_fit_args(m, pts, dtype, svar, user_status);
  timer_mark(m, KSDF_TIMER_FIT, 0, s);
  if (m->precision == KSDF_FP64) {
    A.list = sel;
    A.list_count = n_sel;
    A.emit32 = 0;
    launch_fit64(m, A, budget, s);
  } else {
    const int minb = m->tuning.fit_min_bucket;
    hipLaunchKernelGGL(refit_bucket_kernel, dim3(gb), dim3(256), 0, s, sel, n_sel, m->offsets, minb,
                       budget, blist, bcount);
    hipLaunchKernelGGL(set_int_kernel, dim3(1), dim3(1), 0, s, m->fb_count, 0);
    // grid per bucket: at most the budget and at most the cells of that bucket
    const int* bs = m->bucket_start;
    const int lo32 = minb >= 32 ? bs[0] : bs[1];
    const int lo64 = minb >= 64 ? bs[0] : bs[2];
    const int n[4] = {minb < 32 ? bs[1] - bs[0] : 0, minb < 64 ? bs[2] - lo32 : 0, bs[3] - lo64,
                      bs[4] - bs[3]};
    FitList l[4];
    for (int bk = 0; bk < 4; ++bk)
      l[bk] = FitList{blist + (long)bk * budget, bcount + bk, std::min(n[bk], budget)};
    launch_fit32(A, l, 0, 0, s);
    A.list = m->fb_list;
    A.list_count = m->fb_count;
    A.emit32 = 1;
    launch_fit64(m, A, std::min(budget, 1024), s);
  }
  if (m->precision != KSDF_FP64) launch_linv(m, s);
  timer_mark(m, KSDF_TIMER_FIT, 1, s);
  hipLaunchKernelGGL(refit_reset_kernel, dim3(gb), dim3(256), 0, s, sel, n_sel, dirty, qcount);
  KSDF_HIP_TRY(hipGetLastError());
  return KSDF_OK;
}

size_t count_queries_workspace_bytes(const ksdf_model* m) {
  return (size_t)std::max(m->n_cells, 1) * sizeof(unsigned);
}

int launch_count_queries(const ksdf_model* m, const int* argmin, long Q, float* qcount, float cap,
                         void* ws, hipStream_t s) {
  const int n = m->n_cells;
  if (n == 0) return KSDF_OK;
  unsigned* hist = static_cast<unsigned*>(ws);
  const unsigned gc = (unsigned)((n + 255) / 256);
  hipLaunchKernelGGL(zero_kernel, dim3(gc), dim3(256), 0, s, hist, n);
  if (Q > 0 && n <= CQ_LDS_CELLS) {
    const long blocks = std::min<long>(1024, (Q + CQ_T - 1) / CQ_T);
    hipLaunchKernelGGL(count_queries_lds_kernel, dim3((unsigned)blocks), dim3(CQ_T), 0, s, argmin, Q,
                       n, hist);
  } else if (Q > 0) {
    hipLaunchKernelGGL(count_queries_kernel, dim3((unsigned)((Q + 255) / 256)), dim3(256), 0, s,
                       argmin, Q, n, hist);
  }
  hipLaunchKernelGGL(count_apply_kernel, dim3(gc), dim3(256), 0, s, hist, qcount, n, cap);
  KSDF_HIP_TRY(hipGetLastError());
  return KSDF_OK;
}

int launch_fit(ksdf_model* m, const void* pts, int dtype, const void* svar, uint8_t* user_status,
               hipStream_t s) {
  FitArgs A = make_fit_args(m, pts, dtype, svar, user_status);
  if (m->n_cells == 0) return KSDF_OK;
  if (m->precision == KSDF_FP64) {
    A.emit32 = 0;
    timer_mark(m, KSDF_TIMER_FIT, 0, s);
    launch_fit64_all(m, A, s);
    timer_mark(m, KSDF_TIMER_FIT, 1, s);
  } else {
    hipLaunchKernelGGL(set_int_kernel, dim3(1), dim3(1), 0, s, m->fb_count, 0);
    timer_mark(m, KSDF_TIMER_FIT, 0, s);
    // m buckets: cells below the tuned smallest bucket merge into it
    const int* lists = m->bucket_cells;
    const int* bs = m->bucket_start;
    const int minb = m->tuning.fit_min_bucket;
    const int lo32 = minb >= 32 ? bs[0] : bs[1];
    const int lo64 = minb >= 64 ? bs[0] : bs[2];
    const FitList l[4] = {{lists + bs[0], nullptr, minb < 32 ? bs[1] - bs[0] : 0},
                          {lists + lo32, nullptr, minb < 64 ? bs[2] - lo32 : 0},
                          {lists + lo64, nullptr, bs[3] - lo64},
                          {lists + bs[3], nullptr, bs[4] - bs[3]}};
    const bool own = minb < 32;
    launch_fit32(A, l, own ? m->bucket_small[0] : 0, own ? m->bucket_small[1] : 0, s);
    A.list = m->fb_list;
    A.list_count = m->fb_count;
    A.emit32 = 1;
    launch_fit64(m, A, std::min(m->n_cells, 1024), s);
    launch_linv(m, s);
    timer_mark(m, KSDF_TIMER_FIT, 1, s);
  }
  KSDF_HIP_TRY(hipGetLastError());
  return KSDF_OK;
}

}  // namespace ksdf
