// FP64 fit of one cell with a whole workgroup: every cell of an FP64 model, and the cells of
// an FP32 model whose condition estimate (or a failed pivot) asks for FP64.
//
// The factor lives in LDS (66 KB at m = 128): with it in global memory every pivot waited on
// a round trip through the caches, three barriers apart.  A column step has two barriers
// (column scaled, trailing update), the vectors of the solves stay in the registers of one
// wave, and the two adjoint solves run in two waves side by side.
#pragma once

#include "fit_dev.h"

namespace ksdf {
namespace {

constexpr int FIT64_VEC = 10 * MAXM;   // samples (3), variances, pivots, column, vectors
__host__ __device__ constexpr int fit64_smem_doubles(int m) { return FIT64_VEC + m * (m + 1) / 2; }

// Right-looking Cholesky of the packed lower triangle Ap in LDS; the pivots' L_jj go to dg
// and their reciprocals to rd (the diagonal of Ap keeps the pivots until the end).  False,
// uniformly over the block, on a non-positive pivot.
__device__ __forceinline__ bool fit64_cholesky(double* Ap, int m, double* col, double* dg, double* rd) {
  const int tid = threadIdx.x;
  for (int j = 0; j < m; ++j) {
    __syncthreads();
    const double d = Ap[pk(j, j)];
    if (!(d > 0.0)) return false;
    const double ljj = sqrt(d), inv = 1.0 / ljj;
    for (int i = j + 1 + tid; i < m; i += blockDim.x) {
      const double l = Ap[pk(i, j)] * inv;
      Ap[pk(i, j)] = l;
      col[i] = l;
    }
    if (tid == 0) {
      dg[j] = ljj;
      rd[j] = inv;
    }
    __syncthreads();
    for (int r = j + 1 + tid / 16; r < m; r += blockDim.x / 16) {
      const double lr = col[r];
      double* row = Ap + pk(r, 0);
      for (int c = j + 1 + (tid & 15); c <= r; c += 16) row[c] -= lr * col[c];
    }
  }
  __syncthreads();
  for (int j = tid; j < m; j += blockDim.x) Ap[pk(j, j)] = dg[j];
  __syncthreads();
  return true;
}

// x = A^{-1} b by one wave from the factor in LDS: the unknowns leave their lanes by
// readlane and every lane subtracts its own entry's column
__device__ __forceinline__ WVec<double> fit64_solve(const double* Lp, const double* rd, int m,
                                                    const WVec<double>& b) {
  const int lane = threadIdx.x & 63;
  double q[SLOTS], r[SLOTS];
  WVec<double> y;
#pragma unroll
  for (int t = 0; t < SLOTS; ++t) {
    const int i = t * 64 + lane;
    q[t] = i < m ? rd[i] : 0.0;
    r[t] = i < m ? b.s[t] : 0.0;
    y.s[t] = 0.0;
  }
#pragma unroll
  for (int s = 0; s < SLOTS; ++s) {
    const int lim = min(m - 64 * s, 64);
#pragma unroll 4
    for (int jj = 0; jj < lim; ++jj) {
      const int j = s * 64 + jj;
      const double yj = readlane(r[s] * q[s], jj);
      if (lane == jj) y.s[s] = yj;
#pragma unroll
      for (int t = s; t < SLOTS; ++t) {
        const int i = t * 64 + lane;
        if (i > j && i < m) r[t] -= Lp[pk(i, j)] * yj;
      }
    }
  }
  r[0] = y.s[0];
#pragma unroll
  for (int t = 1; t < SLOTS; ++t) r[t] = y.s[t];
  WVec<double> x;
#pragma unroll
  for (int t = 0; t < SLOTS; ++t) x.s[t] = 0.0;
#pragma unroll
  for (int s = SLOTS - 1; s >= 0; --s) {
    const int lim = min(m - 64 * s, 64);
#pragma unroll 4
    for (int ii = lim - 1; ii >= 0; --ii) {
      const int i = s * 64 + ii;
      const double xi = readlane(r[s] * q[s], ii);
      if (lane == ii) x.s[s] = xi;
#pragma unroll
      for (int t = 0; t <= s; ++t) {
        const int k = t * 64 + lane;
        if (k < i) r[t] -= Lp[pk(i, k)] * xi;
      }
    }
  }
  return x;
}

// Fit cell c with the whole block; smem holds fit64_smem_doubles(m) doubles for its m.
// emit32 writes the FP32 store.
__device__ void fit64_cell(const FitArgs& A, int c, double* smem) {
  double* xs = smem;
  double* sv = xs + 3 * MAXM;
  double* col = sv + MAXM;
  double* dg = col + MAXM;
  double* rd = dg + MAXM;
  double* a_s = rd + MAXM;
  double* g_s = a_s + MAXM;
  double* p_s = g_s + MAXM;
  double* Ap = smem + FIT64_VEC;
  const int lane = threadIdx.x & 63, wave = threadIdx.x / 64;
  const int b = A.offsets[c], m = A.offsets[c + 1] - b;
  __syncthreads();   // the previous task of this block may still read smem
  for (int i = threadIdx.x; i < m; i += blockDim.x) {
    const long s = A.samples[b + i];
    for (int d = 0; d < 3; ++d)
      xs[3 * i + d] = load_coord<double>(A.pts, A.pts_f64, s, d) - A.centre64[3 * c + d];
    sv[i] = A.svar ? (A.pts_f64 ? static_cast<const double*>(A.svar)[s]
                                : (double)static_cast<const float*>(A.svar)[s])
                   : A.noise;
  }
  __syncthreads();
  assemble<double>(Ap, xs, sv, m, 1.0 / (2.0 * A.ell * A.ell), A.kernel, std::sqrt(3.0) / A.ell);
  const bool ok = fit64_cholesky(Ap, m, col, dg, rd);
  __syncthreads();
  WVec<double> a;
#pragma unroll
  for (int t = 0; t < SLOTS; ++t) a.s[t] = 0.0;
  if (wave == 0 && ok) {
    WVec<double> ones;
#pragma unroll
    for (int t = 0; t < SLOTS; ++t) ones.s[t] = 1.0;
    a = fit64_solve(Ap, rd, m, ones);
#pragma unroll
    for (int t = 0; t < SLOTS; ++t) {
      const int i = t * 64 + lane;
      if (i < m) a_s[i] = a.s[t];
    }
  }
  if (A.adjoint && ok) {
    // adjoint vectors of the fit in FP64: xi_l = A^{-1} (dA/dl) a, xi_s = A^{-1} a
    __syncthreads();
    const double inv2l2 = 1.0 / (2.0 * A.ell * A.ell), il3 = 1.0 / (A.ell * A.ell * A.ell);
    const bool matern = A.kernel == KSDF_KERNEL_MATERN32;
    const double mcd = std::sqrt(3.0) / A.ell;
    // dA_ij/dl without the 1/l^3 (RBF) or 1/l (Matern 3/2) factor
    auto dkl = [&](double r2) {
      return matern ? mcd * mcd * r2 * exp(-mcd * sqrt(r2)) : exp(-r2 * inv2l2) * r2;
    };
    const double lfac = matern ? 1.0 / A.ell : il3;
    // rows over the lanes of a half block each, the columns split between the halves
    const int half = threadIdx.x / 128, i = threadIdx.x & 127;
    double acc = 0.0;
    if (i < m)
      for (int k = half; k < m; k += 2) {
        if (k == i) continue;
        const double dx = xs[3 * i] - xs[3 * k], dy = xs[3 * i + 1] - xs[3 * k + 1],
                     dz = xs[3 * i + 2] - xs[3 * k + 2];
        const double r2 = dx * dx + dy * dy + dz * dz;
        acc += dkl(r2) * a_s[k];
      }
    if (i < m && half == 1) p_s[i] = acc;
    __syncthreads();
    if (i < m && half == 0) g_s[i] = (acc + p_s[i]) * lfac;
    __syncthreads();
    if (wave < 2) {
      WVec<double> v;
#pragma unroll
      for (int t = 0; t < SLOTS; ++t) {
        const int e = t * 64 + lane;
        v.s[t] = e < m ? (wave == 0 ? g_s[e] : a_s[e]) : 0.0;
      }
      const bool zero = wave == 1 && A.svar;   // per-sample variances: no uniform adjoint
      if (!zero) v = fit64_solve(Ap, rd, m, v);
#pragma unroll
      for (int t = 0; t < SLOTS; ++t) {
        const int e = t * 64 + lane;
        if (e < m) {
          const double x = zero ? 0.0 : v.s[t];
          if (A.emit32) {
            const float hi = (float)x;
            A.xi32[4L * (b + e) + wave] = hi;
            A.xi32[4L * (b + e) + 2 + wave] = (float)(x - (double)hi);
          } else {
            A.xi64[2L * (b + e) + wave] = x;
          }
        }
      }
    }
    if (A.D32 || A.D64) {
      for (int e = threadIdx.x; e < m * (m + 1) / 2; e += blockDim.x) {
        int i2 = (int)((sqrt(8.0 * (double)e + 1.0) - 1.0) * 0.5);
        while (i2 * (i2 + 1) / 2 > e) --i2;
        while ((i2 + 1) * (i2 + 2) / 2 <= e) ++i2;
        const int k = e - i2 * (i2 + 1) / 2;
        const double dx = xs[3 * i2] - xs[3 * k], dy = xs[3 * i2 + 1] - xs[3 * k + 1],
                     dz = xs[3 * i2 + 2] - xs[3 * k + 2];
        const double r2 = dx * dx + dy * dy + dz * dz;
        const double dv = (i2 == k) ? 0.0 : dkl(r2) * lfac;
        if (A.emit32) A.D32[A.loff[c] + e] = (float)dv;
        else A.D64[A.loff[c] + e] = dv;
      }
    }
  }
  __syncthreads();
  if (A.emit32) {
    write_cell<double, float>(Ap, xs, sv, a, m, ok, A.ps32 + 4L * b, A.sv32 + b,
                              A.L32 + A.loff[c], A.box32 + 8L * c, A.plo32 + 4L * b);
  } else {
    write_cell<double, double>(Ap, xs, sv, a, m, ok, A.ps64 + 4L * b, A.sv64 + b,
                               A.L64 + A.loff[c], A.box32 ? A.box32 + 8L * c : nullptr);
  }
  if (threadIdx.x == 0) {
    const uint8_t st = (A.emit32 ? KSDF_C_FP64 : 0) | (ok ? 0 : KSDF_C_FAILED);
    A.cstatus[c] = st;
    if (A.user_status) A.user_status[c] = st;
  }
}

}  // namespace
}  // namespace ksdf
