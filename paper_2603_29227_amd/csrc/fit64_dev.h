// FP64 fit of one cell with a workgroup of 256 threads: every cell of an FP64 model, and the
// cells of an FP32 model whose condition estimate (or a failed pivot) asks for FP64.
//
// It is bound by the chain of pivots, so a pivot costs one barrier: the threads form a
// 16 x 16 grid that holds the matrix in registers (rows and columns 16 apart), the owners of
// column j pass it through LDS, and every thread scales what it needs of it and updates its
// entries.  The finished columns collect in a packed factor in LDS, from which one wave
// solves with the vectors in its registers (two waves side by side for the two adjoint
// vectors).  With the factor in global memory and three barriers a pivot, the 47
// ill-conditioned cells of the uneven room took 724 us; with it in LDS 287.
#pragma once

#include "fit_dev.h"
#include "wave_ops.h"

namespace ksdf {
namespace {

constexpr int FIT64_THREADS = 256;
constexpr int FIT64_VEC = 10 * MAXM;   // samples (3), variances, pivots, columns (2), vectors
__host__ __device__ constexpr int fit64_smem_doubles(int m) { return FIT64_VEC + m * (m + 1) / 2; }

// 1 / b and a / b to the last bit (Markstein 1990) from a reciprocal within a few ulp and from
// the reciprocal itself: what the division would give, for a chain of 4 or 5 operations in the
// place of its 11.  (Cells with the same samples tie but for the last bits of their weights, so
// these decide which of them a query names.)  The 5485 cells of the room take 538 us with
// them; 458 us with rsqrt and products of reciprocals in their place, for other last bits.
__device__ __forceinline__ double reciprocal(double b, double y) {
  y = fma(fma(-b, y, 1.0), y, y);
  return fma(fma(-b, y, 1.0), y, y);
}
__device__ __forceinline__ double quotient(double a, double b, double inv) {
  double q = a * inv;
  q = fma(fma(-q, b, a), inv, q);
  return fma(fma(-q, b, a), inv, q);
}

// Right-looking Cholesky of A = K + Sigma, entries from entry(row, column) for column <= row <
// m: the packed factor with its true diagonal to Lp, the pivots' reciprocals to rd.  col: two
// columns of MB.  False, uniformly over the block, on a non-positive pivot.
template <int MB, class F>
__device__ __forceinline__ bool fit64_cholesky(F&& entry, int m, double* Lp, double* col, double* rd) {
  constexpr int NB = MB / 16;
  const int tr = threadIdx.x / 16, tc = threadIdx.x & 15;
  double a[NB][NB];   // entry (tr + 16 i, tc + 16 k) for k <= i; the identity past m
  static_for<0, NB>([&](auto I) {
    constexpr int i = I;
    static_for<0, i + 1>([&](auto K) {
      constexpr int k = K;
      const int r = tr + 16 * i, c = tc + 16 * k;
      a[i][k] = r == c ? 1.0 : 0.0;
      if (c <= r && r < m) a[i][k] = entry(r, c);
    });
  });
  bool ok = true;
  static_for<0, NB>([&](auto B) {
    constexpr int bj = B;
    for (int jj = 0; jj < 16; ++jj) {
      const int j = 16 * bj + jj;
      if (!ok || j >= m) break;   // uniform
      // two columns in turn: the next but one is written after every thread has passed the
      // next barrier, which it reaches with this column read
      double* cj = col + (j & 1) * MAXM;
      if (tc == jj)
        static_for<bj, NB>([&](auto I) { cj[tr + 16 * I] = a[I][bj]; });
      __syncthreads();
      const double d = cj[j];
      if (!(d > 0.0)) {
        ok = false;
        break;
      }
      const double ljj = sqrt(d);
      // an infinite pivot (a sample of infinite variance) divides to 0, which the corrections
      // would make NaN
      const double inv = ljj < INFINITY ? reciprocal(ljj, rsqrt(d)) : 0.0;
      double lr[NB], lc[NB];
      static_for<bj, NB>([&](auto I) {
        constexpr int i = I;
        lr[i] = cj[tr + 16 * i] * inv;
        lc[i] = cj[tc + 16 * i] * inv;
      });
      if (tc == jj)
        static_for<bj, NB>([&](auto I) {
          const int r = tr + 16 * I;
          if (r >= j && r < m) Lp[pk(r, j)] = r == j ? ljj : lr[I];
        });
      if (threadIdx.x == 0) rd[j] = inv;
      if (tr <= jj) lr[bj] = 0.0;   // rows and columns up to j are finished
      if (tc <= jj) lc[bj] = 0.0;
      static_for<bj, NB>([&](auto I) {
        constexpr int i = I;
        static_for<bj, i + 1>([&](auto K) { a[i][K] = fma(-lr[i], lc[K], a[i][K]); });
      });
    }
  });
  __syncthreads();
  return ok;
}

// x = A^{-1} b by one wave from the factor in LDS: the unknowns leave their lanes by
// readlane and every lane subtracts its own entry's column.  The factor's reads do not depend
// on the chain (lanes past the column read an entry they do not use), so they run ahead.
__device__ __forceinline__ WVec<double> fit64_solve(const double* Lp, const double* rd, int m,
                                                    const WVec<double>& b) {
  const int lane = threadIdx.x & 63;
  // the rows' pivots and their reciprocals q; an infinite pivot (q = 0) is taken as 0, from
  // which quotient gives the 0 of a division by it
  double q[SLOTS], p[SLOTS], r[SLOTS];
  int row[SLOTS];
  WVec<double> y, x;
#pragma unroll
  for (int t = 0; t < SLOTS; ++t) {
    row[t] = min(t * 64 + lane, m - 1);
    const bool in = t * 64 + lane < m;
    q[t] = in ? rd[row[t]] : 0.0;
    p[t] = Lp[pk(row[t], row[t])];
    if (!(p[t] < INFINITY)) p[t] = 0.0;
    r[t] = in ? b.s[t] : 0.0;
    y.s[t] = 0.0;
    x.s[t] = 0.0;
  }
#pragma unroll
  for (int s = 0; s < SLOTS; ++s) {
    const int lim = min(m - 64 * s, 64);
#pragma unroll 8
    for (int jj = 0; jj < lim; ++jj) {
      const int j = s * 64 + jj;
      double l[SLOTS];
#pragma unroll
      for (int t = s; t < SLOTS; ++t) l[t] = Lp[pk(row[t], min(j, row[t]))];
      const double yj = readlane(quotient(r[s], p[s], q[s]), jj);
      y.s[s] = lane == jj ? yj : y.s[s];
#pragma unroll
      for (int t = s; t < SLOTS; ++t) r[t] = t * 64 + lane > j ? fma(-l[t], yj, r[t]) : r[t];
    }
  }
#pragma unroll
  for (int t = 0; t < SLOTS; ++t) r[t] = y.s[t];
#pragma unroll
  for (int s = SLOTS - 1; s >= 0; --s) {
    const int lim = min(m - 64 * s, 64);
#pragma unroll 8
    for (int ii = lim - 1; ii >= 0; --ii) {
      const int i = s * 64 + ii;
      double l[SLOTS];
#pragma unroll
      for (int t = 0; t <= s; ++t) l[t] = Lp[pk(i, min(t * 64 + lane, i))];
      const double xi = readlane(quotient(r[s], p[s], q[s]), ii);
      x.s[s] = lane == ii ? xi : x.s[s];
#pragma unroll
      for (int t = 0; t <= s; ++t) r[t] = t * 64 + lane < i ? fma(-l[t], xi, r[t]) : r[t];
    }
  }
  return x;
}

// Fit cell c (m <= MB) with the whole block; smem holds fit64_smem_doubles(MB) doubles.
// emit32 writes the FP32 store.
template <int MB>
__device__ void fit64_cell(const FitArgs& A, int c, double* smem) {
  double* xs = smem;
  double* sv = xs + 3 * MAXM;
  double* col = sv + MAXM;
  double* rd = col + 2 * MAXM;
  double* a_s = rd + MAXM;
  double* g_s = a_s + MAXM;
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
  const double inv2l2 = 1.0 / (2.0 * A.ell * A.ell), il3 = 1.0 / (A.ell * A.ell * A.ell);
  const bool matern = A.kernel == KSDF_KERNEL_MATERN32;
  const double mcd = std::sqrt(3.0) / A.ell;
  auto dist2 = [&](int i, int k) {
    const double dx = xs[3 * i] - xs[3 * k], dy = xs[3 * i + 1] - xs[3 * k + 1],
                 dz = xs[3 * i + 2] - xs[3 * k + 2];
    return dx * dx + dy * dy + dz * dz;
  };
  const bool ok = fit64_cholesky<MB>(
      [&](int i, int k) {
        const double r2 = dist2(i, k);
        double v;
        if (matern) {
          const double t = mcd * sqrt(r2);
          v = (1.0 + t) * exp(-t);
        } else {
          v = exp(-r2 * inv2l2);
        }
        return i == k ? v + sv[i] : v;
      },
      m, Ap, col, rd);
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
    // dA_ij/dl without the 1/l^3 (RBF) or 1/l (Matern 3/2) factor
    auto dkl = [&](double r2) {
      return matern ? mcd * mcd * r2 * exp(-mcd * sqrt(r2)) : exp(-r2 * inv2l2) * r2;
    };
    const double lfac = matern ? 1.0 / A.ell : il3;
    // each row's sum by FIT64_THREADS / MB threads; their parts pass through the columns'
    // space, which is free by now
    constexpr int PARTS = FIT64_THREADS / MB;
    static_assert(PARTS * MB <= 2 * MAXM);
    const int part = threadIdx.x / MB, i = threadIdx.x % MB;
    double acc = 0.0;
    if (i < m)
      for (int k = part; k < m; k += PARTS)
        if (k != i) acc += dkl(dist2(i, k)) * a_s[k];
    col[part * MB + i] = acc;
    __syncthreads();
    if (part == 0 && i < m) {
      double g = 0.0;
#pragma unroll
      for (int p = 0; p < PARTS; ++p) g += col[p * MB + i];
      g_s[i] = g * lfac;
    }
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
        const double r2 = dist2(i2, k);
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
