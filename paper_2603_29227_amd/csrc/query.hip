// Query forward: the per-point SDF prediction of Sec. IV-B.
//
// For each query x*: the K nearest occupied cell centres (ties by id); for each of
// them the log-GP mean with App. D scaling, f' = sum_i a_i exp(-(z_i^2 - d^2)/2l^2)
// and u_c = sqrt(d^2 - 2 l^2 ln f') (Table I; f' <= 0 excludes the cell, u^2 < 0
// clamps to 0); min-fusion u = min_c u_c (ties to the lowest id); then, on the
// argmin cell, the UDF gradient w/|w| with w = sum_i a_i e_i (x* - x_i), the GP
// variance 1 - |L^{-1} k*|^2 by forward substitution, and the softmin variance
// sum_i c_i^2 sigma_i^2, c_i = s_i (alpha h - alpha z_i + 1).  d = s u (sign input).
//
// The Matern 3/2 kernel of Table I replaces k by (1 + c r) exp(-c r), c = sqrt(3)/l,
// the transform by u = d - ln(f')/c (App. D scaling gamma = exp(c d)) and e_i in w
// by exp(-c (z_i - d)), since dk/dr = -c^2 r exp(-c r); u < 0 clamps to 0.
//
// This file holds the plain path of FP64 models: every candidate evaluated, every read
// straight from the per-cell store (no bucketing).
#include <cmath>

#include "ksdf_internal.h"
#include "group_dev.h"

namespace ksdf {

template <class T>
struct QueryArgs {
  const T* pts;
  long Q;
  long first;         // the launch's first query
  const int8_t* sign;
  T* mean;
  T* grad;
  T* var;
  T* var_f;
  T* grad_var;
  int* argmin;
  uint8_t* qst;
  int n_cells;
  int k;
  const int* offsets;
  const long* loff;
  const T* ps;        // [nnz,4] (px,py,pz,a) cell-local
  const T* sv;        // [nnz]
  const T* L;         // packed rows, reciprocal diagonal
  const float* centre32;
  const double* centre64;
  double origin[3];
  double h;
  int lo[3];
  int dims[3];
  double cand_slack;  // margin of the candidate scan's end (cand_slack_of)
  long n_boxes;
  const int* box_off;
  const int* box_list;
  T inv2l2;           // 1/(2 l^2)
  T two_l2;           // 2 l^2
  T alpha;            // softmin temperature
  int kernel;         // KSDF_KERNEL_*
  T mc;               // Matern 3/2 rate sqrt(3) / l
};

namespace {

// Candidate distances: an integer decision, so both precisions use a fixed
// rounding sequence (float: sub, mul, two fma; double: sub, mul, add in order).
__device__ __forceinline__ float cand_d2(float qx, float qy, float qz, const float* c) {
  const float dx = __fsub_rn(qx, c[0]), dy = __fsub_rn(qy, c[1]), dz = __fsub_rn(qz, c[2]);
  float t = __fmul_rn(dx, dx);
  t = __fmaf_rn(dy, dy, t);
  return __fmaf_rn(dz, dz, t);
}
__device__ __forceinline__ double cand_d2(double qx, double qy, double qz, const double* c) {
  const double dx = __dsub_rn(qx, c[0]), dy = __dsub_rn(qy, c[1]), dz = __dsub_rn(qz, c[2]);
  return __dadd_rn(__dadd_rn(__dmul_rn(dx, dx), __dmul_rn(dy, dy)), __dmul_rn(dz, dz));
}
template <class T> __device__ __forceinline__ const T* centre_of(const QueryArgs<T>& A, int c);
template <> __device__ __forceinline__ const float* centre_of(const QueryArgs<float>& A, int c) {
  return A.centre32 + 4L * c;
}
template <> __device__ __forceinline__ const double* centre_of(const QueryArgs<double>& A, int c) {
  return A.centre64 + 3L * c;
}

template <class T>
__device__ T cell_udf(const QueryArgs<T>& A, int c, T qx, T qy, T qz, bool* clamped) {
  const int b = A.offsets[c], m = A.offsets[c + 1] - b;
  const double* cc = A.centre64 + 3L * c;
  const T lx = qx - (T)cc[0], ly = qy - (T)cc[1], lz = qz - (T)cc[2];
  const T* p = A.ps + 4L * b;
  T d2 = (T)INFINITY;
  for (int i = 0; i < m; ++i) {
    const T dx = lx - p[4 * i], dy = ly - p[4 * i + 1], dz = lz - p[4 * i + 2];
    d2 = min(d2, dx * dx + dy * dy + dz * dz);
  }
  T f = T(0);
  *clamped = false;
  if (A.kernel == KSDF_KERNEL_MATERN32) {
    const T d = sqrt(d2);
    for (int i = 0; i < m; ++i) {
      const T dx = lx - p[4 * i], dy = ly - p[4 * i + 1], dz = lz - p[4 * i + 2];
      const T z = sqrt(dx * dx + dy * dy + dz * dz);
      f += p[4 * i + 3] * (T(1) + A.mc * z) * exp(-A.mc * (z - d));
    }
    if (!(f > T(0))) return (T)INFINITY;
    const T u = d - log(f) / A.mc;
    if (u < T(0)) {
      *clamped = true;
      return T(0);
    }
    return u;
  }
  for (int i = 0; i < m; ++i) {
    const T dx = lx - p[4 * i], dy = ly - p[4 * i + 1], dz = lz - p[4 * i + 2];
    const T z2 = dx * dx + dy * dy + dz * dz;
    f += p[4 * i + 3] * exp(-(z2 - d2) * A.inv2l2);
  }
  if (!(f > T(0))) return (T)INFINITY;
  const T u2 = d2 - A.two_l2 * log(f);
  if (u2 < T(0)) {
    *clamped = true;
    return T(0);
  }
  return sqrt(u2);
}

// Eight lanes per query (group_dev.h): each lane scans every eighth entry of the candidate
// list and evaluates one or two of the candidates, and the argmin cell's sums and its
// triangular solve are shared as in query_group.hip.  One thread per query had to keep the
// kernel vector of m doubles in memory and left most of the chip idle below some hundred
// thousand queries (room of 64-sample cells: 4,000 points 1.21 ms, 64,000 1.48 and 1e6
// 22.3; eight lanes take 0.074, 0.63 and 9.1; a 128^3 grid 11.7 and 9.7).
template <class T>
struct QueryGroupLds {
  alignas(16) T t[8 * GT_STRIDE];
  alignas(16) T k[GQ * GK_STRIDE];
};

template <class T, int KM>
__global__ void __launch_bounds__(64) query_plain_kernel(QueryArgs<T> A) {
  __shared__ QueryGroupLds<T> S;
  constexpr int NC = KM / GL;
  const int lane = threadIdx.x & 63, g = lane & (GL - 1), base = lane - g;
  const long q = A.first + (long)blockIdx.x * GQ + lane / GL;
  const bool active = q < A.Q;
  const long qq = active ? q : 0;
  const T qx = A.pts[3 * qq], qy = A.pts[3 * qq + 1], qz = A.pts[3 * qq + 2];
  // the K nearest centres: sorted private lists, then group-wide minima of (distance, id)
  T cd[KM];
  int ci[KM];
#pragma unroll
  for (int r = 0; r < KM; ++r) {
    cd[r] = (T)INFINITY;
    ci[r] = 0x7fffffff;
  }
  const long key[3] = {(long)floor(((double)qx - A.origin[0]) / A.h) - A.lo[0],
                       (long)floor(((double)qy - A.origin[1]) / A.h) - A.lo[1],
                       (long)floor(((double)qz - A.origin[2]) / A.h) - A.lo[2]};
  const bool inside = A.n_boxes > 0 && key[0] >= 0 && key[0] < A.dims[0] && key[1] >= 0 &&
                      key[1] < A.dims[1] && key[2] >= 0 && key[2] < A.dims[2];
  int beg = 0, end = active ? A.n_cells : 0;
  if (active && inside) {
    const long bx = (key[0] * A.dims[1] + key[1]) * A.dims[2] + key[2];
    beg = A.box_off[bx];
    end = A.box_off[bx + 1];
  }
  // two entries a lane at a time, until no later centre of a list in the order of distances
  // from the box's centre can enter (cand_scan_over in query_dev.h)
  const bool sorted = inside && end - beg <= INDEX_SORTED_MAX;
  T mid[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) mid[d] = (T)(A.origin[d] + ((double)(key[d] + A.lo[d]) + 0.5) * A.h);
  const T rho = sqrt(cand_d2(qx, qy, qz, mid));
  for (int t0 = beg; t0 < end; t0 += 2 * GL) {   // uniform in the group
    T at = (T)0;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int t = t0 + g + u * GL;
      int xi = inside ? A.box_list[min(t, end - 1)] : min(t, end - 1);
      const auto ce = centre_of(A, xi);
      at = cand_d2(mid[0], mid[1], mid[2], ce);
      T x = cand_d2(qx, qy, qz, ce);
      if (t < end && (x < cd[KM - 1] || (x == cd[KM - 1] && xi < ci[KM - 1]))) {
#pragma unroll
        for (int r = 0; r < KM; ++r) {
          if (x < cd[r] || (x == cd[r] && xi < ci[r])) {
            const T tx = cd[r];
            const int ti = ci[r];
            cd[r] = x;
            ci[r] = xi;
            x = tx;
            xi = ti;
          }
        }
      }
    }
    const T far = (sqrt(group_max(cd[KM / GL - 1])) + rho) * (T)(1 + 0x1p-14) + (T)A.cand_slack;
    if (sorted && group_all(at > far * far)) break;
  }
  const int n = min(A.k, end - beg);
  int mine[NC];   // the lane's candidates: ranks g and g + 8
#pragma unroll
  for (int s = 0; s < NC; ++s) mine[s] = 0x7fffffff;
#pragma unroll
  for (int r = 0; r < KM; ++r) {
    T d = cd[0];
    int id = ci[0];
    group_min(d, id);
    if (r % GL == g && r < n) mine[r / GL] = id;
    if (ci[0] == id) {   // ids are unique: one lane drops its head
#pragma unroll
      for (int j = 0; j + 1 < KM; ++j) {
        cd[j] = cd[j + 1];
        ci[j] = ci[j + 1];
      }
      cd[KM - 1] = (T)INFINITY;
      ci[KM - 1] = 0x7fffffff;
    }
  }
  // min-fusion, ties to the lower id
  T best = (T)INFINITY;
  int bc = 0x7fffffff;
  bool cl = false;
#pragma unroll
  for (int s = 0; s < NC; ++s) {
    if (mine[s] != 0x7fffffff) {
      bool c1;
      const T u = cell_udf(A, mine[s], qx, qy, qz, &c1);
      if (u < best || (u == best && u < (T)INFINITY && mine[s] < bc)) {
        best = u;
        bc = mine[s];
        cl = c1;
      }
    }
  }
  const int own = bc;
  group_min(best, bc);
  const bool bclamp = ((__ballot(cl && own == bc) >> base) & 0xffull) != 0ull;
  const T sgn = active && A.sign ? (T)A.sign[qq] : T(1);
  const bool outside = !inside;
  uint8_t st = outside ? KSDF_Q_OUTSIDE_INDEX : 0;
  if (bc == 0x7fffffff) {   // uniform over each group
    if (active && g == 0) {
      A.mean[q] = (T)INFINITY;
      for (int d = 0; d < 3; ++d) A.grad[3 * q + d] = T(0);
      A.var[q] = (T)INFINITY;
      if (A.var_f) A.var_f[q] = T(1);
      if (A.grad_var)
        for (int d = 0; d < 3; ++d) A.grad_var[3 * q + d] = (T)INFINITY;
      if (A.argmin) A.argmin[q] = -1;
      if (A.qst) A.qst[q] = st | KSDF_Q_NO_VALID_CELL;
    }
    return;
  }
  if (bclamp) st |= KSDF_Q_CLAMPED;
  const int b = A.offsets[bc], m = A.offsets[bc + 1] - b;
  const double* cc = A.centre64 + 3L * bc;
  const T lx = qx - (T)cc[0], ly = qy - (T)cc[1], lz = qz - (T)cc[2];
  const T* p = A.ps + 4L * b;
  const T* sv = A.sv + b;
  T* row = S.t + lane;
  T* k = S.k + lane / GL * GK_STRIDE;
  auto put = [&](int r, T v) { row[r * GT_STRIDE] = v; };
  auto offset = [&](int i, T e[3]) {
    e[0] = lx - p[4 * i];
    e[1] = ly - p[4 * i + 1];
    e[2] = lz - p[4 * i + 2];
    return e[0] * e[0] + e[1] * e[1] + e[2] * e[2];
  };
  T d2 = (T)INFINITY;
  for (int i = g; i < m; i += GL) {
    T e[3];
    d2 = min(d2, offset(i, e));
  }
  d2 = min(d2, dpp<DPP_XOR1>(d2));
  d2 = min(d2, dpp<DPP_XOR2>(d2));
  d2 = min(d2, dpp<DPP_MIRROR8>(d2));
  const T gs = exp(-d2 * A.inv2l2);   // 1/gamma: k_i = e_i / gamma
  const T zmin = sqrt(d2);
  const bool matern = A.kernel == KSDF_KERNEL_MATERN32;
  // w (3), S, H and the kernel vector
  T acc = T(0);
  put(7, T(1));
  for (int i0 = 0; i0 < m; i0 += GL) {
    const int i = i0 + g;
    const bool in = i < m;
    const int j = in ? i : 0;
    T d[3];
    const T z2 = offset(j, d);
    const T z = sqrt(z2);
    T e, t;
    if (matern) {
      e = exp(-A.mc * (z - zmin));
      t = (T(1) + A.mc * z) * exp(-A.mc * z);
    } else {
      e = exp(-(z2 - d2) * A.inv2l2);
      t = e * gs;
    }
    put(0, in ? p[4 * j + 3] * e : T(0));
    put(1, d[0]);
    put(2, d[1]);
    put(3, d[2]);
    put(4, in ? exp(-A.alpha * (z - zmin)) : T(0));
    put(5, z);
    if (in) k[i] = t;
    wave_lds_sync();
    group_fma(S.t, lane_entry(lanes8(0, 0, 0, 7, 4, 7, 7, 7)),
              lane_entry(lanes8(1, 2, 3, 4, 5, 7, 7, 7)), acc);
    wave_lds_sync();
  }
  const T w0 = group_lane<0>(acc), w1 = group_lane<1>(acc), w2 = group_lane<2>(acc);
  const T Ss = group_lane<3>(acc);
  const T h = group_lane<4>(acc) / Ss;
  const T vv = A.var_f ? group_forward_subst(k, A.L + A.loff[bc], m) : T(0);
  // the softmin variance, and the sums Vs = sum s_i v_i, g = sum c_i v_i of the gradient's
  acc = T(0);
  for (int i0 = 0; i0 < m; i0 += GL) {
    const int i = i0 + g;
    const bool in = i < m;
    const int j = in ? i : 0;
    T d[3];
    const T z = sqrt(offset(j, d));
    const T s = in ? exp(-A.alpha * (z - zmin)) / Ss : T(0);
    const T c = s * (A.alpha * h - A.alpha * z + T(1));
    const T rz = z > T(0) ? T(1) : T(0);
    put(0, c * c);
    put(1, in ? sv[j] : T(0));   // not 0 times an infinite variance
    put(2, rz > T(0) ? d[0] / z : T(0));
    put(3, rz > T(0) ? d[1] / z : T(0));
    put(4, rz > T(0) ? d[2] / z : T(0));
    put(5, s);
    put(6, c);
    wave_lds_sync();
    group_fma(S.t, lane_entry(lanes8(0, 5, 5, 5, 6, 6, 6, 7)),
              lane_entry(lanes8(1, 2, 3, 4, 2, 3, 4, 7)), acc);
    wave_lds_sync();
  }
  const T var = group_lane<0>(acc);
  if (A.grad_var) {
    const T Vs[3] = {group_lane<1>(acc), group_lane<2>(acc), group_lane<3>(acc)};
    const T gg[3] = {group_lane<4>(acc), group_lane<5>(acc), group_lane<6>(acc)};
    acc = T(0);
    for (int i0 = 0; i0 < m; i0 += GL) {
      const int i = i0 + g;
      const bool in = i < m;
      const int j = in ? i : 0;
      T dd[3];
      const T z = sqrt(offset(j, dd));
      const bool ok = in && z > T(0);   // a sample at the query has no direction
      const T s = exp(-A.alpha * (z - zmin)) / Ss;
      const T li = s * (A.alpha * h - A.alpha * z + T(1));
      const T lz2 = (li / z) * (li / z);
      put(0, ok ? sv[j] : T(0));
      for (int d = 0; d < 3; ++d) {
        const T vd = dd[d] / z;
        const T w = li * (vd - Vs[d]) + s * (vd - gg[d]);
        put(1 + d, ok ? A.alpha * A.alpha * w * w + lz2 * (T(1) - vd * vd) : T(0));
      }
      wave_lds_sync();
      group_fma(S.t, 0, lane_entry(lanes8(1, 2, 3, 1, 1, 1, 1, 1)), acc);
      wave_lds_sync();
    }
    const T gv[3] = {group_lane<0>(acc), group_lane<1>(acc), group_lane<2>(acc)};
    if (g == 0)
      for (int d = 0; d < 3; ++d) A.grad_var[3 * q + d] = gv[d];
  }
  if (g != 0) return;
  const T wn = sqrt(w0 * w0 + w1 * w1 + w2 * w2);
  T gx = 0, gy = 0, gz = 0;
  if (wn > T(0)) {
    gx = w0 / wn;
    gy = w1 / wn;
    gz = w2 / wn;
  } else {
    st |= KSDF_Q_GRAD_ZERO;
  }
  A.mean[q] = sgn * best;
  A.grad[3 * q] = sgn * gx;
  A.grad[3 * q + 1] = sgn * gy;
  A.grad[3 * q + 2] = sgn * gz;
  A.var[q] = var;
  if (A.var_f) A.var_f[q] = max(T(1) - vv, T(0));
  if (A.argmin) A.argmin[q] = bc;
  if (A.qst) A.qst[q] = st;
}

template <class T>
QueryArgs<T> make_args(const ksdf_model* m, const void* points, long Q, const int8_t* sign,
                       void* mean, void* grad, void* var, void* var_f, void* grad_var, int* argmin,
                       uint8_t* q_status) {
  QueryArgs<T> A{};
  A.pts = static_cast<const T*>(points);
  A.Q = Q;
  A.sign = sign;
  A.mean = static_cast<T*>(mean);
  A.grad = static_cast<T*>(grad);
  A.var = static_cast<T*>(var);
  A.var_f = static_cast<T*>(var_f);
  A.grad_var = static_cast<T*>(grad_var);
  A.argmin = argmin;
  A.qst = q_status;
  A.n_cells = m->n_cells;
  A.k = std::min(m->k_fuse, m->n_cells);
  A.offsets = m->offsets;
  A.loff = m->loff;
  A.centre32 = m->centre32;
  A.centre64 = m->centre64;
  for (int d = 0; d < 3; ++d) {
    A.origin[d] = m->origin[d];
    A.lo[d] = m->index.lo[d];
    A.dims[d] = m->index.dims[d];
  }
  A.h = m->h;
  A.cand_slack = cand_slack_of(m);
  A.n_boxes = m->index.n_boxes;
  A.box_off = m->index.box_off;
  A.box_list = m->index.box_list;
  A.inv2l2 = (T)(1.0 / (2.0 * m->ell * m->ell));
  A.two_l2 = (T)(2.0 * m->ell * m->ell);
  A.alpha = (T)m->alpha;
  A.kernel = m->kernel;
  A.mc = (T)(std::sqrt(3.0) / m->ell);
  return A;
}

}  // namespace

size_t query_workspace_bytes(const ksdf_model* m, long Q) {
  return m->precision == KSDF_FP32 ? query_fast_workspace_bytes(m, Q) : 0;
}

int launch_query(const ksdf_model* m, const void* points, long Q, const int8_t* sign, void* mean,
                 void* grad, void* var, void* var_f, void* grad_var, int* argmin, uint8_t* q_status, void* ws,
                 size_t ws_bytes, hipStream_t s, bool prebucketed) {
  if (Q == 0) return KSDF_OK;
  if (m->precision == KSDF_FP64) {
    QueryArgs<double> A = make_args<double>(m, points, Q, sign, mean, grad, var, var_f, grad_var, argmin, q_status);
    A.ps = m->ps64;
    A.sv = m->sv64;
    A.L = m->L64;
    timer_mark(m, KSDF_TIMER_QUERY, 0, s);
    group_launches(Q, [&](long first, unsigned grid) {
      A.first = first;
      if (m->k_fuse <= 8) hipLaunchKernelGGL((query_plain_kernel<double, 8>), dim3(grid), dim3(64), 0, s, A);
      else hipLaunchKernelGGL((query_plain_kernel<double, 16>), dim3(grid), dim3(64), 0, s, A);
    });
    timer_mark(m, KSDF_TIMER_QUERY, 1, s);
  } else {
    return launch_query_fast(m, points, Q, sign, mean, grad, var, var_f, grad_var, argmin, q_status, ws,
                             ws_bytes, s, prebucketed);
  }
  KSDF_HIP_TRY(hipGetLastError());
  return KSDF_OK;
}

}  // namespace ksdf
