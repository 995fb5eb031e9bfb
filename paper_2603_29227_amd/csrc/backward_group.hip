// Query backward with eight lanes per query (see backward.hip for the derivatives).
//
// One thread per query leaves most of the chip idle unless there are some hundred thousand
// queries, a wave that walks the cells of 64 unlike queries takes them one after the other,
// and the two triangular solves of the GP variance's adjoint need a vector of m values per
// thread, which then lives in memory.  Here the eight lanes of a query form the terms of
// eight samples at a time, pass them through LDS, and each carries some of the running sums
// in sample order; the kernel vector lives in LDS and the solves run over blocks of eight
// rows (group_dev.h).  Terms, sums and their order are those of the per-thread functions.
#include <cmath>

#include "backward_dev.h"
#include "group_dev.h"

namespace ksdf {
namespace {

template <class T, int ROWS, bool VARF>
struct BwdGroupLds {
  alignas(16) T t[ROWS * GT_STRIDE];            // terms of 8 samples x 8 queries, by kind
  alignas(16) T k[VARF ? GQ * GK_STRIDE : 4];   // k, then L^{-1} k, then A^{-1} k
};

// v^T D v for the packed strict lower triangle D (twice the lower part), v in LDS
template <class T>
__device__ __forceinline__ T group_quadratic(const T* v, const T* __restrict__ Dc, int m) {
  const int g = threadIdx.x & (GL - 1);
  T acc = T(0);
  for (int b0 = 0; b0 < m; b0 += GL) {
    const int i = b0 + g;
    const bool row = i < m;
    const T* Di = Dc + (row ? i * (i + 1) / 2 : 0);
    T t = T(0);
    for (int j0 = 0; j0 <= b0; j0 += GL) {
      T d[GL], x[GL];
#pragma unroll
      for (int e = 0; e < GL; ++e) {
        const bool in = row && j0 + e < i;
        d[e] = in ? Di[j0 + e] : T(0);
        x[e] = in ? v[j0 + e] : T(0);
      }
#pragma unroll
      for (int e = 0; e < GL; ++e) t = fma(d[e], x[e], t);
    }
    const T vi = row ? v[i] : T(0);
    static_for<0, GL>([&](auto E) {
      constexpr int e = E;
      const T te = group_lane<e>(t), ve = group_lane<e>(vi);
      if (b0 + e < m) acc = fma(T(2) * ve, te, acc);
    });
  }
  return acc;
}

// the smallest value of each group
template <class T>
__device__ __forceinline__ T group_fmin(T d) {
  d = fmin(d, dpp<DPP_XOR1>(d));
  d = fmin(d, dpp<DPP_XOR2>(d));
  return fmin(d, dpp<DPP_MIRROR8>(d));
}

// query_vjp (RBF; FP64 models, and FP32 models with a var_f cotangent)
template <class T, bool VARF>
__global__ void __launch_bounds__(64) bwd_group_kernel(BwdArgs<T> A, const int* perm) {
  __shared__ BwdGroupLds<T, 17, VARF> S;
  const int lane = threadIdx.x & 63, g = lane & (GL - 1);
  const long sq = A.first + xcd_block(gridDim.x) * GQ + lane / GL;
  const bool active = sq < A.Q;
  const long q = active ? (perm ? (long)perm[sq] : sq) : 0;
  int c = active ? A.argmin[q] : -1;
  if (c >= A.n_cells) c = -1;   // not a cell of this model: no contribution
  T gm = T(0), gv = T(0);
  if (active) mean_var_cotangents(A, q, gm, gv);
  T out_dx[3] = {T(0), T(0), T(0)};
  double out_th[2] = {0.0, 0.0};
  if (c >= 0) {   // uniform over each group
    const T lt = A.ell;
    const T x0 = A.pts[3 * q], x1 = A.pts[3 * q + 1], x2 = A.pts[3 * q + 2];
    const T s = A.sign ? (T)A.sign[q] : T(1);
    T gg[3] = {T(0), T(0), T(0)};
    if (A.d_grad)
      for (int d = 0; d < 3; ++d) gg[d] = A.d_grad[3 * q + d];
    const T gf = VARF && A.d_var_f ? A.d_var_f[q] : T(0);
    const int b = A.offsets[c], m = A.offsets[c + 1] - b;
    const T* p = A.ps + 4L * b;
    const T* sv = A.sv + b;
    const T* Lc = A.L + A.loff[c];
    constexpr int XS = sizeof(T) == 4 ? 4 : 2;   // FP32 store: float-float pairs, hi first
    const T* xi = A.xi + XS * (long)b;
    const double* cc = A.centre64 + 3L * c;
    const T l0 = x0 - (T)cc[0], l1 = x1 - (T)cc[1], l2 = x2 - (T)cc[2];
    const T inv2l2 = T(1) / A.two_l2;
    T* row = S.t + lane;
    T* k = S.k + (VARF ? lane / GL * GK_STRIDE : 0);
    auto put = [&](int r, T v) { row[r * GT_STRIDE] = v; };
    // scaling reference: the exact nearest sample
    T d2 = (T)INFINITY;
    for (int i = g; i < m; i += GL) {
      const T dx = l0 - p[4 * i], dy = l1 - p[4 * i + 1], dz = l2 - p[4 * i + 2];
      d2 = fmin(d2, dx * dx + dy * dy + dz * dz);
    }
    d2 = group_fmin(d2);
    const T ginv = exp(-d2 * inv2l2);
    const T zmin = sqrt(d2);
    // pass A: f', w' (3), Z, softmin moments S, M1, M2; k
    put(10, T(1));
    T acc = T(0);
    for (int i0 = 0; i0 < m; i0 += GL) {
      const int i = i0 + g;
      const bool in = i < m;
      const int j = in ? i : 0;
      const T dx = l0 - p[4 * j], dy = l1 - p[4 * j + 1], dz = l2 - p[4 * j + 2];
      const T z2 = dx * dx + dy * dy + dz * dz;
      const T e = in ? exp(-(z2 - d2) * inv2l2) : T(0);
      const T ae = p[4 * j + 3] * e;
      const T t = sqrt(z2) - zmin;
      const T sm = in ? exp(-A.alpha * t) : T(0);
      put(0, p[4 * j + 3]);
      put(1, e);
      put(2, ae);
      put(3, dx);
      put(4, dy);
      put(5, dz);
      put(6, z2);
      put(7, sm);
      put(8, t);
      put(9, sm * t);
      if constexpr (VARF)
        if (in) k[i] = e * ginv;
      wave_lds_sync();
      group_fma(S.t, lane_entry(lanes8(0, 2, 2, 2, 2, 10, 7, 9)),
                lane_entry(lanes8(1, 3, 4, 5, 6, 7, 8, 8)), acc);
      wave_lds_sync();
    }
    const T f = group_lane<0>(acc);
    const T w[3] = {group_lane<1>(acc), group_lane<2>(acc), group_lane<3>(acc)};
    const T Za = group_lane<4>(acc), Ss = group_lane<5>(acc), M1 = group_lane<6>(acc),
            M2 = group_lane<7>(acc);
    T vv = T(0);
    if constexpr (VARF) {
      vv = group_forward_subst(k, Lc, m);
      group_backward_subst(k, Lc, m);
    }
    const T u2 = f > T(0) ? d2 - A.two_l2 * log(f) : T(-1);
    const bool mean_live = u2 > T(0);
    const T u = mean_live ? sqrt(u2) : T(0);
    const T wn = sqrt(w[0] * w[0] + w[1] * w[1] + w[2] * w[2]);
    T y[3] = {T(0), T(0), T(0)};
    if (wn > T(0)) {
      const T gw = (gg[0] * w[0] + gg[1] * w[1] + gg[2] * w[2]) / wn;
      for (int d = 0; d < 3; ++d) y[d] = (gg[d] - gw * w[d] / wn) / wn;
    }
    const bool varf_live = VARF && (T(1) - vv) > T(0);
    const T m1 = M1 / Ss;
    const T h = zmin + m1;
    const T Vz = M2 / Ss - m1 * m1;
    // pass B: V, P, sum c^2, d var / d alpha
    acc = T(0);
    for (int i0 = 0; i0 < m; i0 += GL) {
      const int i = i0 + g;
      const bool in = i < m;
      const int j = in ? i : 0;
      const T dx = l0 - p[4 * j], dy = l1 - p[4 * j + 1], dz = l2 - p[4 * j + 2];
      const T z = sqrt(dx * dx + dy * dy + dz * dz);
      const T si = in ? exp(-A.alpha * (z - zmin)) / Ss : T(0);
      const T Bi = A.alpha * (h - z) + T(1);
      const T ci = si * Bi;
      const T svj = in ? sv[j] : T(0);   // not 0 times an infinite variance
      put(0, svj * ci);
      put(1, ci);
      put(2, si);
      put(3, T(2) * svj * ci);
      put(4, si * (h - z) * (Bi + T(1)) - A.alpha * si * Vz);
      wave_lds_sync();
      group_fma(S.t, lane_entry(lanes8(0, 0, 1, 3, 0, 0, 0, 0)),
                lane_entry(lanes8(1, 2, 1, 4, 1, 1, 1, 1)), acc);
      wave_lds_sync();
    }
    const T V = group_lane<0>(acc), P = group_lane<1>(acc), C2 = group_lane<2>(acc),
            dVa = group_lane<3>(acc);
    // pass C: the point derivative's and the weights' sums, three per lane
    put(0, T(1));
    T a0 = T(0), a1 = T(0), a2 = T(0);
    for (int i0 = 0; i0 < m; i0 += GL) {
      const int i = i0 + g;
      const bool in = i < m;
      const int j = in ? i : 0;
      const T di[3] = {l0 - p[4 * j], l1 - p[4 * j + 1], l2 - p[4 * j + 2]};
      const T z2 = di[0] * di[0] + di[1] * di[1] + di[2] * di[2];
      const T z = sqrt(z2);
      const T e = in ? exp(-(z2 - d2) * inv2l2) : T(0);
      const T ae = p[4 * j + 3] * e;
      const T si = in ? exp(-A.alpha * (z - zmin)) / Ss : T(0);
      const T ci = si * (A.alpha * (h - z) + T(1));
      const T dvdz = in ? T(2) * A.alpha * (-sv[j] * ci * (ci + si) + si * V + ci * P) : T(0);
      const T dy = di[0] * y[0] + di[1] * y[1] + di[2] * y[2];
      const T vi = VARF && in ? k[i] : T(0);
      for (int d = 0; d < 3; ++d) {
        put(1 + d, z > T(0) ? dvdz * di[d] / z : T(0));
        put(4 + d, di[d]);
      }
      put(7, ae * dy);
      put(8, ae * z2);
      if constexpr (VARF) put(9, vi * e * ginv);
      put(10, e * xi[XS * j]);
      put(11, e * xi[XS * j + 1]);
      put(12, z2);
      if constexpr (VARF) put(13, vi);
      put(14, e);
      put(15, xi[XS * j]);
      put(16, xi[XS * j + 1]);
      wave_lds_sync();
      // dxv (3), Hy (3), Wz (2) | Wz, bk (3), Eld (3), Esd | Esd (2), bkz, bb, El, Es
      group_fma(S.t, lane_entry(lanes8(0, 0, 0, 7, 7, 7, 8, 8)),
                lane_entry(lanes8(1, 2, 3, 4, 5, 6, 4, 5)), a0);
      if constexpr (VARF) {
        group_fma(S.t, lane_entry(lanes8(8, 9, 9, 9, 10, 10, 10, 11)),
                  lane_entry(lanes8(6, 4, 5, 6, 4, 5, 6, 4)), a1);
        group_fma(S.t, lane_entry(lanes8(11, 11, 9, 13, 14, 14, 0, 0)),
                  lane_entry(lanes8(5, 6, 12, 13, 15, 16, 0, 0)), a2);
      } else {
        group_fma(S.t, lane_entry(lanes8(8, 0, 0, 0, 10, 10, 10, 11)),
                  lane_entry(lanes8(6, 0, 0, 0, 4, 5, 6, 4)), a1);
        group_fma(S.t, lane_entry(lanes8(11, 11, 0, 0, 14, 14, 0, 0)),
                  lane_entry(lanes8(5, 6, 0, 0, 15, 16, 0, 0)), a2);
      }
      wave_lds_sync();
    }
    const T dxv[3] = {group_lane<0>(a0), group_lane<1>(a0), group_lane<2>(a0)};
    const T Hy[3] = {group_lane<3>(a0), group_lane<4>(a0), group_lane<5>(a0)};
    const T Wz[3] = {group_lane<6>(a0), group_lane<7>(a0), group_lane<0>(a1)};
    const T Eld[3] = {group_lane<4>(a1), group_lane<5>(a1), group_lane<6>(a1)};
    const T Esd[3] = {group_lane<7>(a1), group_lane<0>(a2), group_lane<1>(a2)};
    const T El = group_lane<4>(a2), Es = group_lane<5>(a2);
    T bk[3] = {T(0), T(0), T(0)}, bkz = T(0), bb = T(0), bDb = T(0);
    if constexpr (VARF) {
      bk[0] = group_lane<1>(a1);
      bk[1] = group_lane<2>(a1);
      bk[2] = group_lane<3>(a1);
      bkz = group_lane<2>(a2);
      bb = group_lane<3>(a2);
      if (A.D && gf != T(0) && varf_live) bDb = group_quadratic(k, A.D + A.loff[c], m);
    }
    const T l3 = lt * lt * lt;
    // d_points
    for (int d = 0; d < 3; ++d) {
      T r = s * (f * y[d] - Hy[d] / (lt * lt)) + gv * dxv[d];
      if (mean_live) r += s * gm * w[d] / (f * u);
      if (varf_live) r += gf * T(2) * bk[d] / (lt * lt);
      out_dx[d] = r;
    }
    // weight cotangent . xi (through the fit)
    T aXl = s * (y[0] * Eld[0] + y[1] * Eld[1] + y[2] * Eld[2]);
    T aXs = s * (y[0] * Esd[0] + y[1] * Esd[1] + y[2] * Esd[2]);
    if (mean_live) {
      const T cm = -s * gm * lt * lt / (u * f);
      aXl += cm * El;
      aXs += cm * Es;
    }
    T dl = 0, ds = 0;
    if (mean_live) dl += s * gm * (u2 - Za / f) / (lt * u);
    dl += s * (y[0] * Wz[0] + y[1] * Wz[1] + y[2] * Wz[2]) / l3;
    if (A.alpha_tied) dl += gv * dVa * (-T(2) * A.alpha / lt);
    if (varf_live) dl += gf * (-T(2) * bkz / l3 + bDb);
    dl -= aXl;
    if (A.uniform_noise) {
      ds += gv * C2;
      if (varf_live) ds += gf * bb;
      ds -= aXs;
    }
    out_th[0] = (double)dl;
    out_th[1] = (double)ds;
  }
  if (active && g == 0) {
    for (int d = 0; d < 3; ++d) A.d_points[3 * q + d] = out_dx[d];
    store_theta(A, q, out_th);
  }
}

// Eight steps of a compensated sum per lane over a row of the exchanged terms
__device__ __forceinline__ void group_cadd(const float* terms, int r, CAcc& acc) {
  const float* x = static_cast<const float*>(
      __builtin_assume_aligned(terms + r * GT_STRIDE + (threadIdx.x & 63) / GL * GL, 16));
  float v[GL];
#pragma unroll
  for (int s = 0; s < GL; ++s) v[s] = x[s];
#pragma unroll
  for (int s = 0; s < GL; ++s) acc.add(v[s]);
}

// vjp_f32 (RBF without a var_f cotangent) and vjp_matern_f32: FP32 models, with the
// differences as float pairs and compensated sums where the terms cancel
template <bool MAT, bool VARF>
__global__ void __launch_bounds__(64) bwd_group_ff_kernel(BwdArgs<float> A, const int* perm) {
  static_assert(MAT || !VARF, "the RBF's var_f cotangent runs in bwd_group_kernel");
  // rows 0..15 compensated sums, 16.. the factors of the plain ones
  __shared__ BwdGroupLds<float, 28, VARF> S;
  const int lane = threadIdx.x & 63, g = lane & (GL - 1);
  const long sq = A.first + xcd_block(gridDim.x) * GQ + lane / GL;
  const bool active = sq < A.Q;
  const long q = active ? (perm ? (long)perm[sq] : sq) : 0;
  int c = active ? A.argmin[q] : -1;
  if (c >= A.n_cells) c = -1;
  float gm = 0.f, gv = 0.f;
  if (active) mean_var_cotangents(A, q, gm, gv);
  float out_dx[3] = {0.f, 0.f, 0.f};
  double out_th[2] = {0.0, 0.0};
  if (c >= 0) {   // uniform over each group
    const float lt = A.ell, al = A.alpha, two_l2 = A.two_l2;
    const float ca = 1.4426950408889634f * al;
    const float mc = A.mc_ff[0];
    const ff mclf{A.mcl_ff[0], A.mcl_ff[1]}, c2f{A.c2_ff[0], A.c2_ff[1]};
    const float s = A.sign ? (float)A.sign[q] : 1.f;
    float gg[3] = {0.f, 0.f, 0.f};
    if (A.d_grad)
      for (int d = 0; d < 3; ++d) gg[d] = A.d_grad[3 * q + d];
    const float gf = VARF && A.d_var_f ? A.d_var_f[q] : 0.f;
    const int b = A.offsets[c], m = A.offsets[c + 1] - b;
    const float* Lc = A.L + A.loff[c];
    const float4* __restrict__ P4 = reinterpret_cast<const float4*>(A.ps);
    const float4* __restrict__ PL = reinterpret_cast<const float4*>(A.plo);
    const float4* __restrict__ X4 = reinterpret_cast<const float4*>(A.xi);
    const ff lx = ff_two_sum(A.pts[3 * q], -(float)A.centre64[3L * c]);
    const ff ly = ff_two_sum(A.pts[3 * q + 1], -(float)A.centre64[3L * c + 1]);
    const ff lz = ff_two_sum(A.pts[3 * q + 2], -(float)A.centre64[3L * c + 2]);
    float* row = S.t + lane;
    float* k = S.k + (VARF ? lane / GL * GK_STRIDE : 0);
    auto put = [&](int r, float v) { row[r * GT_STRIDE] = v; };
    auto unpack = [&](float4 h, float4 lo, float di[3], ff& z2, float& pa) {
      const ff dx = ff_sub_lean(lx.hi, lx.lo, h.x, lo.x);
      const ff dy = ff_sub_lean(ly.hi, ly.lo, h.y, lo.y);
      const ff dz = ff_sub_lean(lz.hi, lz.lo, h.z, lo.z);
      di[0] = dx.hi;
      di[1] = dy.hi;
      di[2] = dz.hi;
      z2 = ff_norm2_lean(dx, dy, dz);
      pa = h.w + lo.w;
    };
    // f(i, sample's high and low parts) for the lane's sample i of each eight, the next
    // ones' loads in flight (i past the last repeats it)
    auto each = [&](auto&& f) {
      float4 h = P4[b + min(g, m - 1)], lo = PL[b + min(g, m - 1)];
      for (int i0 = 0; i0 < m; i0 += GL) {
        const float4 ch = h, cl = lo;
        const int j = b + min(i0 + GL + g, m - 1);
        h = P4[j];
        lo = PL[j];
        f(i0 + g, ch, cl);
      }
    };
    // 2^-t for a float-pair t >= 0
    auto exp2n = [&](ff t) {
      const float n = floorf(t.hi);
      const float e = __builtin_amdgcn_exp2f(n - t.hi) * (1.f - 0.6931471805599453f * t.lo);
      return ldexpf(e, -(int)n);
    };
    ff d2f{INFINITY, 0.f};
    each([&](int, float4 h, float4 lo) {
      float di[3], pa;
      ff z2;
      unpack(h, lo, di, z2, pa);
      if (z2.hi < d2f.hi || (z2.hi == d2f.hi && z2.lo < d2f.lo)) d2f = z2;
    });
    auto fmin2 = [&](float oh, float ol) {
      if (oh < d2f.hi || (oh == d2f.hi && ol < d2f.lo)) d2f = ff{oh, ol};
    };
    fmin2(dpp<DPP_XOR1>(d2f.hi), dpp<DPP_XOR1>(d2f.lo));
    fmin2(dpp<DPP_XOR2>(d2f.hi), dpp<DPP_XOR2>(d2f.lo));
    fmin2(dpp<DPP_MIRROR8>(d2f.hi), dpp<DPP_MIRROR8>(d2f.lo));
    const float d2 = d2f.hi + d2f.lo;
    const ff zminf = MAT ? ff_sqrt(d2f) : ff{0.f, 0.f};
    const float zmin = MAT ? zminf.hi + zminf.lo : sqrtf(d2);
    // the terms of one sample: e (scaled kernel factor), z, t = z - zmin, and for the
    // Matern kernel z as a float pair
    auto sample = [&](float4 h, float4 lo, bool in, float di[3], float& pa, float& z2, float& z,
                      float& t, float& e, ff& zf) {
      ff z2f;
      unpack(h, lo, di, z2f, pa);
      z2 = z2f.hi + z2f.lo;
      if constexpr (MAT) {
        zf = ff_sqrt(z2f);
        z = zf.hi + zf.lo;
        const ff tf = ff_sub_lean(zf.hi, zf.lo, zminf.hi, zminf.lo);
        t = tf.hi + tf.lo;
        e = in ? exp2n(ff_mul(tf, mclf)) : 0.f;
      } else {
        z = sqrtf(z2);
        t = z - zmin;
        e = in ? exp2n(ff_mul(ff_sub_lean(z2f.hi, z2f.lo, d2f.hi, d2f.lo), c2f)) : 0.f;
      }
    };
    // pass A: f', w' (3), Z and (Matern) sum a e compensated; softmin moments
    put(16, 1.f);
    CAcc ca0;
    float acc = 0.f;
    put(5, 0.f);
    put(6, 0.f);
    put(7, 0.f);
    each([&](int i, float4 ph, float4 pl) {
      const bool in = i < m;
      float di[3], pa, z2, z, t, e;
      ff zf;
      sample(ph, pl, in, di, pa, z2, z, t, e, zf);
      const float ae = pa * e;
      put(0, MAT ? ae * fmaf(mc, z, 1.f) : ae);
      put(1, ae * di[0]);
      put(2, ae * di[1]);
      put(3, ae * di[2]);
      put(4, ae * z2);
      if constexpr (MAT) put(5, ae);
      const float sm = in ? __builtin_amdgcn_exp2f(-ca * t) : 0.f;
      put(17, sm);
      put(18, t);
      put(19, sm * t);
      if constexpr (VARF)
        if (in) k[i] = fmaf(mc, z, 1.f) * exp2n(ff_mul(zf, mclf));
      wave_lds_sync();
      group_cadd(S.t, g, ca0);
      group_fma(S.t, lane_entry(lanes8(16, 17, 19, 16, 16, 16, 16, 16)),
                lane_entry(lanes8(17, 18, 18, 17, 17, 17, 17, 17)), acc);
      wave_lds_sync();
    });
    const float sum0 = ca0.val();
    const float fv = group_lane<0>(sum0);
    const float wv[3] = {group_lane<1>(sum0), group_lane<2>(sum0), group_lane<3>(sum0)};
    const float Za = group_lane<4>(sum0), fev = group_lane<5>(sum0);
    const float Ss = group_lane<0>(acc), M1 = group_lane<1>(acc), M2 = group_lane<2>(acc);
    float vv = 0.f;
    if constexpr (VARF) {
      vv = group_forward_subst(k, Lc, m);
      group_backward_subst(k, Lc, m);
    }
    float u2 = 0.f, u;
    bool mean_live;
    if constexpr (MAT) {
      u = fv > 0.f ? zmin - logf(fv) / mc : -1.f;
      mean_live = u > 0.f;
    } else {
      u2 = fv > 0.f ? d2 - two_l2 * logf(fv) : -1.f;
      mean_live = u2 > 0.f;
      u = mean_live ? sqrtf(u2) : 0.f;
    }
    const float wn = sqrtf(wv[0] * wv[0] + wv[1] * wv[1] + wv[2] * wv[2]);
    float y[3] = {0.f, 0.f, 0.f};
    if (wn > 0.f) {
      const float gw = (gg[0] * wv[0] + gg[1] * wv[1] + gg[2] * wv[2]) / wn;
      for (int d = 0; d < 3; ++d) y[d] = (gg[d] - gw * wv[d] / wn) / wn;
    }
    const bool varf_live = VARF && (1.f - vv) > 0.f;
    const float iS = 1.f / Ss;
    const float m1 = M1 * iS;
    const float h = zmin + m1;
    const float Vz = M2 * iS - m1 * m1;
    // pass B: Hy (3), Wz (3), El, Es | Eld (3), Esd (3) compensated; plain: V, P, C2, dVa
    // and (RBF) the point derivative's parts.  d var / d z_j = 2 alpha (-sigma_j^2 c_j (c_j +
    // s_j) + s_j V + c_j P) needs V and P of the same pass, so its parts stay apart (Q1, Q2, Q3)
    // for the RBF kernel; for the Matern kernel they are added per sample in a pass of their own,
    // which keeps the digits that cancel (a variance's gradient alone over the uneven room's cells
    // of up to 128 samples: 7.4e-7 off FP64, 9.5e-7 with the parts apart).
    CAcc cb0, cb1;
    float a0 = 0.f, a1 = 0.f;
    put(14, 0.f);
    put(15, 0.f);
    put(27, 0.f);
    float svn = A.sv[b + min(g, m - 1)];   // the next sample's variance and adjoint vectors,
    float4 xqn = X4[b + min(g, m - 1)];    // on their way while this one's are used
    each([&](int i, float4 ph, float4 pl) {
      const bool in = i < m;
      const float svc = svn;
      const float4 xq = xqn;
      svn = A.sv[b + min(i + GL, m - 1)];
      xqn = X4[b + min(i + GL, m - 1)];
      float di[3], pa, z2, z, t, e;
      ff zf;
      sample(ph, pl, in, di, pa, z2, z, t, e, zf);
      const float svj = in ? svc : 0.f;   // not 0 times an infinite variance
      const float xl = xq.x + xq.z, xs = xq.y + xq.w;
      const float ae = pa * e;
      const float si = in ? __builtin_amdgcn_exp2f(-ca * t) * iS : 0.f;
      const float Bi = al * (h - z) + 1.f;
      const float ci = si * Bi;
      const float rz = z > 0.f ? 1.f / z : 0.f;
      const float dy = di[0] * y[0] + di[1] * y[1] + di[2] * y[2];
      const float kp = MAT ? fmaf(mc, z, 1.f) * e : e;
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        put(d, MAT ? ae * dy * di[d] * rz : ae * dy * di[d]);
        put(3 + d, MAT ? ae * z * di[d] : ae * z2 * di[d]);
        put(8 + d, e * xl * di[d]);
        put(11 + d, e * xs * di[d]);
        if constexpr (!MAT) put(24 + d, di[d]);
      }
      put(6, kp * xl);
      put(7, kp * xs);
      put(16, svj * ci);
      put(17, ci);
      put(18, si);
      put(19, 2.f * svj * ci);
      put(20, si * (h - z) * (Bi + 1.f) - al * si * Vz);
      if constexpr (!MAT) {
        put(21, var_part1_f32(svj, ci, si, rz));
        put(22, si * rz);
        put(23, ci * rz);
      }
      wave_lds_sync();
      group_cadd(S.t, g, cb0);
      group_cadd(S.t, 8 + g, cb1);
      if constexpr (MAT) {
        // V, P, C2, dVa
        group_fma(S.t, lane_entry(lanes8(16, 16, 17, 19, 27, 27, 27, 27)),
                  lane_entry(lanes8(17, 18, 17, 20, 27, 27, 27, 27)), a0);
      } else {
        // V, P, C2, dVa, Q1 (3), Q2 | Q2 (2), Q3 (3)
        group_fma(S.t, lane_entry(lanes8(16, 16, 17, 19, 21, 21, 21, 22)),
                  lane_entry(lanes8(17, 18, 17, 20, 24, 25, 26, 24)), a0);
        group_fma(S.t, lane_entry(lanes8(22, 22, 23, 23, 23, 27, 27, 27)),
                  lane_entry(lanes8(25, 26, 24, 25, 26, 27, 27, 27)), a1);
      }
      wave_lds_sync();
    });
    const float s0 = cb0.val(), s1 = cb1.val();
    const float Hy[3] = {group_lane<0>(s0), group_lane<1>(s0), group_lane<2>(s0)};
    const float Wz[3] = {group_lane<3>(s0), group_lane<4>(s0), group_lane<5>(s0)};
    const float El = group_lane<6>(s0), Es = group_lane<7>(s0);
    const float Eld[3] = {group_lane<0>(s1), group_lane<1>(s1), group_lane<2>(s1)};
    const float Esd[3] = {group_lane<3>(s1), group_lane<4>(s1), group_lane<5>(s1)};
    const float V = group_lane<0>(a0), Pp = group_lane<1>(a0), C2 = group_lane<2>(a0),
                dVa = group_lane<3>(a0);
    const float Q1[3] = {group_lane<4>(a0), group_lane<5>(a0), group_lane<6>(a0)};
    const float Q2[3] = {group_lane<7>(a0), group_lane<0>(a1), group_lane<1>(a1)};
    const float Q3[3] = {group_lane<2>(a1), group_lane<3>(a1), group_lane<4>(a1)};
    // d var / dx; without a variance cotangent only where it is not finite (0 times it is NaN)
    float dxv[3] = {0.f, 0.f, 0.f};
    if constexpr (MAT) {
      if (gv != 0.f || !(V < INFINITY)) {
        acc = 0.f;
        each([&](int i, float4 ph, float4 pl) {
          const bool in = i < m;
          float di[3], pa, z2, z, t, e;
          ff zf;
          sample(ph, pl, in, di, pa, z2, z, t, e, zf);
          const float svj = in ? A.sv[b + i] : 0.f;
          const float si = in ? __builtin_amdgcn_exp2f(-ca * t) * iS : 0.f;
          const float ci = si * (al * (h - z) + 1.f);
          const float dvdz = in ? 2.f * al * (-svj * ci * (ci + si) + si * V + ci * Pp) : 0.f;
#pragma unroll
          for (int d = 0; d < 3; ++d) put(d, dvdz * di[d]);
          put(3, z > 0.f ? 1.f / z : 0.f);
          wave_lds_sync();
          group_fma(S.t, lane_entry(lanes8(0, 1, 2, 27, 27, 27, 27, 27)),
                    lane_entry(lanes8(3, 3, 3, 27, 27, 27, 27, 27)), acc);
          wave_lds_sync();
        });
        dxv[0] = group_lane<0>(acc);
        dxv[1] = group_lane<1>(acc);
        dxv[2] = group_lane<2>(acc);
      }
    }
    // the GP variance's sums: bk (3), bkz, bb
    float bk[3] = {0.f, 0.f, 0.f}, bkz = 0.f, bb = 0.f, bDb = 0.f;
    if constexpr (VARF) {
      acc = 0.f;
      each([&](int i, float4 ph, float4 pl) {
        const bool in = i < m;
        float di[3], pa, z2, z, t, e;
        ff zf;
        sample(ph, pl, in, di, pa, z2, z, t, e, zf);
        const float vi = in ? k[i] : 0.f;
        put(0, vi * exp2n(ff_mul(zf, mclf)));
        put(1, di[0]);
        put(2, di[1]);
        put(3, di[2]);
        put(4, z2);
        put(5, vi);
        wave_lds_sync();
        group_fma(S.t, lane_entry(lanes8(0, 0, 0, 0, 5, 27, 27, 27)),
                  lane_entry(lanes8(1, 2, 3, 4, 5, 27, 27, 27)), acc);
        wave_lds_sync();
      });
      bk[0] = group_lane<0>(acc);
      bk[1] = group_lane<1>(acc);
      bk[2] = group_lane<2>(acc);
      bkz = group_lane<3>(acc);
      bb = group_lane<4>(acc);
      if (A.D && gf != 0.f && varf_live) bDb = group_quadratic(k, A.D + A.loff[c], m);
    }
    const float l3 = lt * lt * lt;
    for (int d = 0; d < 3; ++d) {
      if constexpr (MAT) {
        float r = s * (fev * y[d] - mc * Hy[d]) + gv * dxv[d];
        if (mean_live) r += s * gm * mc * wv[d] / fv;
        if (varf_live) r += gf * 2.f * mc * mc * bk[d];
        out_dx[d] = r;
      } else {
        out_dx[d] = point_grad_f32(A, s, gm, gv, fv, u, mean_live, V, Pp, y[d], Hy[d], wv[d], Q1[d],
                                   Q2[d], Q3[d]);
      }
    }
    float aXl = s * (y[0] * Eld[0] + y[1] * Eld[1] + y[2] * Eld[2]);
    float aXs = s * (y[0] * Esd[0] + y[1] * Esd[1] + y[2] * Esd[2]);
    if (mean_live) {
      const float cm = MAT ? -s * gm / (mc * fv) : -s * gm * lt * lt / (u * fv);
      aXl += cm * El;
      aXs += cm * Es;
    }
    float dl = 0.f, ds = 0.f;
    if constexpr (MAT) {
      if (mean_live) dl += s * gm * (u - mc * Za / fv) / lt;
      dl += s * (mc / lt) * (y[0] * Wz[0] + y[1] * Wz[1] + y[2] * Wz[2]);
    } else {
      if (mean_live) dl += s * gm * (u2 - Za / fv) / (lt * u);
      dl += s * (y[0] * Wz[0] + y[1] * Wz[1] + y[2] * Wz[2]) / l3;
    }
    if (A.alpha_tied) dl += gv * dVa * (-2.f * al / lt);
    if (varf_live) dl += gf * (-2.f * mc * mc * bkz / lt + bDb);
    dl -= aXl;
    if (A.uniform_noise) {
      if constexpr (MAT) {
        ds += gv * C2;
        if (varf_live) ds += gf * bb;
        ds -= aXs;
      } else {
        ds += gv * C2 - aXs;
      }
    }
    out_th[0] = (double)dl;
    out_th[1] = (double)ds;
  }
  if (active && g == 0) {
    for (int d = 0; d < 3; ++d) A.d_points[3 * q + d] = out_dx[d];
    store_theta(A, q, out_th);
  }
}

}  // namespace

void launch_backward_group(const ksdf_model* m, BwdArgs<float> A, bool varf, const int* perm,
                           hipStream_t s) {
  group_launches(A.Q, [&](long first, unsigned n) {
    const dim3 grid(n), block(64);
    A.first = first;
    if (m->kernel == KSDF_KERNEL_MATERN32) {
      if (varf) hipLaunchKernelGGL((bwd_group_ff_kernel<true, true>), grid, block, 0, s, A, perm);
      else hipLaunchKernelGGL((bwd_group_ff_kernel<true, false>), grid, block, 0, s, A, perm);
    } else {
      if (varf) hipLaunchKernelGGL((bwd_group_kernel<float, true>), grid, block, 0, s, A, perm);
      else hipLaunchKernelGGL((bwd_group_ff_kernel<false, false>), grid, block, 0, s, A, perm);
    }
  });
}

void launch_backward_group(const ksdf_model* m, BwdArgs<double> A, bool varf, const int* perm,
                           hipStream_t s) {
  (void)m;
  group_launches(A.Q, [&](long first, unsigned n) {
    const dim3 grid(n), block(64);
    A.first = first;
    if (varf) hipLaunchKernelGGL((bwd_group_kernel<double, true>), grid, block, 0, s, A, perm);
    else hipLaunchKernelGGL((bwd_group_kernel<double, false>), grid, block, 0, s, A, perm);
  });
}

}  // namespace ksdf
