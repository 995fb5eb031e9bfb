// Arguments and small device helpers of the backward kernels (backward.hip,
// backward_group.hip).
#pragma once

#include "ff.h"
#include "ksdf_internal.h"
#include "wave_ops.h"

namespace ksdf {

// (shared by the translation units that launch them, hence outside the file-local namespace)
template <class T>
struct BwdArgs {
  const T* __restrict__ pts;
  long Q;
  long first;              // eight lanes per query: the launch's first query
  const int8_t* sign;
  const int* argmin;
  const T* d_mean;
  const T* d_grad;
  const T* d_var;
  const T* d_var_f;
  T* d_points;
  double* part;            // [Q,2] per-query (dL/dl, dL/dsigma^2)
  int n_cells;
  const int* offsets;
  const long* loff;
  const T* ps;             // [nnz,4] (px,py,pz,a) cell-local
  const float* plo;        // FP32 store: float-float low parts of ps
  const T* sv;
  const T* L;              // packed rows, reciprocal diagonal
  const T* xi;             // [nnz,2] (FP64) or [nnz+pad,4] float-float (FP32)
  const T* D;              // packed dA/dl or null
  const double* centre64;
  T ell, two_l2, alpha;
  float c2_ff[2];          // log2(e) / (2 l^2) as a float pair (FP32 models)
  float mc_ff[2];          // Matern c = sqrt(3) / l and c log2(e) as float pairs
  float mcl_ff[2];
  int alpha_tied;
  int uniform_noise;
  // the softplus margin cost (ksdf_cost_backward): when c_mean is set, the mean and
  // var cotangents are formed from the forward outputs instead of read
  const T* c_mean;
  const T* c_var;
  T c_margin, c_kvar;
  T* c_cost;               // per-query cost, or null
};

namespace {

// Cotangents of mean and var for query q: the given ones, or those of the cost
// softplus(t), t = margin - mean + kvar sqrt(var): d/dmean = -sigmoid(t) and
// d/dvar = kvar sigmoid(t) / (2 sqrt(var)), with the stable forms of sigmoid and
// softplus (max(t, 0) + log1p(e^-|t|)); var is clamped below at 1e-30.
template <class T>
__device__ __forceinline__ void mean_var_cotangents(const BwdArgs<T>& A, long q, T& gm, T& gv) {
  gm = A.d_mean ? A.d_mean[q] : T(0);
  gv = A.d_var ? A.d_var[q] : T(0);
  if (A.c_mean) {
    const T sd = sqrt(fmax(A.c_var[q], T(1e-30)));
    const T t = A.c_margin - A.c_mean[q] + A.c_kvar * sd;
    const T e = exp(-fabs(t));
    const T sg = t >= T(0) ? T(1) / (T(1) + e) : e / (T(1) + e);
    gm = -sg;
    gv = A.c_kvar * sg / (T(2) * sd);
    if (A.c_cost) A.c_cost[q] = fmax(t, T(0)) + log1p(e);
  }
}

// the per-query hyperparameter terms: FP64 models keep doubles; FP32 models keep
// float pairs (dl, ds), summed afterwards in float-float
template <class T>
__device__ __forceinline__ void store_theta(const BwdArgs<T>& A, long q, const double th[2]) {
  if constexpr (sizeof(T) == 8) {
    A.part[2 * q] = th[0];
    A.part[2 * q + 1] = th[1];
  } else {
    reinterpret_cast<float2*>(A.part)[q] = make_float2((float)th[0], (float)th[1]);
  }
}

// Compensated FP32 sum (TwoSum, Knuth): the running sum and the sum of its rounding
// errors, so that m terms carry about one rounding of the result instead of m.
struct CAcc {
  float s = 0.f, c = 0.f;
  __device__ __forceinline__ void add(float x) {
#pragma clang fp contract(off)
    const float t = s + x;
    const float bb = t - s;
    c += (s - (t - bb)) + (x - bb);
    s = t;
  }
  __device__ __forceinline__ float val() const { return s + c; }
};

// The first part of d var / d z_j over z_j, -sigma_j^2 c_j (c_j + s_j) / z_j, each operation
// rounded by itself (see point_grad_f32).
__device__ __forceinline__ float var_part1_f32(float sv, float ci, float si, float rz) {
#pragma clang fp contract(off)
  return -sv * ci * (ci + si) * rz;
}

// The point derivative of one component of an FP32 RBF query from its sums, every operation
// rounded by itself: the eight-lane and the per-thread kernels then agree bit for bit, so
// that a point's gradient does not depend on the batch it is in.
__device__ __forceinline__ float point_grad_f32(const BwdArgs<float>& A, float s, float gm, float gv,
                                                float f, float u, bool mean_live, float V, float P,
                                                float y, float Hy, float w, float Q1, float Q2,
                                                float Q3) {
#pragma clang fp contract(off)
  const float dxv = 2.f * A.alpha * (Q1 + V * Q2 + P * Q3);
  float r = s * (f * y - Hy / (A.ell * A.ell)) + gv * dxv;
  if (mean_live) r += s * gm * w / (f * u);
  return r;
}

}  // namespace

// eight lanes per query (backward_group.hip); perm null: the queries in the caller's order
void launch_backward_group(const ksdf_model* m, BwdArgs<float> A, bool varf, const int* perm,
                           hipStream_t s);
void launch_backward_group(const ksdf_model* m, BwdArgs<double> A, bool varf, const int* perm,
                           hipStream_t s);

}  // namespace ksdf
