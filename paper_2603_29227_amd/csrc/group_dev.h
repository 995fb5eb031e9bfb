// Eight lanes per query: the helpers shared by the group kernels of the query and the
// backward (query_group.hip, query.hip, backward_group.hip).  The lanes of a query work on
// eight samples (or eight factor rows) of its cell at a time; terms and vectors pass through
// LDS, and every running sum is carried by one lane in sample order, so that the results are
// those of one thread per query bit for bit.
#pragma once

#include "ksdf_internal.h"
#include "wave_ops.h"

namespace ksdf {
namespace {

constexpr int GL = 8;          // lanes per query
constexpr int GQ = 64 / GL;    // queries per wave
// queries of one launch: a launch holds fewer than 2^32 threads, so larger calls take several
constexpr long GROUP_LAUNCH_MAX = 1L << 28;
// f(first query, workgroups) for each launch of Q queries, 64 threads a workgroup
template <class F>
inline void group_launches(long Q, F&& f) {
  for (long first = 0; first < Q; first += GROUP_LAUNCH_MAX) {
    const long n = Q - first < GROUP_LAUNCH_MAX ? Q - first : GROUP_LAUNCH_MAX;
    f(first, (unsigned)((n + GQ - 1) / GQ));
  }
}
// elements between the queries' vectors and between the rows of exchanged terms in LDS
// (padded, so that the eight queries of a wave fall in different banks)
constexpr int GK_STRIDE = KSDF_MAX_M + 4;
constexpr int GT_STRIDE = 72;

// lane S of each eight-lane group, to the whole group
template <int S>
__device__ __forceinline__ int group_lane(int v) {
  return __builtin_amdgcn_ds_swizzle(v, (S << 5) | 0x18);
}
template <int S>
__device__ __forceinline__ float group_lane(float v) {
  return __builtin_bit_cast(float, group_lane<S>(__builtin_bit_cast(int, v)));
}
template <int S>
__device__ __forceinline__ double group_lane(double v) {
  const long long u = __builtin_bit_cast(long long, v);
  const unsigned lo = (unsigned)group_lane<S>((int)(u & 0xffffffffLL));
  const int hi = group_lane<S>((int)(u >> 32));
  return __builtin_bit_cast(double, ((long long)hi << 32) | lo);
}
// the neighbour of a three-step reduction over each group: lane ^ 1, lane ^ 2, 7 - lane
template <int CTRL>
__device__ __forceinline__ int dpp(int v) {
  return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __builtin_bit_cast(float, dpp<CTRL>(__builtin_bit_cast(int, v)));
}
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  const long long u = __builtin_bit_cast(long long, v);
  const unsigned lo = (unsigned)dpp<CTRL>((int)(u & 0xffffffffLL));
  const int hi = dpp<CTRL>((int)(u >> 32));
  return __builtin_bit_cast(double, ((long long)hi << 32) | lo);
}
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_MIRROR8 = 0x141;

// group_lane without LDS, for broadcasts on a chain (two moves and a select against the LDS
// pipe's latency)
template <int S, class T>
__device__ __forceinline__ T group_lane_quick(T v) {
  constexpr int s = S & 3;
  const T x = dpp<s | s << 2 | s << 4 | s << 6>(v);   // each four lanes' own lane s
  const T y = dpp<DPP_MIRROR8>(x);
  return ((threadIdx.x & 4) == 0) == (S < 4) ? x : y;
}

// the greatest value of each group
template <class T>
__device__ __forceinline__ T group_max(T v) {
  v = max(v, dpp<DPP_XOR1>(v));
  v = max(v, dpp<DPP_XOR2>(v));
  return max(v, dpp<DPP_MIRROR8>(v));
}
// whether v holds on all lanes of the group (which must be active together)
__device__ __forceinline__ bool group_all(bool v) {
  return ((__ballot(v) >> (threadIdx.x & 56)) & 0xff) == 0xff;
}

// the smallest (distance, id) pair of each group
template <class T>
__device__ __forceinline__ void group_min(T& d, int& id) {
  auto step = [&](T od, int oi) {
    if (od < d || (od == d && oi < id)) {
      d = od;
      id = oi;
    }
  };
  step(dpp<DPP_XOR1>(d), dpp<DPP_XOR1>(id));
  step(dpp<DPP_XOR2>(d), dpp<DPP_XOR2>(id));
  step(dpp<DPP_MIRROR8>(d), dpp<DPP_MIRROR8>(id));
}

// eight 5-bit entries, one per lane of a group (the rows that the lane's sum takes)
constexpr unsigned long long lanes8(int a, int b, int c, int d, int e, int f, int g, int h) {
  const int v[8] = {a, b, c, d, e, f, g, h};
  unsigned long long t = 0;
  for (int i = 0; i < 8; ++i) t |= (unsigned long long)v[i] << (5 * i);
  return t;
}
__device__ __forceinline__ int lane_entry(unsigned long long t) {
  return (int)(t >> (5 * (threadIdx.x & (GL - 1)))) & 31;
}

// Eight steps of a running sum per lane: acc += x y over the group's eight samples in order,
// x and y the rows xr and yr of the exchanged terms
template <class T>
__device__ __forceinline__ void group_fma(const T* terms, int xr, int yr, T& acc) {
  const int q8 = (threadIdx.x & 63) / GL * GL;
  const T* x = static_cast<const T*>(__builtin_assume_aligned(terms + xr * GT_STRIDE + q8, 16));
  const T* y = static_cast<const T*>(__builtin_assume_aligned(terms + yr * GT_STRIDE + q8, 16));
  T xv[GL], yv[GL];
#pragma unroll
  for (int s = 0; s < GL; ++s) {
    xv[s] = x[s];
    yv[s] = y[s];
  }
#pragma unroll
  for (int s = 0; s < GL; ++s) acc = fma(xv[s], yv[s], acc);
}

// eight consecutive factor entries, 16 bytes a load (rows start at any multiple of a value)
__device__ __forceinline__ void load_row8(const float* p, float (&l)[GL]) {
  typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));
  const f4 a = *reinterpret_cast<const f4*>(p), b = *reinterpret_cast<const f4*>(p + 4);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    l[e] = a[e];
    l[4 + e] = b[e];
  }
}
__device__ __forceinline__ void load_row8(const double* p, double (&l)[GL]) {
  typedef double d2 __attribute__((ext_vector_type(2), aligned(8)));
#pragma unroll
  for (int e = 0; e < GL; e += 2) {
    const d2 a = *reinterpret_cast<const d2*>(p + e);
    l[e] = a[0];
    l[e + 1] = a[1];
  }
}

// L^{-1} k for each group's cell (m samples, packed factor Lc with reciprocal diagonal), in
// place in the group's vector k in LDS; returns |L^{-1} k|^2.  Blocks of eight rows, one per
// lane: the columns before the block from LDS, then the block's own triangle through the
// group.  Every entry subtracts its columns in order, as a sequential substitution does.
// The loads of the next eight columns, and those of the next block's start, are in flight
// during the current ones' steps.
template <class T>
__device__ __forceinline__ T group_forward_subst(T* k, const T* __restrict__ Lc, int m) {
  const int g = threadIdx.x & (GL - 1);
  T vv = T(0);
  T ld[GL], l[GL];   // the row's entries in the block (its diagonal the reciprocal); columns
  // lanes past the last row read it too (their results are not used)
  auto row_of_block = [&](int b0) { return min(b0 + g, m - 1); };
  auto load_block = [&](int b0) {
    const int ir = row_of_block(b0);
    const T* Li = Lc + ir * (ir + 1) / 2;
#pragma unroll
    for (int e = 0; e < GL; ++e) ld[e] = Li[min(b0 + e, ir)];
    if (b0 > 0) load_row8(Li, l);
  };
  if (m > 0) load_block(0);
  for (int b0 = 0; b0 < m; b0 += GL) {
    const int i = b0 + g, ir = row_of_block(b0);
    const T* Li = Lc + ir * (ir + 1) / 2;
    T t = k[ir];
    for (int j = 0; j < b0; j += GL) {
      const T* kj = static_cast<const T*>(__builtin_assume_aligned(k + j, 16));
      T lc[GL], v[GL];
#pragma unroll
      for (int e = 0; e < GL; ++e) lc[e] = l[e];
      load_row8(Li + min(j + GL, b0 - GL), l);   // b0 - 1 < ir: within the row
#pragma unroll
      for (int e = 0; e < GL; ++e) v[e] = kj[e];
#pragma unroll
      for (int e = 0; e < GL; ++e) t = fma(-lc[e], v[e], t);
    }
    T rd = T(0), x = T(0), lb[GL];
#pragma unroll
    for (int e = 0; e < GL; ++e) {
      lb[e] = ld[e];
      if (e == g) rd = ld[e];
    }
    if (b0 + GL < m) load_block(b0 + GL);
    static_for<0, GL>([&](auto E) {
      constexpr int e = E;
      const T xe = group_lane_quick<e>(t * rd);   // row b0 + e is final at this step
      if (g == e) x = xe;
      if (g > e) t = fma(-lb[e], xe, t);
      if (b0 + e < m) vv = fma(xe, xe, vv);
    });
    if (i < m) k[i] = x;
    wave_lds_sync();
  }
  return vv;
}

// L^{-T} v in place, the last block first: the rows after the block in descending order,
// then the block's own triangle
template <class T>
__device__ __forceinline__ void group_backward_subst(T* k, const T* __restrict__ Lc, int m) {
  const int g = threadIdx.x & (GL - 1);
  for (int b0 = (m - 1) / GL * GL; b0 >= 0; b0 -= GL) {
    const int i = b0 + g;
    const bool row = i < m;
    T t = row ? k[i] : T(0);
    T ld[GL];   // column i of the block's rows
#pragma unroll
    for (int e = 0; e < GL; ++e)
      ld[e] = row && e >= g && b0 + e < m ? Lc[(b0 + e) * (b0 + e + 1) / 2 + i] : T(0);
    for (int r0 = (m - 1) / GL * GL; r0 > b0; r0 -= GL) {
      T l[GL], v[GL];
#pragma unroll
      for (int e = 0; e < GL; ++e) {
        const int r = r0 + e;
        l[e] = r < m ? Lc[r * (r + 1) / 2 + i] : T(0);   // i < r0 <= r
        v[e] = k[r < m ? r : 0];
      }
#pragma unroll
      for (int e = GL - 1; e >= 0; --e)
        if (r0 + e < m) t = fma(-l[e], v[e], t);
    }
    T rd = T(0), x = T(0);
#pragma unroll
    for (int e = 0; e < GL; ++e)
      if (e == g) rd = ld[e];
    static_for<0, GL>([&](auto E) {
      constexpr int e = GL - 1 - E;
      const T xe = group_lane_quick<e>(t * rd);
      if (g == e) x = xe;
      if (g < e && b0 + e < m) t = fma(-ld[e], xe, t);
    });
    if (row) k[i] = x;
    wave_lds_sync();
  }
}

}  // namespace
}  // namespace ksdf
