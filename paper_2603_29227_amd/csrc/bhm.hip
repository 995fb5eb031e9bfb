// SDF sign from Bayesian-Hilbert-map weights (Sec. IV-A sign prediction, App. B).
//
// The occupancy log-odds of a local BHM is l(x) = mu^T phi(x) with features
// phi(x) = [k(x, h_1), ..., k(x, h_M), 1], k(x, h) = exp(-gamma |x - h|^2) over the
// hinge points h of the local map; the sign is +1 (free) where l(x) < tau and -1
// otherwise, and tau follows a moving average of the log-odds at hit points.
//
// Local maps sit on a lattice of boxes of edge B; each holds n_h^3 hinge points at
// the lattice points of its box (spacing B / (n_h - 1)) plus the bias feature.  A
// query uses the map of the box it lies in.  The RBF over a lattice separates by axis,
// k = exp(-gamma dx^2) exp(-gamma dy^2) exp(-gamma dz^2), so a query takes 3 n_h
// exponentials and n_h^3 multiply-adds instead of n_h^3 exponentials.  Double points
// are evaluated in FP64, float points in FP32 with a compensated outer sum (the
// decision l < tau is then the FP32 one).
#include <climits>
#include <cmath>

#include "ff.h"
#include "ksdf_internal.h"

namespace ksdf {
namespace {

constexpr int BT = 256;
constexpr int MAX_HINGES = 16;

struct BhmArgs {
  double origin[3];
  double box, inv_box;
  double spacing;
  int dims[3];
  int nh;
  double gamma;
  const int* box_bhm;
  const double* weights;
  // float pairs of the layout for the FP32 evaluation
  float origin_ff[3][2];
  float box_ff[2];
  float spacing_ff[2];
};

// The map box of a point: its lattice key and the flat box index (-1: outside the lattice).
template <class T>
__device__ __forceinline__ long bhm_flat(const BhmArgs& A, const T x3[3], long key[3]) {
  for (int d = 0; d < 3; ++d) {
    // x / B to the last bit from 1 / B (two corrections by the exact remainder: Markstein
    // 1990) where it is in range: the division itself takes three times the instructions.
    // (Edges so small that the remainder is not exact have a NaN for 1 / B: make_bhm_args.)
    const double x = (double)x3[d] - A.origin[d];
    double t = x * A.inv_box;
    const double t1 = fma(fma(-t, A.box, x), A.inv_box, t);
    const double t2 = fma(fma(-t1, A.box, x), A.inv_box, t1);
    if (fabs(t) < 1e9) key[d] = (int)floor(t2);   // converts in one instruction
    else key[d] = (long)floor(x / A.box);
  }
  bool in = true;
  for (int d = 0; d < 3; ++d) in = in && key[d] >= 0 && key[d] < A.dims[d];
  return in ? (key[0] * A.dims[1] + key[1]) * A.dims[2] + key[2] : -1;
}
// its map id (-1: none, or outside the lattice)
template <class T>
__device__ __forceinline__ int bhm_box(const BhmArgs& A, const T* pts, long q, long key[3]) {
  const T x3[3] = {pts[3 * q], pts[3 * q + 1], pts[3 * q + 2]};
  const long flat = bhm_flat(A, x3, key);
  return flat < 0 ? -1 : A.box_bhm[flat];
}

// Log-odds of a point in FP64 (double points): per-axis factors, then the separable sum.
__device__ double bhm_logodds64(const BhmArgs& A, const double* pts, long q, const long key[3],
                                const double* w) {
  const int nh = A.nh;
  double e[3][MAX_HINGES];
  for (int d = 0; d < 3; ++d) {
    const double lo = A.origin[d] + (double)key[d] * A.box;
    for (int i = 0; i < nh; ++i) {
      const double t = pts[3 * q + d] - (lo + (double)i * A.spacing);
      e[d][i] = exp(-A.gamma * t * t);
    }
  }
  const long m = (long)nh * nh * nh;
  double l = w[m];   // bias feature
  for (int i = 0; i < nh; ++i)
    for (int j = 0; j < nh; ++j) {
      const double eij = e[0][i] * e[1][j];
      const double* wr = w + ((long)i * nh + j) * nh;
      double acc = 0.0;
      for (int k = 0; k < nh; ++k) acc += wr[k] * e[2][k];
      l += eij * acc;
    }
  return l;
}

// The same for float points, in FP32: the offsets to the hinges from the exact
// difference of the point and the hinge coordinate (the hinge as a float pair), the
// factors from the FP32 exp, the inner sums over the last axis plain and the outer sum
// with TwoSum compensation.  The error is a few float roundings of sum |terms|; where
// |l - tau| is below that, the sign is the FP32 decision.
// The FP32 log-odds with the hinge count as a compile-time constant NH: every loop
// unrolls and the per-axis factors stay in registers.  The same operations in the same
// order as bhm_logodds32_any below.
// (w: the weights in rows of ROW, then the bias)
template <int NH, int ROW, class W>
__device__ __forceinline__ float bhm_logodds32_t(const BhmArgs& A, const float* pts, long q,
                                                 const long key[3], const W* w) {
  float e[3][NH];
  const float g = (float)A.gamma;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    // x - (box corner) as a float pair, the corner origin + key B from the layout's pairs
    const ff lo = ff_add(ff{A.origin_ff[d][0], A.origin_ff[d][1]},
                         ff_mul_f(ff{A.box_ff[0], A.box_ff[1]}, (float)key[d]));
    const ff t0 = ff_add(ff{pts[3 * q + d], 0.f}, ff_neg(lo));
#pragma unroll
    for (int i = 0; i < NH; ++i) {
      const float fi = (float)i;
      const float tt = fmaf(-fi, A.spacing_ff[0], t0.hi) + fmaf(-fi, A.spacing_ff[1], t0.lo);
      e[d][i] = expf(-g * tt * tt);
    }
  }
  constexpr int m = NH * NH * ROW;
  float s = (float)w[m], c = 0.f;   // bias feature; compensated outer sum
#pragma unroll
  for (int i = 0; i < NH; ++i)
#pragma unroll
    for (int j = 0; j < NH; ++j) {
      const float eij = e[0][i] * e[1][j];
      const W* wr = w + (i * NH + j) * ROW;
      float acc = 0.f;
#pragma unroll
      for (int k = 0; k < NH; ++k) acc = fmaf((float)wr[k], e[2][k], acc);
      const ff p = ff_two_sum(s, eij * acc);
      s = p.hi;
      c += p.lo;
    }
  return s + c;
}

// Any hinge count (read from the layout; the factor arrays live in private memory).
__device__ float bhm_logodds32_any(const BhmArgs& A, const float* pts, long q, const long key[3],
                                   const double* w) {
  const int nh = A.nh;
  float e[3][MAX_HINGES];
  const float g = (float)A.gamma;
  for (int d = 0; d < 3; ++d) {
    const ff lo = ff_add(ff{A.origin_ff[d][0], A.origin_ff[d][1]},
                         ff_mul_f(ff{A.box_ff[0], A.box_ff[1]}, (float)key[d]));
    const ff t0 = ff_add(ff{pts[3 * q + d], 0.f}, ff_neg(lo));
    for (int i = 0; i < nh; ++i) {
      const float fi = (float)i;
      const float tt = fmaf(-fi, A.spacing_ff[0], t0.hi) + fmaf(-fi, A.spacing_ff[1], t0.lo);
      e[d][i] = expf(-g * tt * tt);
    }
  }
  const int m = nh * nh * nh;
  float s = (float)w[m], c = 0.f;
  for (int i = 0; i < nh; ++i)
    for (int j = 0; j < nh; ++j) {
      const float eij = e[0][i] * e[1][j];
      const double* wr = w + (i * nh + j) * nh;
      float acc = 0.f;
      for (int k = 0; k < nh; ++k) acc = fmaf((float)wr[k], e[2][k], acc);
      const ff p = ff_two_sum(s, eij * acc);
      s = p.hi;
      c += p.lo;
    }
  return s + c;
}

// 7 hinges per axis (the indoor setting) in registers; other counts the general form
__device__ __forceinline__ float bhm_logodds32(const BhmArgs& A, const float* pts, long q,
                                               const long key[3], const double* w) {
  if (A.nh == 7) return bhm_logodds32_t<7, 7>(A, pts, q, key, w);
  return bhm_logodds32_any(A, pts, q, key, w);
}

// Signs of many points.  Most lie in no map's box: they are answered at once, and a block's
// others are gathered in LDS (in the points' order), so that whole waves evaluate maps or none do.  Float
// points and 7 hinges: the block's maps (a few: neighbouring points share them; found through a
// small hash table) are converted to FP32 into LDS once, in rows of 8, where every lane reads
// its own map's.  Maps beyond BHM_MAPS, other hinge counts and double points: every lane loads
// its map's weights.
// The kernel moves 21 bytes a point; the sorted form with FP64 divisions takes 590 us for the
// 256^3 grid, a fifth of whose points have a map, and whose bytes take 75; this one 383 us.
// BHM_MAPS: points on the surface meet up to 16 maps a block, a grid few, and the weights' LDS
// (1.6 KB a map) takes waves from the CU.  us for 4, 8, 12, 16, 24, 32 maps, 16,777,216 points:
//   boxes of 0.16 m   grid     351    322   315   325   332   447
//                     surface 10302  9947  8716  7413  7373  7471
//   boxes of 0.5 m    grid     526    338   343   357   417   566
//                     surface 6267   5606  4158  3483  3498  3727
constexpr int BS = 256;
constexpr int BHM_MAPS = 16;                 // maps of a block in LDS
constexpr int BHM_STRIDE = 7 * 7 * 8 + 8;    // floats per map: 49 rows of 8, the bias
constexpr int BHM_HASH = 64, BHM_PROBES = 4;
__device__ __forceinline__ int bhm_hash(int id, int p) {
  return ((int)((unsigned)id * 2654435761u >> 26) + p) % BHM_HASH;
}
constexpr int BHM_PT = 4;                    // points per thread of the gathered form
// The sorted form's chain is shorter, and fills the chip's gaps with few points; the gathered
// form does less per point while its front (map ids, gathers) is a good part of the work, or its
// maps are staged.  us, sorted / gathered, a grid over a room with boxes of 0.16 m, and points on
// the surface, all of them in a map:
//     points         7 hinges, float  3, float   3, double   5, float    5, double     7, double
//     2,197,000 grid    80 / 85       55 / 45    65 / 56    127 / 158   180 / 184    475 / 467
//       surface       1254 / 1049    271 / 270  317 / 317  1355 / 1383 1504 / 1538  4508 / 4353
//     16,777,216 grid  511 / 326     337 / 210  455 / 346   751 / 632  1240 / 1086  2984 / 2651
//       surface       9430 / 7403   2012 / 1979 2476 / 2450 10610 / 10405 11649 / 11727 37122 / 36590
//     boxes of 0.5 m  4452 / 3491   1664 / 1665 2001 / 1964  7660 / 7749 8181 / 8491 23024 / 25189
// (the last row on the surface).  16 hinges: 22.0 / 24.7 ms for the grid of floats, 388 / 516 on
// the surface.
inline bool bhm_gathered(long Q, int hinges, bool f32) {
  if (hinges <= 3 || (f32 && hinges == 7)) return Q > 1L << 21;
  return hinges <= 6 && Q > 1L << 23;
}
// Workgroups go to the 8 XCDs (each with its own L2) in turn; neighbouring blocks of
// points read the same maps, so each XCD takes one contiguous range of the blocks (a
// bijection of [0, n); the results do not depend on it).
__device__ __forceinline__ long bhm_block(long n) {
  constexpr long NX = 8;
  const long i = blockIdx.x, q = n / NX, r = n % NX;
  const long x = i % NX, k = i / NX;
  return (x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q) + k;
}

// The sorted form: points sorted by map box within each block (bitonic sort of (map id, slot)
// keys in LDS), so that a wave's points mostly share a map and load each weight from a few
// addresses.  Each point's result goes back to its own index.
template <class T>
__device__ __forceinline__ void bhm_sorted_slot(const BhmArgs& A, const T* pts, long Q, long* q_out,
                                                int* id_out) {
  __shared__ unsigned long long keys[BS];
  const long blk = bhm_block(gridDim.x);
  const long q = blk * BS + threadIdx.x;
  long key[3];
  const int id = q < Q ? bhm_box(A, pts, q, key) : INT_MAX - 1;
  keys[threadIdx.x] = ((unsigned long long)(unsigned)(id + 1) << 32) | threadIdx.x;
  for (int k = 2; k <= BS; k <<= 1)
    for (int j = k >> 1; j > 0; j >>= 1) {
      __syncthreads();
      const int t = threadIdx.x, o = t ^ j;
      if (o > t) {
        const unsigned long long a = keys[t], b = keys[o];
        const bool up = (t & k) == 0;
        if ((a > b) == up) {
          keys[t] = b;
          keys[o] = a;
        }
      }
    }
  __syncthreads();
  const unsigned long long k = keys[threadIdx.x];
  *q_out = blk * BS + (long)(k & 0xffffffffu);
  *id_out = (int)(k >> 32) - 1;
}

template <class T>
__global__ void __launch_bounds__(BS) bhm_sign_sorted_kernel(BhmArgs A, const T* pts, long Q, double tau,
                                                      int8_t* sign, double* logodds) {
  long q;
  int id;
  bhm_sorted_slot(A, pts, Q, &q, &id);
  if (q >= Q) return;
  long key[3];
  bhm_box(A, pts, q, key);
  const long m = (long)A.nh * A.nh * A.nh;
  double l = 0.0;
  const bool have = id >= 0;
  if (have) {
    // one map for the whole wave: its weights through scalar loads
    const int w0 = __builtin_amdgcn_readfirstlane(id);
    const bool uni = __ballot(id != w0) == 0ull;
    const double* w = A.weights + (long)(uni ? w0 : id) * (m + 1);
    if constexpr (sizeof(T) == 8) l = bhm_logodds64(A, pts, q, key, w);
    else l = (double)bhm_logodds32(A, pts, q, key, w);
  }
  // no local map: the box holds no occupied voxel, taken as free space
  sign[q] = (!have || l < tau) ? 1 : -1;
  if (logodds) logodds[q] = have ? l : -INFINITY;
}

// The gathered form
template <class T>
__global__ void __launch_bounds__(BS) bhm_sign_kernel(BhmArgs A, const T* pts, long Q, double tau,
                                                      int8_t* sign, double* logodds) {
  constexpr bool F32 = sizeof(T) == 4;
  constexpr int PT = BHM_PT;
  __shared__ int slot[BS * PT], map[BS * PT], count[PT][BS / 64];
  __shared__ int hash[BHM_HASH], local[BHM_HASH], maps[BHM_MAPS], n_maps;
  __shared__ alignas(16) float wl[F32 ? BHM_MAPS * BHM_STRIDE : 1];
  const long base = bhm_block(gridDim.x) * (BS * PT);
  const int lane = threadIdx.x & 63, wave = threadIdx.x / 64;
  const bool staged = F32 && A.nh == 7;
  if (threadIdx.x < BHM_HASH) hash[threadIdx.x] = -1;
  if (threadIdx.x == 0) n_maps = 0;
  long key[3];
  int id[PT], before[PT];
  {
    T x[PT][3];
    long flat[PT];
#pragma unroll
    for (int i = 0; i < PT; ++i) {
      const long q = min(base + i * BS + threadIdx.x, Q - 1);
#pragma unroll
      for (int d = 0; d < 3; ++d) x[i][d] = pts[3 * q + d];
    }
#pragma unroll
    for (int i = 0; i < PT; ++i) flat[i] = bhm_flat(A, x[i], key);
#pragma unroll
    for (int i = 0; i < PT; ++i) id[i] = A.box_bhm[max(flat[i], 0L)];
#pragma unroll
    for (int i = 0; i < PT; ++i)
      if (flat[i] < 0 || base + i * BS + threadIdx.x >= Q) id[i] = -1;
  }
#pragma unroll
  for (int i = 0; i < PT; ++i) {
    const long q = base + i * BS + threadIdx.x;
    const unsigned long long have = __ballot(id[i] >= 0);
    before[i] = __popcll(have & ((1ull << lane) - 1ull));
    if (lane == 0) count[i][wave] = __popcll(have);
    if (q < Q && id[i] < 0) {
      // no local map: the box holds no occupied voxel, taken as free space
      sign[q] = 1;
      if (logodds) logodds[q] = -INFINITY;
    }
  }
  __syncthreads();
  int total = 0;
#pragma unroll
  for (int i = 0; i < PT; ++i)
#pragma unroll
    for (int w = 0; w < BS / 64; ++w) {
      if (w == wave && id[i] >= 0) {
        slot[total + before[i]] = i * BS + threadIdx.x;
        map[total + before[i]] = id[i];
      }
      total += count[i][w];
    }
  const long m = (long)A.nh * A.nh * A.nh;
  if (staged) {
    // each map's number in the block, its own or another lane's
#pragma unroll
    for (int i = 0; i < PT; ++i)
      if (id[i] >= 0) {
        for (int p = 0; p < BHM_PROBES; ++p) {
          const int h = bhm_hash(id[i], p), was = atomicCAS(&hash[h], -1, id[i]);
          if (was == -1) {
            const int k = atomicAdd(&n_maps, 1);
            local[h] = k;
            if (k < BHM_MAPS) maps[k] = id[i];
          }
          if (was == -1 || was == id[i]) break;
        }
      }
    __syncthreads();
    const int n = min(n_maps, BHM_MAPS);
    for (int e = threadIdx.x; e < n * 344; e += BS) {
      const int k = e / 344, r = e - k * 344;
      wl[k * BHM_STRIDE + (r < 343 ? r / 7 * 8 + r % 7 : 392)] = (float)A.weights[(long)maps[k] * 344 + r];
    }
  }
  __syncthreads();
  for (int t = threadIdx.x; t < total; t += BS) {
    const long q = base + slot[t];
    const int c = map[t];
    bhm_box(A, pts, q, key);
    const double* w = A.weights + (long)c * (m + 1);
    double l;
    if constexpr (F32) {
      int k = BHM_MAPS;
      for (int p = 0; staged && p < BHM_PROBES; ++p) {
        const int h = bhm_hash(c, p);
        if (hash[h] == c) k = local[h];
      }
      if (k < BHM_MAPS) l = (double)bhm_logodds32_t<7, 8>(A, pts, q, key, wl + k * BHM_STRIDE);
      else l = (double)bhm_logodds32(A, pts, q, key, w);
    } else {
      l = bhm_logodds64(A, pts, q, key, w);
    }
    sign[q] = l < tau ? 1 : -1;
    if (logodds) logodds[q] = l;
  }
}

// per-block sums of l at the hit points, in a fixed order (tree in LDS): FP64 for
// double points; float-float for float points (the FP32 log-odds summed by TwoSum)
template <class T>
__global__ void __launch_bounds__(BT) bhm_tau_partial_kernel(BhmArgs A, const T* pts, long K,
                                                             double* part) {
  __shared__ double red[BT];
  __shared__ float rh[BT], rl[BT];
  const long q = (long)blockIdx.x * BT + threadIdx.x;
  double l = 0.0;
  float lf = 0.f;
  if (q < K) {
    long key[3];
    const int id = bhm_box(A, pts, q, key);
    if (id >= 0) {
      const double* w = A.weights + (long)id * ((long)A.nh * A.nh * A.nh + 1);
      if constexpr (sizeof(T) == 8) l = bhm_logodds64(A, pts, q, key, w);
      else lf = bhm_logodds32(A, pts, q, key, w);
    }
  }
  if constexpr (sizeof(T) == 8) {
    red[threadIdx.x] = l;
    __syncthreads();
    for (int o = BT / 2; o > 0; o >>= 1) {
      if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
      __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
  } else {
    rh[threadIdx.x] = lf;
    rl[threadIdx.x] = 0.f;
    __syncthreads();
    for (int o = BT / 2; o > 0; o >>= 1) {
      if ((int)threadIdx.x < o) {
        const ff a = ff_add(ff{rh[threadIdx.x], rl[threadIdx.x]},
                            ff{rh[threadIdx.x + o], rl[threadIdx.x + o]});
        rh[threadIdx.x] = a.hi;
        rl[threadIdx.x] = a.lo;
      }
      __syncthreads();
    }
    if (threadIdx.x == 0) reinterpret_cast<float2*>(part)[blockIdx.x] = make_float2(rh[0], rl[0]);
  }
}

// tau <- (1 - alpha) tau + (alpha / K) sum_k l(x_k), the partial sums in block order;
// FP64 for double points, float-float for float points (tau converted in and out)
template <bool F64>
__global__ void __launch_bounds__(BT) bhm_tau_final_kernel(const double* part, long n_part, long K,
                                                           double alpha, double* tau) {
  if constexpr (F64) {
    __shared__ double red[BT];
    double s = 0.0;
    for (long i = threadIdx.x; i < n_part; i += BT) s += part[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = BT / 2; o > 0; o >>= 1) {
      if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
      __syncthreads();
    }
    if (threadIdx.x == 0) *tau = (1.0 - alpha) * *tau + alpha / (double)K * red[0];
  } else {
    __shared__ float rh[BT], rl[BT];
    const float2* pf = reinterpret_cast<const float2*>(part);
    ff s{0.f, 0.f};
    for (long i = threadIdx.x; i < n_part; i += BT) s = ff_add(s, ff{pf[i].x, pf[i].y});
    rh[threadIdx.x] = s.hi;
    rl[threadIdx.x] = s.lo;
    __syncthreads();
    for (int o = BT / 2; o > 0; o >>= 1) {
      if ((int)threadIdx.x < o) {
        const ff a = ff_add(ff{rh[threadIdx.x], rl[threadIdx.x]},
                            ff{rh[threadIdx.x + o], rl[threadIdx.x + o]});
        rh[threadIdx.x] = a.hi;
        rl[threadIdx.x] = a.lo;
      }
      __syncthreads();
    }
    if (threadIdx.x == 0) {
      const double t0 = *tau, wk = alpha / (double)K, keep = 1.0 - alpha;
      const float th = (float)t0, wh = (float)wk, kh = (float)keep;
      const ff t{th, (float)(t0 - (double)th)}, w{wh, (float)(wk - (double)wh)},
          kp{kh, (float)(keep - (double)kh)};
      const ff r = ff_add(ff_mul(kp, t), ff_mul(w, ff{rh[0], rl[0]}));
      *tau = (double)r.hi + (double)r.lo;
    }
  }
}
bool make_bhm_args(const ksdf_bhm_layout* L, const int* box_bhm, const double* weights, BhmArgs* A) {
  if (!L || !box_bhm || !weights || !(L->box > 0) || !std::isfinite(L->box) || !(L->gamma > 0) ||
      !std::isfinite(L->gamma) || L->hinges < 2 || L->hinges > MAX_HINGES || L->dims[0] < 1 ||
      L->dims[1] < 1 || L->dims[2] < 1)
    return false;
  for (int d = 0; d < 3; ++d) {
    if (!std::isfinite(L->origin[d])) return false;
    A->origin[d] = L->origin[d];
    A->dims[d] = L->dims[d];
  }
  A->box = L->box;
  // the remainder x - t B of a quotient near 1 or more is exact down to 2^-1022 + 53
  A->inv_box = L->box >= 0x1p-960 ? 1.0 / L->box : (double)NAN;
  A->spacing = L->box / (double)(L->hinges - 1);
  A->nh = L->hinges;
  A->gamma = L->gamma;
  A->box_bhm = box_bhm;
  A->weights = weights;
  auto split = [](double v, float out[2]) {
    out[0] = (float)v;
    out[1] = (float)(v - (double)out[0]);
  };
  for (int d = 0; d < 3; ++d) split(A->origin[d], A->origin_ff[d]);
  split(A->box, A->box_ff);
  split(A->spacing, A->spacing_ff);
  return true;
}

}  // namespace

size_t bhm_tau_workspace_bytes(long K) { return (size_t)((K + BT - 1) / BT + 1) * sizeof(double); }

int launch_bhm_sign(const ksdf_bhm_layout* L, const int* box_bhm, const double* weights,
                    const void* points, int dtype, long Q, double tau, int8_t* sign,
                    double* logodds, hipStream_t s) {
  BhmArgs A;
  if (!make_bhm_args(L, box_bhm, weights, &A) || Q < 0 || (Q > 0 && (!points || !sign)) ||
      !std::isfinite(tau) || (dtype != KSDF_DTYPE_F32 && dtype != KSDF_DTYPE_F64)) {
    set_error("ksdf_bhm_sign: invalid argument");
    return KSDF_ERR_INVALID_ARGUMENT;
  }
  if (Q == 0) return KSDF_OK;
  const bool many = bhm_gathered(Q, L->hinges, dtype == KSDF_DTYPE_F32);
  const int pt = many ? BHM_PT : 1;
  const dim3 g((unsigned)((Q + BS * pt - 1) / (BS * pt)));
  if (dtype == KSDF_DTYPE_F64) {
    const double* p = static_cast<const double*>(points);
    if (many) hipLaunchKernelGGL(bhm_sign_kernel<double>, g, dim3(BS), 0, s, A, p, Q, tau, sign, logodds);
    else hipLaunchKernelGGL(bhm_sign_sorted_kernel<double>, g, dim3(BS), 0, s, A, p, Q, tau, sign, logodds);
  } else {
    const float* p = static_cast<const float*>(points);
    if (many) hipLaunchKernelGGL(bhm_sign_kernel<float>, g, dim3(BS), 0, s, A, p, Q, tau, sign, logodds);
    else hipLaunchKernelGGL(bhm_sign_sorted_kernel<float>, g, dim3(BS), 0, s, A, p, Q, tau, sign, logodds);
  }
  KSDF_HIP_TRY(hipGetLastError());
  return KSDF_OK;
}

int launch_bhm_update_tau(const ksdf_bhm_layout* L, const int* box_bhm, const double* weights,
                          const void* hits, int dtype, long K, double alpha, double* tau, void* ws,
                          size_t ws_bytes, hipStream_t s) {
  BhmArgs A;
  if (!make_bhm_args(L, box_bhm, weights, &A) || K < 1 || !hits || !tau || !(alpha > 0) ||
      alpha > 1 || (dtype != KSDF_DTYPE_F32 && dtype != KSDF_DTYPE_F64)) {
    set_error("ksdf_bhm_update_tau: invalid argument");
    return KSDF_ERR_INVALID_ARGUMENT;
  }
  if (!ws || ws_bytes < bhm_tau_workspace_bytes(K)) {
    set_error("ksdf_bhm_update_tau: workspace too small");
    return KSDF_ERR_WORKSPACE;
  }
  double* part = static_cast<double*>(ws);
  const long g = (K + BT - 1) / BT;
  if (dtype == KSDF_DTYPE_F64)
    hipLaunchKernelGGL(bhm_tau_partial_kernel<double>, dim3((unsigned)g), dim3(BT), 0, s, A,
                       static_cast<const double*>(hits), K, part);
  else
    hipLaunchKernelGGL(bhm_tau_partial_kernel<float>, dim3((unsigned)g), dim3(BT), 0, s, A,
                       static_cast<const float*>(hits), K, part);
  if (dtype == KSDF_DTYPE_F64)
    hipLaunchKernelGGL(bhm_tau_final_kernel<true>, dim3(1), dim3(BT), 0, s, part, g, K, alpha, tau);
  else
    hipLaunchKernelGGL(bhm_tau_final_kernel<false>, dim3(1), dim3(BT), 0, s, part, g, K, alpha, tau);
  KSDF_HIP_TRY(hipGetLastError());
  return KSDF_OK;
}

}  // namespace ksdf
