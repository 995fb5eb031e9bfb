// FP32 query with eight lanes per query, for query sets too sparse to share cells.
//
// The two-kernel query (query_split.h) lets a wave walk the cells of 64 neighbouring
// queries; where neighbours share few cells, or where there are few queries, its waves
// walk many cells one after the other and most of the chip idles.  Here a wave holds
// eight queries and the eight lanes of a query work side by side:
//   candidates   each lane scans every eighth entry of the box's list, the sorted private
//                lists are merged by group-wide minima of (distance, id);
//   UDF          lane g evaluates the candidates of rank g (and g + 8), every one of
//                them; the walk's pruning is then replayed in rank order;
//   fusion       resolve_min on the group's replicated values;
//   outputs      eight samples of the argmin cell at a time: lane g forms the terms of
//                sample g, they pass through LDS, and each lane carries one of the eight
//                running sums, so that every sum is taken in sample order; the GP
//                variance's substitution runs over blocks of eight rows, a row per lane.
// Every operation and every sum keeps the order of the per-lane kernels, so the outputs
// are theirs bit for bit, whatever the launch.
//
// With few queries it is bound by the length of one query's chain (64 waypoints 30 us, of
// which the wave walk took 650); from some 30,000 on by instruction issue, about 5,000
// vector instructions and 250 gathers per wave of eight queries (262,144 trajectory points
// 0.48 ms).  Loads of the next samples are in flight during the current ones' terms, and the
// factor's rows come 16 bytes a load (0.62 ms without either).
#include "query_dev.h"
#include "group_dev.h"

namespace ksdf {
namespace {

constexpr int GT_ROWS = 11;

struct GroupLds {
  alignas(16) float k[GQ * GK_STRIDE];      // kernel vector, then L^{-1} k
  alignas(16) float t[GT_ROWS * GT_STRIDE]; // terms of 8 samples x 8 queries, by kind
};

// K nearest cells of the group's query (see query_candidates), the same in all its lanes
template <int KM>
__device__ __forceinline__ void group_candidates(const FastArgs& A, bool active, float qx, float qy,
                                                 float qz, int (&cid)[KM], int& n, bool& outside) {
  const int g = threadIdx.x & (GL - 1);
  float cd[KM];
  int ci[KM];
#pragma unroll
  for (int r = 0; r < KM; ++r) {
    cd[r] = INFINITY;
    ci[r] = 0x7fffffff;
  }
  int subkey;
  const long bkey = box_key(A, qx, qy, qz, &subkey);
  outside = bkey < 0;
  int beg = 0, end = 0;
  if (active) {
    end = A.n_cells;
    if (!outside) {
      beg = A.box_off[bkey];
      end = A.box_off[bkey + 1];
    }
  }
  const bool sorted = !outside && end - beg <= INDEX_SORTED_MAX;
  const float4 bc = box_centre(A, qx, qy, qz);
  const float rho = __builtin_amdgcn_sqrtf(cand_d2(qx, qy, qz, bc));
  for (int t0 = beg; t0 < end; t0 += 4 * GL) {   // uniform in the group
    int cc[4];
    float4 ce[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int t = min(t0 + g + u * GL, end - 1);
      cc[u] = outside ? t : A.box_list[t];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) ce[u] = A.centre[cc[u]];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (t0 + g + u * GL < end) cand_insert<KM>(cd, ci, cand_d2(qx, qy, qz, ce[u]), cc[u]);
    // every lane holds KM / 8 entries within the greatest of the lanes' KM / 8-th
    const float kth = group_max(cd[KM / GL - 1]);
    if (sorted && group_all(cand_scan_over(A, cand_d2(bc.x, bc.y, bc.z, ce[3]), kth, rho))) break;
  }
  n = active ? min(A.k, end - beg) : 0;
#pragma unroll
  for (int r = 0; r < KM; ++r) {
    float d = cd[0];
    int id = ci[0];
    group_min(d, id);
    cid[r] = id;
    if (ci[0] == id) {   // ids are unique: one lane drops its head
#pragma unroll
      for (int j = 0; j + 1 < KM; ++j) {
        cd[j] = cd[j + 1];
        ci[j] = ci[j + 1];
      }
      cd[KM - 1] = INFINITY;
      ci[KM - 1] = 0x7fffffff;
    }
  }
}

// cell_u2_lane with the next eight samples' loads in flight during the current eight's terms
// (entries past m contribute nothing)
__device__ __forceinline__ void cell_u2_group(const FastArgs& A, int b, int m, float lx, float ly,
                                              float lz, float& d2ref, float& u2, float& del) {
  constexpr int C = 8;
  const float c2 = A.c2;
  float f = 0.f, R = 0.f, RZ = 0.f;
  u2 = INFINITY;
  del = 0.f;
  const float4* __restrict__ ps = A.ps + b;
  for (int pass = 0; pass < 2; ++pass) {
    const float c2d = c2 * d2ref;
    float emax = 0.f;
    f = 0.f;
    R = 0.f;
    RZ = 0.f;
    float4 N[C];
#pragma unroll
    for (int j = 0; j < C; ++j) N[j] = ps[min(j, m - 1)];
    for (int i0 = 0; i0 < m; i0 += C) {
      float4 P[C];
#pragma unroll
      for (int j = 0; j < C; ++j) P[j] = N[j];
#pragma unroll
      for (int j = 0; j < C; ++j) N[j] = ps[min(i0 + C + j, m - 1)];
#pragma unroll
      for (int j = 0; j < C; ++j) {
        const bool in = i0 + j < m;
        const float dx = lx - P[j].x, dy = ly - P[j].y, dz = lz - P[j].z;
        const float z2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
        const float e = in ? __builtin_amdgcn_exp2f(fmaf(z2, -c2, c2d)) : 0.f;
        const float ae = fabsf(P[j].w) * e;
        f = fmaf(P[j].w, e, f);
        R += ae;
        RZ = fmaf(ae, z2, RZ);
        emax = fmaxf(emax, e);
      }
    }
    if (emax >= 0x1p-24f) break;
    float d2 = INFINITY;
    for (int i = 0; i < m; ++i) {
      const float4 p = ps[i];
      const float dx = lx - p.x, dy = ly - p.y, dz = lz - p.z;
      d2 = fminf(d2, fmaf(dz, dz, fmaf(dy, dy, dx * dx)));
    }
    d2ref = d2;
  }
  if (f > 0.f) {
    u2 = d2ref - A.two_l2 * LN2 * __log2f(f);
    del = A.two_l2 * EPS32 * (6.f * R + 3.5f * c2 * RZ) / f;
  }
}

// cell_u_matern_lane, the same way
__device__ __forceinline__ void cell_u_matern_group(const FastArgs& A, int b, int m, float lx, float ly,
                                                    float lz, float& d2ref, float& u, float& del) {
  constexpr int C = 8;
  const float mc = A.mc, mcl = A.mc_l2e;
  float f = 0.f, R = 0.f, RZ = 0.f;
  u = INFINITY;
  del = 0.f;
  const float4* __restrict__ ps = A.ps + b;
  for (int pass = 0; pass < 2; ++pass) {
    const float dref = __builtin_amdgcn_sqrtf(d2ref);
    float emax = 0.f;
    f = 0.f;
    R = 0.f;
    RZ = 0.f;
    float4 N[C];
#pragma unroll
    for (int j = 0; j < C; ++j) N[j] = ps[min(j, m - 1)];
    for (int i0 = 0; i0 < m; i0 += C) {
      float4 P[C];
#pragma unroll
      for (int j = 0; j < C; ++j) P[j] = N[j];
#pragma unroll
      for (int j = 0; j < C; ++j) N[j] = ps[min(i0 + C + j, m - 1)];
#pragma unroll
      for (int j = 0; j < C; ++j) {
        const bool in = i0 + j < m;
        const float dx = lx - P[j].x, dy = ly - P[j].y, dz = lz - P[j].z;
        const float z = __builtin_amdgcn_sqrtf(fmaf(dz, dz, fmaf(dy, dy, dx * dx)));
        const float ex = in ? __builtin_amdgcn_exp2f(mcl * (dref - z)) : 0.f;
        const float g = fmaf(mc, z, 1.f) * ex;
        const float ag = fabsf(P[j].w) * g;
        f = fmaf(P[j].w, g, f);
        R += ag;
        RZ = fmaf(ag, z, RZ);
        emax = fmaxf(emax, ex);
      }
    }
    if (emax >= 0x1p-24f) break;
    float d2 = INFINITY;
    for (int i = 0; i < m; ++i) {
      const float4 p = ps[i];
      const float dx = lx - p.x, dy = ly - p.y, dz = lz - p.z;
      d2 = fminf(d2, fmaf(dz, dz, fmaf(dy, dy, dx * dx)));
    }
    d2ref = d2;
  }
  if (f > 0.f) {
    u = __builtin_amdgcn_sqrtf(d2ref) - LN2 * __log2f(f) / mc;
    del = EPS32 * (8.f * R + 4.f * mc * RZ) / (mc * f);
  }
}

template <int KM, bool MAT>
__global__ void __launch_bounds__(64) query_group_kernel(FastArgs A) {
  __shared__ GroupLds S;
  constexpr int NC = KM / GL;   // candidates per lane
  const int lane = threadIdx.x & 63, g = lane & (GL - 1), base = lane - g;
  const long sq = xcd_block(gridDim.x) * GQ + lane / GL;
  const bool active = sq < A.Q;
  const long qi = active ? (A.perm ? (long)A.perm[sq] : sq) : 0;
  const float qx = A.pts[3 * qi], qy = A.pts[3 * qi + 1], qz = A.pts[3 * qi + 2];
  int cid[KM];
  int n = 0;
  bool outside = false;
  group_candidates<KM>(A, active, qx, qy, qz, cid, n, outside);

  // every candidate's u^2 (or u), one lane each
  float mu[NC], mdel[NC], mlb[NC], mref[NC];
#pragma unroll
  for (int s = 0; s < NC; ++s) {
    mu[s] = INFINITY;
    mdel[s] = 0.f;
    mlb[s] = 0.f;
    mref[s] = 0.f;
    int c = 0x7fffffff;
#pragma unroll
    for (int r = 0; r < GL; ++r)
      if (r == g) c = cid[s * GL + r];
    if (s * GL + g < n && c != 0x7fffffff) {
      const int b = A.offsets[c];
      const int m = A.offsets[c + 1] - b;
      const float4 ctr = A.centre[c];
      const float* bx = A.box + 8L * c;
      const float lx = qx - ctr.x, ly = qy - ctr.y, lz = qz - ctr.z;
      float d2ref = aabb_d2(bx, lx, ly, lz);
      mlb[s] = cell_lower_bound(A, d2ref, bx[3]);
      if constexpr (MAT) cell_u_matern_group(A, b, m, lx, ly, lz, d2ref, mu[s], mdel[s]);
      else cell_u2_group(A, b, m, lx, ly, lz, d2ref, mu[s], mdel[s]);
      mref[s] = d2ref;
    }
  }
  // the values the walk in rank order would keep (a candidate whose lower bound cannot
  // improve on the minimum so far is left out)
  float cu2[KM], cdl[KM];
  float best = INFINITY, best_del = 0.f;
  static_for<0, KM>([&](auto R) {
    constexpr int r = R;
    const float u2 = group_lane<r % GL>(mu[r / GL]), del = group_lane<r % GL>(mdel[r / GL]),
                lb = group_lane<r % GL>(mlb[r / GL]);
    const bool ev = r < n && !(lb > best + 2.f * best_del + 1e-6f);
    cu2[r] = ev ? u2 : INFINITY;
    cdl[r] = ev ? del : 0.f;
    if (cu2[r] < best) {
      best = cu2[r];
      best_del = cdl[r];
    }
  });
  const int bc = resolve_min<KM, GL>(A, active, qx, qy, qz, cid, n, cu2, cdl, best);
  int slot = 0;
#pragma unroll
  for (int r = 0; r < KM; ++r)
    if (r < n && cid[r] == bc) slot = r;
  float bref = __shfl(mref[0], base + (slot & (GL - 1)), 64);
  if constexpr (NC > 1) {
    const float b1 = __shfl(mref[1], base + (slot & (GL - 1)), 64);
    if (slot >= GL) bref = b1;
  }

  // ---- the argmin cell's outputs (query_finish_t's terms and sums)
  float w0 = 0.f, w1 = 0.f, w2 = 0.f, vv = 0.f, var = 0.f, gv0 = 0.f, gv1 = 0.f, gv2 = 0.f;
  const bool have = bc >= 0;
  if (__ballot(have)) {
    const float c2 = A.c2;
    const int c = have ? bc : 0;
    const int b = A.offsets[c];
    const int m = have ? A.offsets[c + 1] - b : 0;
    const float* Lc = A.L + A.loff[c];
    const float4 ctr = A.centre[c];
    const float lx = qx - ctr.x, ly = qy - ctr.y, lz = qz - ctr.z;
    const float c2d = c2 * bref;
    const float ginv = __builtin_amdgcn_exp2f(-c2d);
    const float zref = __builtin_amdgcn_sqrtf(bref);
    const float ll = fmaf(lz, lz, fmaf(ly, ly, lx * lx));
    const bool farl = ll > A.far2;
    const float k0 = c2 * (bref - ll);
    const float tx = 2.f * c2 * lx, ty = 2.f * c2 * ly, tz = 2.f * c2 * lz;
    const float ginvm = MAT ? __builtin_amdgcn_exp2f(-A.mc_l2e * zref) : 0.f;
    const float bm = bref - ll;
    float* kq = S.k + lane / GL * GK_STRIDE;
    float* row = S.t + lane;
    row[8 * GT_STRIDE] = 1.f;
    // lane c's running sum: w (3), S, T1, X0, X1, X2 as x(c) y(c) with the terms' rows
    // ae, dx, dy, dz, sm, ti, q, q ti, 1, sm^2 and sigma^2 (q = sm^2 sigma^2 joins X0 as one
    // fused step)
    const int xr = lane_entry(lanes8(0, 0, 0, 8, 4, 9, 6, 7));
    const int yr = lane_entry(lanes8(1, 2, 3, 4, 5, 10, 5, 5));
    float acc = 0.f;
    const int last = max(m - 1, 0);
    float4 Pn = A.ps[b + min(g, last)];
    float SVn = A.sv[b + min(g, last)];
    for (int i0 = 0; __ballot(i0 < m); i0 += GL) {
      const int i = i0 + g;
      const bool in = i < m;
      const float4 P = Pn;
      const float SV = SVn;
      Pn = A.ps[b + min(i + GL, last)];
      SVn = A.sv[b + min(i + GL, last)];
      const float dx = lx - P.x, dy = ly - P.y, dz = lz - P.z;
      const float z2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
      const float pp = fmaf(P.z, P.z, fmaf(P.y, P.y, P.x * P.x));
      const float z = __builtin_amdgcn_sqrtf(z2);
      float e, kv;
      if constexpr (MAT) {
        const float lp2 = fmaf(2.f * lx, P.x, fmaf(2.f * ly, P.y, fmaf(2.f * lz, P.z, bm - pp)));
        const float dd = farl ? lp2 / (zref + z) : zref - z;
        e = in ? __builtin_amdgcn_exp2f(A.mc_l2e * dd) : 0.f;
        kv = fmaf(A.mc, z, 1.f) * e * ginvm;
      } else {
        const float arg_far = fmaf(tx, P.x, fmaf(ty, P.y, fmaf(tz, P.z, fmaf(-c2, pp, k0))));
        const float arg = farl ? arg_far : fmaf(z2, -c2, c2d);
        e = in ? __builtin_amdgcn_exp2f(arg) : 0.f;
        kv = e * ginv;
      }
      const float ti = A.alpha * (z - zref);
      const float sm = in ? __builtin_amdgcn_exp2f(-A.alpha_l2e * (z - zref)) : 0.f;
      const float q = sm * sm * SV;
      row[0 * GT_STRIDE] = P.w * e;
      row[1 * GT_STRIDE] = dx;
      row[2 * GT_STRIDE] = dy;
      row[3 * GT_STRIDE] = dz;
      row[4 * GT_STRIDE] = sm;
      row[5 * GT_STRIDE] = ti;
      row[6 * GT_STRIDE] = q;
      row[7 * GT_STRIDE] = q * ti;
      row[9 * GT_STRIDE] = sm * sm;
      row[10 * GT_STRIDE] = SV;
      kq[i] = in ? kv : 0.f;   // i < 128
      wave_lds_sync();
      group_fma(S.t, xr, yr, acc);
      wave_lds_sync();
    }
    w0 = group_lane<0>(acc);
    w1 = group_lane<1>(acc);
    w2 = group_lane<2>(acc);
    const float Ssum = group_lane<3>(acc), T1 = group_lane<4>(acc), X0 = group_lane<5>(acc),
                X1 = group_lane<6>(acc), X2 = group_lane<7>(acc);
    const float Tb = 1.f + T1 / Ssum;
    var = (Tb * Tb * X0 - 2.f * Tb * X1 + X2) / (Ssum * Ssum);
    if (A.var_f) vv = group_forward_subst(kq, Lc, m);
    if (A.grad_var) {
      // grad_var_cell's two passes, the same way
      const float invS = 1.f / Ssum;
      float V[3] = {0.f, 0.f, 0.f}, G[3] = {0.f, 0.f, 0.f};
      const float a2 = A.alpha * A.alpha;
      for (int pass = 0; pass < 2; ++pass) {
        acc = 0.f;
        for (int i0 = 0; __ballot(i0 < m); i0 += GL) {
          const int i = i0 + g;
          const bool in = i < m;
          const int j = in ? i : 0;
          const float4 P = A.ps[b + j];
          const float dx = lx - P.x, dy = ly - P.y, dz = lz - P.z;
          const float z = __builtin_amdgcn_sqrtf(fmaf(dz, dz, fmaf(dy, dy, dx * dx)));
          const bool ok = in && z > 0.f;   // a sample at the query has no direction
          const float s = __builtin_amdgcn_exp2f(-A.alpha_l2e * (z - zref)) * invS;
          const float l = s * (Tb - A.alpha * (z - zref));
          const float iz = 1.f / z;
          const float v0 = dx * iz, v1 = dy * iz, v2 = dz * iz;
          if (pass == 0) {
            row[0 * GT_STRIDE] = ok ? s : 0.f;
            row[1 * GT_STRIDE] = ok ? l : 0.f;
            row[2 * GT_STRIDE] = ok ? v0 : 0.f;
            row[3 * GT_STRIDE] = ok ? v1 : 0.f;
            row[4 * GT_STRIDE] = ok ? v2 : 0.f;
          } else {
            const float lz2 = (l * iz) * (l * iz);
            const float x0 = l * (v0 - V[0]) + s * (v0 - G[0]);
            const float x1 = l * (v1 - V[1]) + s * (v1 - G[1]);
            const float x2 = l * (v2 - V[2]) + s * (v2 - G[2]);
            row[0 * GT_STRIDE] = ok ? A.sv[b + j] : 0.f;
            row[1 * GT_STRIDE] = ok ? fmaf(a2 * x0, x0, lz2 * (1.f - v0 * v0)) : 0.f;
            row[2 * GT_STRIDE] = ok ? fmaf(a2 * x1, x1, lz2 * (1.f - v1 * v1)) : 0.f;
            row[3 * GT_STRIDE] = ok ? fmaf(a2 * x2, x2, lz2 * (1.f - v2 * v2)) : 0.f;
          }
          wave_lds_sync();
          if (pass == 0) group_fma(S.t, lane_entry(lanes8(0, 0, 0, 1, 1, 1, 0, 0)),
                                   lane_entry(lanes8(2, 3, 4, 2, 3, 4, 2, 2)), acc);
          else group_fma(S.t, 0, lane_entry(lanes8(1, 2, 3, 1, 1, 1, 1, 1)), acc);
          wave_lds_sync();
        }
        if (pass == 0) {
          V[0] = group_lane<0>(acc);
          V[1] = group_lane<1>(acc);
          V[2] = group_lane<2>(acc);
          G[0] = group_lane<3>(acc);
          G[1] = group_lane<4>(acc);
          G[2] = group_lane<5>(acc);
        }
      }
      gv0 = group_lane<0>(acc);
      gv1 = group_lane<1>(acc);
      gv2 = group_lane<2>(acc);
    }
  }
  if (g == 0) write_outputs<MAT>(A, active, outside, 0, qi, bc, best, w0, w1, w2, vv, var, gv0, gv1, gv2);
}

}  // namespace

void launch_query_group(const ksdf_model* m, const FastArgs& A, hipStream_t s) {
  const dim3 grid((unsigned)((A.Q + GQ - 1) / GQ)), block(64);
  if (m->k_fuse <= 8) {
    if (A.matern) hipLaunchKernelGGL((query_group_kernel<8, true>), grid, block, 0, s, A);
    else hipLaunchKernelGGL((query_group_kernel<8, false>), grid, block, 0, s, A);
  } else {
    if (A.matern) hipLaunchKernelGGL((query_group_kernel<16, true>), grid, block, 0, s, A);
    else hipLaunchKernelGGL((query_group_kernel<16, false>), grid, block, 0, s, A);
  }
}

}  // namespace ksdf
