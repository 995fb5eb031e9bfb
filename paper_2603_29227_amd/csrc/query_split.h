// Two-kernel form of the FP32 query (a launch choice with the same outputs as the
// one-kernel form of query_fast.hip).
//
// Pass 1 (candidates, min-fusion) writes one 16-byte record per query in wave order and
// counts the queries of each argmin cell; the records are regrouped by argmin cell;
// pass 2 then meets one or two argmin cells per wave instead of the two to three of
// a spatial bucket, so the per-cell work (gradient, GP variance by forward
// substitution, softmin variance) is not repeated for lanes that idle.
//
// The kernels are instantiated per block size and cell mode in
// query_split{64,256}_{wave,lane}.hip, which compile in parallel.
#pragma once

#include "query_dev.h"

namespace ksdf {
namespace {

template <int KM, int NT, bool LANE, bool MAT = false, bool COOP = false>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(KM == 8 ? (COOP ? 4 : 5) : 1)))
query_p1_kernel(FastArgs A, P1Rec* rec, int* count) {
  const long sq = xcd_block(gridDim.x) * NT + threadIdx.x;
  __shared__ float4 buf[COOP ? NT / 64 * COOP_LDS : 1];
  const Pass1 r = query_pass1<KM, LANE, MAT, COOP>(A, sq, buf + (COOP ? threadIdx.x / 64 * COOP_LDS : 0));
  const bool active = (r.flags & 2) != 0;
  const int slot = wave_slot(count, r.bc < 0 ? A.n_cells : (A.p2rank ? A.p2rank[r.bc] : r.bc), active);
  if (active) {
    rec[sq] = pack_p1(r);
    A.rank[sq] = slot;
  }
}

// Each record to its place: its bin's start plus its place in the bin, which pass 1's count
// gave it: 102 us for the 256^3 grid's 16.8M records (249 us with atomics of its own)
__global__ void __launch_bounds__(256) query_regroup_kernel(const P1Rec* rec, long Q, int n_cells,
                                                            const int* p2rank, const int* start,
                                                            const int* rank, P1Rec* rec2) {
  const long sq = (long)blockIdx.x * 256 + threadIdx.x;
  if (sq >= Q) return;
  const P1Rec r = rec[sq];
  const int bc = p1rec_cell(r);
  rec2[start[bc < 0 ? n_cells : (p2rank ? p2rank[bc] : bc)] + rank[sq]] = r;
}

// split_bin >= 0: the records are grouped by A.p2rank and the launch takes those of
// the cells of rank < split_bin (side 0) or the rest (side 1); their boundary is the
// start of bin split_bin
template <int MB, int NT, bool LANE, bool MF = false, bool MAT = false>
__global__ void __launch_bounds__(NT) query_p2_kernel(FastArgs A, const P1Rec* rec2,
                                                      const int* start, int split_bin,
                                                      int side) {
  long lo = 0, hi = A.Q;
  if (split_bin >= 0) {
    const long S = start[split_bin];
    if (side == 0) hi = S;
    else lo = S;
  }
  // the blocks of this launch's side [lo, hi) are spread over the 8 XCDs, each XCD one
  // contiguous range of them (as xcd_block does for a whole launch); the launch has a
  // block for every query, rounded up to a multiple of 8, so the blocks past the
  // side's count leave at once
  const long base = lo / NT * NT;
  const long nb = (hi - base + NT - 1) / NT;
  const long per = (nb + N_XCD - 1) / N_XCD;
  const long bx = (long)blockIdx.x % N_XCD, bk = (long)blockIdx.x / N_XCD;
  if (bk >= per || bx * per + bk >= nb) return;   // uniform over the block
  const long sq = base + (bx * per + bk) * NT + threadIdx.x;
  if (split_bin >= 0) {
    const long w0 = sq - (threadIdx.x & 63);
    if (w0 + 64 <= lo || w0 >= hi) return;   // the whole wave is on the other side
  }
  Pass1 r{};
  r.bc = -1;
  if (sq >= lo && sq < hi) {
    const P1Rec o = rec2[sq];
    r.qi = o.qi;
    r.bc = p1rec_cell(o);
    r.flags = (int)(o.cf >> P1REC_CELL_BITS);
    r.best = o.best;
    r.bref = o.bref;
    r.qx = A.pts[3L * o.qi];
    r.qy = A.pts[3L * o.qi + 1];
    r.qz = A.pts[3L * o.qi + 2];
  }
  query_finish_t<MB, LANE, MF, MAT>(A, r);
}

// Per-lane cells: with the samples loaded by eight lanes each, but for K > 8 and cells over 64
// samples, whose lanes end at unlike times and whose registers leave two waves per SIMD
// (262,144 points, together / each its own: K = 8, m <= 64 335 / 396 us; K = 8, uneven m <= 128
// 655 / 655; K = 16, m <= 64 575 / 642; K = 16, uneven m <= 128 974 / 864).
template <int NT, bool LANE, bool MAT>
void launch_p1(const ksdf_model* m, const FastArgs& A, P1Rec* rec, int* count, unsigned g, hipStream_t s) {
  if (m->k_fuse <= 8)
    hipLaunchKernelGGL((query_p1_kernel<8, NT, LANE, MAT, LANE>), dim3(g), dim3(NT), 0, s, A, rec, count);
  else if (m->max_m <= 64)
    hipLaunchKernelGGL((query_p1_kernel<16, NT, LANE, MAT, LANE>), dim3(g), dim3(NT), 0, s, A, rec, count);
  else
    hipLaunchKernelGGL((query_p1_kernel<16, NT, LANE, MAT>), dim3(g), dim3(NT), 0, s, A, rec, count);
}

template <int NT, bool LANE>
void launch_split_nt(const ksdf_model* m, const FastArgs& A, P1Rec* rec, P1Rec* rec2, int* count,
                     int* cursor, int* tsum, void* pws, hipStream_t s) {
  const unsigned g = (unsigned)((A.Q + NT - 1) / NT);
  const unsigned g2 = (g + N_XCD - 1) / N_XCD * N_XCD;   // pass 2: whole rounds of the XCDs
  const long nc = (long)m->n_cells + 1;
  hipLaunchKernelGGL(fill_kernel, dim3((unsigned)((nc + 255) / 256)), dim3(256), 0, s, count, nc, 0);
  if (pws) launch_pass1_pairs(m, A, rec, count, pws, s);
  else if (A.matern) launch_p1<NT, LANE, true>(m, A, rec, count, g, s);
  else launch_p1<NT, LANE, false>(m, A, rec, count, g, s);
  launch_scan(count, nc, tsum, cursor, s);
  hipLaunchKernelGGL(query_regroup_kernel, dim3((unsigned)((A.Q + 255) / 256)), dim3(256), 0, s, rec,
                     A.Q, m->n_cells, A.p2rank, cursor, A.rank, rec2);
  if constexpr (!LANE) {
    if (m->tuning.query_mfma && m->Linv32 && m->max_m <= 64) {
      if (!m->linv_ok) launch_linv(m, s);
      hipLaunchKernelGGL((query_p2_kernel<64, NT, false, true>), dim3(g2), dim3(NT), 0, s, A, rec2,
                         cursor, -1, 0);
      return;
    }
  }
  // the kernel function picks the pass-2 instantiation (Matern models carry u, not u^2);
  // with cells of more than 64 samples, the records of the cells of up to 64 run in the
  // launch sized for 64 (fewer registers, more waves per SIMD) and the rest in the one
  // sized for 128
  if (m->max_m <= 64) {
    if (A.matern)
      hipLaunchKernelGGL((query_p2_kernel<64, NT, LANE, false, true>), dim3(g2), dim3(NT), 0, s, A, rec2,
                         cursor, -1, 0);
    else
      hipLaunchKernelGGL((query_p2_kernel<64, NT, LANE>), dim3(g2), dim3(NT), 0, s, A, rec2,
                         cursor, -1, 0);
    return;
  }
  const int split = m->bucket_start[3];   // ranks of the cells of up to 64 samples
  if (A.matern) {
    hipLaunchKernelGGL((query_p2_kernel<64, NT, LANE, false, true>), dim3(g2), dim3(NT), 0, s, A, rec2,
                         cursor, split, 0);
    hipLaunchKernelGGL((query_p2_kernel<128, NT, LANE, false, true>), dim3(g2), dim3(NT), 0, s, A, rec2,
                         cursor, split, 1);
  } else {
    hipLaunchKernelGGL((query_p2_kernel<64, NT, LANE>), dim3(g2), dim3(NT), 0, s, A, rec2,
                       cursor, split, 0);
    hipLaunchKernelGGL((query_p2_kernel<128, NT, LANE>), dim3(g2), dim3(NT), 0, s, A, rec2,
                         cursor, split, 1);
  }
}

}  // namespace
}  // namespace ksdf
