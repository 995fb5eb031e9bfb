// Host side of the FP32 query: the counting sort of the queries, the choice of the
// launch, and its workspace.
#include "query_dev.h"

namespace ksdf {
namespace {

// The counting sort: the count gives every query its place in its bin (one atomic per
// distinct bin of a wave), so that the scatter only reads and writes: 65 us for the 256^3
// grid (230 us with atomics of its own, for which the lanes of a wave waited in turn).
__global__ void bin_kernel(FastArgs A, int* keys, int* ranks, int* counts, long n_bins) {
  const long q = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const bool valid = q < A.Q;
  int key = 0;
  if (valid) {
    int sub;
    const long b = box_key(A, A.pts[3 * q], A.pts[3 * q + 1], A.pts[3 * q + 2], &sub);
    key = b < 0 ? (int)(n_bins - 1) : (int)((long)A.box_rank[b] * A.sub * A.sub * A.sub + sub);
    keys[q] = key;
  }
  const int rank = wave_slot(counts, key, valid);
  if (valid) ranks[q] = rank;
}
__global__ void scatter_kernel(long Q, const int* keys, const int* ranks, const int* start, int* perm) {
  const long q = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (q < Q) perm[start[keys[q]] + ranks[q]] = (int)q;
}

// The permutation written by launch_bucketing (the workspace's second array).
inline int* bucketed_perm(void* ws, long Q) {
  return reinterpret_cast<int*>(static_cast<char*>(ws) + align256(Q * sizeof(int)));
}

// Which kernels answer a query of Q points (the outputs are the same bit for bit).  Eight lanes
// per query fill the chip with few queries but take a time proportional to K and to the cells'
// samples (64 samples, K = 8: 1.9 ns a query); the per-lane and the wave-shared kernels start at
// 150 to 400 us and add 0.5 to 2 ns a query, the wave-shared ones the least once a wave's queries
// share their cells.  us, eight lanes (the points sorted where the rule below sorts them) / per
// lane / wave, points at random in the box of the surface (those that arrive in order take
// eight lanes 140 to 320 us for 65,536):
//                          points    74 to 80 cells    313 cells        5,400 cells
//   RBF, m <= 32, K = 8    131,072  137 / 225 / 225  134 / 288 / 299  182 / 202 / 423
//                          196,608  241 / 272 / 255  249 / 312 / 320  244 / 247 / 418
//   RBF, m <= 64, K = 8     65,536  158 / 262 / 268  167 / 328 / 386  279 / 253 / 1084
//                          131,072  285 / 319 / 312  313 / 349 / 384  561 / 302 / 856
//                          196,608  413 / 386 / 374  420 / 424 / 433  428 / 361 / 736
//   RBF, m <= 64, K = 16   131,072  406 / 433 / 418  432 / 475 / 517  771 / 397 / 1056
//                          196,608  610 / 636 / 492  613 / 662 / 595  623 / 685 / 964
//   RBF, m <= 128, K = 8    65,536  475 / 418 / 450  716 / 499 / 754  963 / 481 / 2986
//                          131,072  643 / 621 / 569  641 / 632 / 712  682 / 654 / 2037
//                          196,608  923 / 791 / 702  912 / 815 / 818  965 / 872 / 1918
//   Matern, m <= 32         131,072  125 / 124 / 140  122 / 135 / 186  175 / 144 / 473
//                          196,608  216 / 151 / 168  216 / 152 / 202  226 / 164 / 443
//   Matern, m <= 64          65,536  148 / 134 / 187  164 / 148 / 258  275 / 170 / 1084
//                          131,072  279 / 176 / 211  319 / 189 / 299  559 / 208 / 894
//   Matern, m <= 128         49,152  341 / 235 / 381  479 / 263 / 638
//                          131,072  608 / 389 / 467  606 / 417 / 567
// and, past 196,608 points, in the room of 5.9k cells:
//                        1,000,000 along    1,000,003 at     2,097,152 grid   (lanes / wave)
//                        trajectories       random
//   RBF, K = 8, m <= 64       881 / 1402       961 / 1074      1670 / 1551
//   RBF, K = 16, m <= 64     1678 / 2180      1782 / 1858      3283 / 2872
//   Matern, m <= 64           812 / 1696       873 / 1339      1528 / 1892
//   RBF, K = 8, m <= 128     1545 / 1518      1570 / 1249      2765 / 1748
constexpr long GROUP_MOST_Q = 196608;
// Points per cell from which waves share their cells also in sets of up to GROUP_MOST_Q points
// (the Matern kernel's per-lane form is the shorter one up to 3,000 where cells end together)
bool dense(const ksdf_model* m, long Q) {
  return Q >= (m->kernel == KSDF_KERNEL_MATERN32 && m->max_m <= 64 ? 3072L : 1024L) * m->n_cells;
}
// Most points for eight lanes each: about where their time meets that of the others
long group_max_q(const ksdf_model* m, long Q) {
  if (m->kernel == KSDF_KERNEL_MATERN32) return m->max_m <= 32 ? 131072 : (m->max_m <= 64 ? 65536 : 57344);
  if (m->max_m <= 32) return GROUP_MOST_Q;
  if (m->max_m <= 64) return dense(m, Q) ? 147456 : GROUP_MOST_Q;
  return dense(m, Q) ? 98304 : 147456;
}
// Points per cell from which waves share their cells in larger sets: about 192 for the RBF and
// 384 for the Matern kernel, whose sums take longer, and 96 with cells over 64 samples, whose
// lanes end at unlike times
long wave_min_per_cell(const ksdf_model* m) {
  return m->max_m > 64 ? 96 : (m->kernel == KSDF_KERNEL_MATERN32 ? 384 : 192);
}
// The eight-lane kernel takes the queries in the caller's order up to this count: the sort
// costs 20 to 50 us, and saves what points at random lose by meeting their cells unsorted: 200
// us of 740 for 262,144 of them with 64 samples a cell, and with 128 samples 361 of 716 for
// 65,536 and 835 of 1476 for 131,072 (316 and 585 us for points that arrive in order).
long group_unsorted_max_q(const ksdf_model* m) { return m->max_m > 64 ? 65536 : 131072; }

bool pairs_used(const ksdf_model* m, long Q) {
  return m->tuning.query_split && m->tuning.query_pairs && query_pairs_usable(m, Q);
}
// the matrix-core pass 2 (wave-shared cells only)
bool mfma_used(const ksdf_model* m) {
  return m->tuning.query_split && m->tuning.query_mfma && !m->tuning.query_lanes && m->Linv32 &&
         m->max_m <= 64;
}
bool group_used(const ksdf_model* m, long Q) {
  return m->tuning.query_split && Q <= group_max_q(m, Q) && !mfma_used(m) && !pairs_used(m, Q);
}
bool lanes_used(const ksdf_model* m, long Q) {
  if (m->tuning.query_lanes) return true;
  if (mfma_used(m) || pairs_used(m, Q)) return false;
  // (K of 9 to 16 of the RBF: the per-lane form's registers leave too few waves in flight)
  if (Q <= GROUP_MOST_Q && (m->k_fuse <= 8 || m->kernel == KSDF_KERNEL_MATERN32) && !dense(m, Q)) return true;
  return Q < wave_min_per_cell(m) * m->n_cells;
}
bool sort_used(const ksdf_model* m, long Q) {
  return !group_used(m, Q) || Q > group_unsorted_max_q(m);
}
// limits of the sorts, checked for every launch so that a model beyond them is refused
// whatever the query count
int check_sorts(const ksdf_model* m) {
  if ((n_bins_of(m) + SCAN_TILE - 1) / SCAN_TILE > (long)SCAN_TILE) {
    set_error("query bucketing: too many bins");
    return KSDF_ERR_UNSUPPORTED;
  }
  if (m->tuning.query_split &&
      ((long)m->n_cells + 1 + SCAN_TILE - 1) / SCAN_TILE > (long)SCAN_TILE) {
    set_error("query: too many cells for the argmin regrouping");
    return KSDF_ERR_UNSUPPORTED;
  }
  return KSDF_OK;
}

size_t bucketing_bytes(const ksdf_model* m, long Q) {
  const long nb = n_bins_of(m);
  const long tiles = (nb + SCAN_TILE - 1) / SCAN_TILE;
  return align256(Q * sizeof(int)) * 2 + align256(nb * sizeof(int)) * 2 +
         align256(tiles * sizeof(int));
}

}  // namespace

// Counting sort of the queries by (index box, sub-box); sets A.perm.
int launch_bucketing(const ksdf_model* m, FastArgs& A, void* ws, hipStream_t s) {
  const long Q = A.Q;
  // workspace carve-up
  const long nb_max = n_bins_of(m), nb = n_bins_of(m, Q);
  char* w = static_cast<char*>(ws);
  int* keys = reinterpret_cast<int*>(w);
  w += align256(Q * sizeof(int));
  int* perm = reinterpret_cast<int*>(w);
  w += align256(Q * sizeof(int));
  int* counts = reinterpret_cast<int*>(w);
  w += align256(nb_max * sizeof(int));
  int* start = reinterpret_cast<int*>(w);
  w += align256(nb_max * sizeof(int));
  int* tsum = reinterpret_cast<int*>(w);
  // the places in the bins lie where the split query's records go later
  int* ranks = reinterpret_cast<int*>(static_cast<char*>(ws) + bucketing_bytes(m, Q));
  if (int r = check_sorts(m)) return r;
  const unsigned g1 = (unsigned)((Q + 255) / 256);
  hipLaunchKernelGGL(fill_kernel, dim3((unsigned)((nb + 255) / 256)), dim3(256), 0, s, counts, nb, 0);
  hipLaunchKernelGGL(bin_kernel, dim3(g1), dim3(256), 0, s, A, keys, ranks, counts, nb);
  launch_scan(counts, nb, tsum, start, s);
  hipLaunchKernelGGL(scatter_kernel, dim3(g1), dim3(256), 0, s, Q, keys, ranks, start, perm);
  A.perm = perm;
  return KSDF_OK;
}

size_t query_fast_workspace_bytes(const ksdf_model* m, long Q) {
  const long nc = (long)m->n_cells + 1;
  const long tiles = (nc + SCAN_TILE - 1) / SCAN_TILE;
  const bool pairs = pairs_used(m, Q);
  return bucketing_bytes(m, Q) + 2 * align256(Q * sizeof(P1Rec)) + 2 * align256(nc * sizeof(int)) +
         align256(tiles * sizeof(int)) + (pairs ? query_pairs_workspace_bytes(m, Q) : 0);
}

int launch_query_bucketing(const ksdf_model* m, const void* points, long Q, void* ws, hipStream_t s) {
  if (Q == 0) return KSDF_OK;
  if (!sort_used(m, Q)) return check_sorts(m);
  FastArgs A = make_fast_args(m, points, Q, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr,
                              nullptr, nullptr);
  return launch_bucketing(m, A, ws, s);
}

int launch_query_fast(const ksdf_model* m, const void* points, long Q, const int8_t* sign,
                      void* mean, void* grad, void* var, void* var_f, void* grad_var, int* argmin,
                      uint8_t* q_status, void* ws, size_t ws_bytes, hipStream_t s, bool prebucketed) {
  (void)ws_bytes;   // checked by the caller against query_workspace_bytes
  if (Q == 0) return KSDF_OK;
  FastArgs A = make_fast_args(m, points, Q, sign, mean, grad, var, var_f, grad_var, argmin, q_status);
  if (int r = check_sorts(m)) return r;
  if (!sort_used(m, Q)) {
    A.perm = nullptr;
  } else if (prebucketed) {
    A.perm = bucketed_perm(ws, Q);
  } else {
    int r = launch_bucketing(m, A, ws, s);
    if (r != KSDF_OK) return r;
  }
  timer_mark(m, KSDF_TIMER_QUERY, 0, s);
  if (group_used(m, Q)) {
    launch_query_group(m, A, s);
  } else if (m->tuning.query_split) {
    char* w = static_cast<char*>(ws) + bucketing_bytes(m, Q);
    A.rank = static_cast<int*>(ws);   // the sort's keys, no longer needed
    const long nc = (long)m->n_cells + 1;
    P1Rec* rec = reinterpret_cast<P1Rec*>(w);
    w += align256(Q * sizeof(P1Rec));
    P1Rec* rec2 = reinterpret_cast<P1Rec*>(w);
    w += align256(Q * sizeof(P1Rec));
    int* count = reinterpret_cast<int*>(w);
    w += align256(nc * sizeof(int));
    int* cursor = reinterpret_cast<int*>(w);
    w += align256(nc * sizeof(int));
    int* tsum = reinterpret_cast<int*>(w);
    w += align256(((nc + SCAN_TILE - 1) / SCAN_TILE) * sizeof(int));
    void* pws = pairs_used(m, Q) ? w : nullptr;
    const bool lane = lanes_used(m, Q);
    if (m->tuning.query_block == 64) {
      if (lane) launch_query_split_64_lane(m, A, rec, rec2, count, cursor, tsum, pws, s);
      else launch_query_split_64_wave(m, A, rec, rec2, count, cursor, tsum, pws, s);
    } else {
      if (lane) launch_query_split_256_lane(m, A, rec, rec2, count, cursor, tsum, pws, s);
      else launch_query_split_256_wave(m, A, rec, rec2, count, cursor, tsum, pws, s);
    }
  } else {
    launch_query_one(m, A, s);
  }
  timer_mark(m, KSDF_TIMER_QUERY, 1, s);
  KSDF_HIP_TRY(hipGetLastError());
  return KSDF_OK;
}

}  // namespace ksdf
