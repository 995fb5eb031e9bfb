// Wave-level helpers shared by the query and the backward.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

namespace ksdf {
namespace {

// f(integral_constant<int, I>) for I = B .. E-1, each index a compile-time constant
// (so that register arrays indexed by it are never placed in memory)
template <int B, int E, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

// LDS traffic between the lanes of one wave: order the writes before the reads.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Workgroups go to the chip's 8 XCDs (each with its own L2) in turn: workgroup i runs
// on XCD i mod 8.  The query kernels read the cells of neighbouring workgroups (a spatial
// bucket, or one argmin cell's run of records), so each XCD is given one contiguous
// range of the logical workgroups instead: a cell's samples and inverse then fill one
// L2, not eight.  The map is a bijection of [0, n); the results do not depend on it.
constexpr int N_XCD = 8;
__device__ __forceinline__ long xcd_block(long n) {
  const long i = blockIdx.x, q = n / N_XCD, r = n % N_XCD;
  const long x = i % N_XCD, k = i / N_XCD;
  return (x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q) + k;
}

// Wave-aggregated counting-sort steps over integer keys: the lanes that share
// a key take one atomic between them (the lowest lane issues it).
__device__ __forceinline__ void wave_count(int* count, int key, bool valid) {
  unsigned long long pending = __ballot(valid);
  const int lane = threadIdx.x & 63;
  while (pending) {
    const int leader = __ffsll((long long)pending) - 1;
    const int k = __builtin_amdgcn_readlane(key, leader);
    const unsigned long long mask = __ballot(valid && key == k);
    if (lane == leader) atomicAdd(count + k, (int)__popcll(mask));
    pending &= ~mask;
  }
}
// The same count, and each valid lane's place among the entries of its key (in no set order).
// The lanes that share a key are found first, without memory, and the lowest of each then
// issues its atomic in one instruction, so that a wave of unlike keys waits once (30 us a
// kernel for 64 of them one after the other).
__device__ __forceinline__ int wave_slot(int* count, int key, bool valid) {
  unsigned long long pending = __ballot(valid);
  const int lane = threadIdx.x & 63;
  int leader = lane, before = 0, n = 0;
  while (pending) {
    const int l = __ffsll((long long)pending) - 1;
    const int k = __builtin_amdgcn_readlane(key, l);
    const unsigned long long mask = __ballot(valid && key == k);
    if (valid && key == k) {
      leader = l;
      before = (int)__popcll(mask & ((1ull << lane) - 1ull));
      n = (int)__popcll(mask);
    }
    pending &= ~mask;
  }
  int base = 0;
  if (valid && leader == lane) base = atomicAdd(count + key, n);
  base = __shfl(base, leader, 64);
  return valid ? base + before : -1;
}

}  // namespace
}  // namespace ksdf
