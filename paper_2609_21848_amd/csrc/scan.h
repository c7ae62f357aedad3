// Helpers of the kernels that work chunk by chunk: a pass that counts per
// chunk, a scan of the counts, and a pass that writes each chunk at its place.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace dbbc {

// Word arrays carved out of one allocation.
struct Carve {
  uint32_t* p = nullptr;
  size_t used = 0;
  static size_t round(size_t words) { return (words + 63) / 64 * 64; }
  uint32_t* take(size_t words) {
    uint32_t* q = p ? p + used : nullptr;
    used += round(words);
    return q;
  }
};

// Exclusive sums of p[0 .. n) in place, by one block of kScanThreads; returns
// the total (in every thread).  n is a number of chunks, some ten thousands
// at most as a rule: tiles of kScanPer elements a thread, whole lines each.
constexpr int kScanThreads = 1024;
constexpr uint32_t kScanPer = 8;

template <class T>
__device__ __forceinline__ T scan_block(T* p, uint32_t n) {
  __shared__ T wsum[kScanThreads / 64];
  const int lane = static_cast<int>(threadIdx.x) & 63, wave = static_cast<int>(threadIdx.x) >> 6;
  T run = 0;
  for (uint32_t t0 = 0; t0 < n; t0 += kScanThreads * kScanPer) {
    const uint32_t i0 = t0 + threadIdx.x * kScanPer;
    T v[kScanPer];
    T sum = 0;
#pragma unroll
    for (uint32_t j = 0; j < kScanPer; ++j) {
      v[j] = i0 + j < n ? p[i0 + j] : T{0};
      sum += v[j];
    }
    T x = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const T up = __shfl_up(x, d, 64);
      if (lane >= d) x += up;
    }
    if (lane == 63) wsum[wave] = x;
    __syncthreads();
    T before = run, all = 0;
#pragma unroll
    for (int w = 0; w < kScanThreads / 64; ++w) {
      before += w < wave ? wsum[w] : T{0};
      all += wsum[w];
    }
    __syncthreads();
    before += x - sum;
#pragma unroll
    for (uint32_t j = 0; j < kScanPer; ++j) {
      if (i0 + j < n) p[i0 + j] = before;
      before += v[j];
    }
    run += all;
  }
  return run;
}

// The same of one sequence of counts; the total to *total unless null.
static __global__ __launch_bounds__(kScanThreads) void k_scan_counts(uint32_t* c, uint32_t n,
                                                                     unsigned long long* total) {
  const uint32_t all = scan_block(c, n);
  if (total && threadIdx.x == 0) *total = all;
}

inline hipError_t scan_counts(uint32_t* c, uint32_t n, unsigned long long* total, hipStream_t st) {
  hipLaunchKernelGGL(k_scan_counts, dim3(1), dim3(kScanThreads), 0, st, c, n, total);
  return hipGetLastError();
}

// A block's exclusive sum of v over its threads (kT of them, whole
// wavefronts), and the block's total; sh holds kT / 64 + 1 words.
template <int kT>
__device__ __forceinline__ uint32_t block_excl(uint32_t v, uint32_t* sh, uint32_t& total) {
  const int lane = static_cast<int>(threadIdx.x) & 63, wave = static_cast<int>(threadIdx.x) >> 6;
  uint32_t x = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t up = __shfl_up(x, d, 64);
    if (lane >= d) x += up;
  }
  __syncthreads();
  if (lane == 63) sh[wave] = x;
  __syncthreads();
  uint32_t before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < kT / 64; ++w) {
    before += w < wave ? sh[w] : 0u;
    all += sh[w];
  }
  total = all;
  return before + x - v;
}

}  // namespace dbbc
