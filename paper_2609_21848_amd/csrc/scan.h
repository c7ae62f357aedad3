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

// Exclusive sums of n counts in place and their total (unless null), by one
// block: n is a number of chunks, a few thousand for 100 MB of input, so each
// thread takes a stretch of them.
constexpr int kScanThreads = 1024;
static __global__ __launch_bounds__(kScanThreads) void k_scan_counts(uint32_t* c, uint32_t n,
                                                                     unsigned long long* total) {
  __shared__ uint32_t sh[kScanThreads];
  const uint32_t tid = threadIdx.x;
  const uint32_t per = (n + kScanThreads - 1) / kScanThreads;
  const uint32_t b = min(n, tid * per), e = min(n, b + per);
  uint32_t sum = 0;
  for (uint32_t i = b; i < e; ++i) sum += c[i];
  sh[tid] = sum;
  __syncthreads();
  for (uint32_t d = 1; d < kScanThreads; d <<= 1) {
    const uint32_t x = tid >= d ? sh[tid - d] : 0u;
    __syncthreads();
    sh[tid] += x;
    __syncthreads();
  }
  uint32_t run = sh[tid] - sum;
  for (uint32_t i = b; i < e; ++i) {
    const uint32_t x = c[i];
    c[i] = run;
    run += x;
  }
  if (total && tid == kScanThreads - 1) *total = sh[tid];
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
