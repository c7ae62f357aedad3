// A stable least-significant-digit radix sort for the graph build, the text
// ingestion and the planner: one histogram launch per sort, one launch per
// digit.  Elements are W 32-bit words, the key the first one or two; the
// first pass reads them through a caller's functor (so keys are formed from
// the input arrays, not written and read back) and the last pass hands each
// element with its final position to another (so the sorted order's arrays
// are written by the sort itself).
//
// A pass handles tiles of kTile elements, in the order of a ticket counter:
//   1. every wavefront ranks its elements of one digit with ballots (the
//      lanes of equal digit) over a running count per digit in LDS, in
//      element order, so the sort is stable;
//   2. the tile's count of each digit is published, and the counts of the
//      tiles before it are added up from their published words (a tile's own
//      count, or its inclusive sum once known: decoupled look-back, four
//      predecessors read at a time).  Tiles start in ticket order, so every
//      tile that is waited for is running or done, and the first publishes
//      its inclusive sum at once: each wait ends;
//   3. the tile is put in digit order in LDS, and written out run by run.
// Bound by memory: two accesses per element and pass, runs of
// kTile / 2^bits elements per digit.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "kernels.h"

namespace dbbc {
namespace radix {

constexpr int kDigits = 256;
constexpr int kMaxPasses = 8;
// Tile shapes: large inputs take 4,096-element tiles (long runs per digit);
// below kSmallN elements 1,024-element tiles, so that more CUs share them.
constexpr int kThreadsL = 512, kItemsL = 8;
constexpr int kThreadsS = 256, kItemsS = 4;
constexpr int64_t kSmallN = int64_t{1} << 20;

template <int W>
struct Elt {
  uint32_t w[W];
};

template <int KW, int W>
__device__ __forceinline__ uint64_t key_of(const Elt<W>& e) {
  if constexpr (KW == 2)
    return (static_cast<uint64_t>(e.w[1]) << 32) | e.w[0];
  else
    return e.w[0];
}

// W arrays of words: a sort's buffer between passes.
template <int W>
struct Soa {
  uint32_t* p[W];
  __device__ __forceinline__ Elt<W> load(uint32_t i) const {
    Elt<W> e;
#pragma unroll
    for (int k = 0; k < W; ++k) e.w[k] = p[k][i];
    return e;
  }
  __device__ __forceinline__ void store(uint32_t i, const Elt<W>& e) const {
#pragma unroll
    for (int k = 0; k < W; ++k) p[k][i] = e.w[k];
  }
};

// The passes of a sort, lowest digit first.
struct Digits {
  int passes = 0;
  int shift[kMaxPasses] = {};
  int bits[kMaxPasses] = {};
};
// Adds the passes of a key's bits [begin, end): of equal width, at most 8 bits.
inline void add_digits(Digits& d, int begin, int end) {
  const int n = std::max(1, end - begin), k = (n + 7) / 8;
  for (int p = 0; p < k; ++p) {
    const int lo = begin + n * p / k, hi = begin + n * (p + 1) / k;
    d.shift[d.passes] = lo;
    d.bits[d.passes++] = hi - lo;
  }
}
inline Digits digits_of(int begin, int end) {
  Digits d;
  add_digits(d, begin, end);
  return d;
}

inline int64_t tiles_of(int64_t n) {
  const int64_t t = n < kSmallN ? kThreadsS * kItemsS : kThreadsL * kItemsL;
  return (n + t - 1) / t;
}

// A tile's published word per digit: a count with two flag bits on top (0 not
// yet, 1 the tile's own count, 2 its inclusive sum).  Counts are at most n,
// so 32-bit words do below 2^30 elements.
template <class S>
struct Word {
  static constexpr int kFlag = 8 * sizeof(S) - 2;
  static constexpr S kCount = (S{1} << kFlag) - 1;
};
inline bool narrow(int64_t n) { return n < (int64_t{1} << 30); }

// 64-bit words of control memory of a sort (all zero before its histogram):
// the digit counts and the ticket counter of every pass, then the tiles'
// published words.
constexpr size_t kHistWords = kMaxPasses * kDigits / 2;
inline size_t control_words(int64_t n, const Digits& d) {
  const size_t words = static_cast<size_t>(d.passes) * static_cast<size_t>(tiles_of(n)) * kDigits;
  return kHistWords + kMaxPasses / 2 + (narrow(n) ? (words + 1) / 2 : words);
}
// The most words that a sort of up to n elements needs.
inline size_t control_bound(int64_t n, const Digits& d) {
  return std::max(control_words(n, d), control_words(std::min(n, kSmallN - 1), d));
}
struct Control {
  unsigned long long* w = nullptr;
  uint32_t* hist(int pass) const { return reinterpret_cast<uint32_t*>(w) + pass * kDigits; }
  uint32_t* ticket(int pass) const { return reinterpret_cast<uint32_t*>(w + kHistWords) + pass; }
  template <class S>
  S* state(int pass, int64_t tiles) const {
    return reinterpret_cast<S*>(w + kHistWords + kMaxPasses / 2) +
           static_cast<size_t>(pass) * static_cast<size_t>(tiles) * kDigits;
  }
};

constexpr int kHistThreads = 256;

// Add one to a digit's LDS counter for every active lane: one add for the
// wavefront where all its lanes share the digit (the high digits of most
// inputs).
__device__ __forceinline__ void count_digit(uint32_t* h, uint32_t g) {
  const uint32_t g0 = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(g)));
  const uint64_t act = __ballot(1);
  if (__ballot(g == g0) == act) {
    if (static_cast<int>(threadIdx.x & 63) == __builtin_ctzll(act))
      atomicAdd(&h[g], static_cast<uint32_t>(__popcll(act)));
  } else {
    atomicAdd(&h[g], 1u);
  }
}
__device__ __forceinline__ void count_digits(uint32_t* h, uint64_t key, const Digits& d) {
  for (int p = 0; p < d.passes; ++p)
    count_digit(h + p * kDigits, static_cast<uint32_t>(key >> d.shift[p]) & ((1u << d.bits[p]) - 1u));
}

// A block's digit counts: LDS counters, cleared and then added to the sort's.
__device__ __forceinline__ void clear_counts(uint32_t* h, const Digits& d) {
  for (int i = threadIdx.x; i < d.passes * kDigits; i += blockDim.x) h[i] = 0;
  __syncthreads();
}
__device__ __forceinline__ void add_counts(const uint32_t* h, const Digits& d, uint32_t* hist) {
  __syncthreads();
  for (int i = threadIdx.x; i < d.passes * kDigits; i += blockDim.x)
    if (h[i]) atomicAdd(&hist[i], h[i]);
}

// Digit counts of every pass.
template <int KW, class In>
__global__ __launch_bounds__(kHistThreads) void k_hist(In in, uint32_t n, Digits d, uint32_t* hist) {
  __shared__ uint32_t h[kMaxPasses * kDigits];
  clear_counts(h, d);
  // four independent loads at a time
  const uint64_t stride = gridDim.x * kHistThreads;
  for (uint64_t i = blockIdx.x * kHistThreads + threadIdx.x; i < n; i += 4 * stride) {
    uint64_t key[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (i + k * stride < n) key[k] = key_of<KW>(in.load(static_cast<uint32_t>(i + k * stride)));
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (i + k * stride < n) count_digits(h, key[k], d);
  }
  add_counts(h, d, hist);
}

// Exclusive sums of a and b over the threads of a block's first four
// wavefronts (the 256 digits); every thread of the block calls it.
__device__ __forceinline__ void scan_digits(uint32_t& a, uint32_t& b, uint32_t* sh) {
  const int tid = static_cast<int>(threadIdx.x), lane = tid & 63, wave = tid >> 6;
  uint32_t x = a, y = b;
#pragma unroll
  for (int s = 1; s < 64; s <<= 1) {
    const uint32_t ux = __shfl_up(x, s, 64), uy = __shfl_up(y, s, 64);
    if (lane >= s) {
      x += ux;
      y += uy;
    }
  }
  if (wave < 4 && lane == 63) {
    sh[wave] = x;
    sh[4 + wave] = y;
  }
  __syncthreads();
  if (wave < 4) {
    for (int w = 0; w < wave; ++w) {
      x += sh[w];
      y += sh[4 + w];
    }
    a = x - a;
    b = y - b;
  }
}

template <int KW, int W, class S, int kThreads, int kItems, class In, class Out>
__global__ __launch_bounds__(kThreads) void k_pass(In in, Out out, uint32_t n, int shift, int bits,
                                                   const uint32_t* hist, S* state, uint32_t* ticket) {
  constexpr int kFlag = Word<S>::kFlag;
  constexpr int kWaves = kThreads / 64;
  constexpr uint32_t kTile = kThreads * kItems;
  static_assert(kThreads >= kDigits, "a thread per digit");
  __shared__ uint32_t whist[kWaves][kDigits];
  __shared__ uint32_t tstart[kDigits], gbase[kDigits];
  __shared__ uint32_t sh[8];
  __shared__ uint32_t tile_sh;
  __shared__ uint32_t buf[W][kTile];
  const int tid = static_cast<int>(threadIdx.x), lane = tid & 63, wave = tid >> 6;
  if (tid == 0) tile_sh = atomicAdd(ticket, 1u);
  for (int i = tid; i < kWaves * kDigits; i += kThreads) (&whist[0][0])[i] = 0;
  __syncthreads();
  const uint32_t tile = tile_sh;
  const uint32_t base = tile * kTile;
  const uint32_t cnt = min(kTile, n - base);
  const uint32_t mask = (1u << bits) - 1u;
  const uint32_t i0 = static_cast<uint32_t>(wave * 64 * kItems + lane);
  Elt<W> e[kItems];
  uint32_t rank[kItems], dig[kItems];
#pragma unroll
  for (int j = 0; j < kItems; ++j)
    if (i0 + j * 64 < cnt) e[j] = in.load(base + i0 + j * 64);
  const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const bool valid = i0 + j * 64 < cnt;
    const uint32_t d = valid ? static_cast<uint32_t>(key_of<KW>(e[j]) >> shift) & mask : 0u;
    uint64_t peers = __ballot(valid);
    for (int b = 0; b < bits; ++b) {
      const bool one = (d >> b) & 1u;
      const uint64_t m = __ballot(one);
      peers &= one ? m : ~m;
    }
    const uint32_t lower = static_cast<uint32_t>(__popcll(peers & below));
    const uint32_t old = whist[wave][d];
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    if (valid && lower == 0) whist[wave][d] = old + static_cast<uint32_t>(__popcll(peers));
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    dig[j] = d;
    rank[j] = old + lower;
  }
  __syncthreads();
  // per digit (one thread each): the wavefronts' offsets, the tile's count
  uint32_t total = 0, first = 0;
  if (tid < kDigits) {
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const uint32_t c = whist[w][tid];
      whist[w][tid] = total;
      total += c;
    }
    first = hist[tid];
    __hip_atomic_store(&state[static_cast<size_t>(tile) * kDigits + tid], (S{tile == 0 ? 2u : 1u} << kFlag) | S{total},
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  uint32_t start = total;
  scan_digits(start, first, sh);
  if (tid < kDigits) {
    S excl = 0;
    int64_t t = static_cast<int64_t>(tile) - 1;
    while (t >= 0) {
      S s[4];
#pragma unroll
      for (int k = 0; k < 4; ++k)
        s[k] = __hip_atomic_load(&state[static_cast<size_t>(t - k > 0 ? t - k : 0) * kDigits + tid], __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_AGENT);
      bool done = false;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (done || t < 0 || (s[k] >> kFlag) == 0) {
          // the sum is whole, or this predecessor has not published yet:
          // read again from it
          break;
        }
        excl += s[k] & Word<S>::kCount;
        done = (s[k] >> kFlag) == 2;
        --t;
      }
      if (done) break;
    }
    if (tile > 0)
      __hip_atomic_store(&state[static_cast<size_t>(tile) * kDigits + tid], (S{2} << kFlag) | (excl + S{total}),
                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    tstart[tid] = start;
    gbase[tid] = first + static_cast<uint32_t>(excl) - start;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    if (i0 + j * 64 < cnt) {
      const uint32_t at = tstart[dig[j]] + whist[wave][dig[j]] + rank[j];
#pragma unroll
      for (int k = 0; k < W; ++k) buf[k][at] = e[j].w[k];
    }
  }
  __syncthreads();
  for (uint32_t i = tid; i < cnt; i += kThreads) {
    Elt<W> x;
#pragma unroll
    for (int k = 0; k < W; ++k) x.w[k] = buf[k][i];
    const uint32_t d = static_cast<uint32_t>(key_of<KW>(x) >> shift) & mask;
    out.store(gbase[d] + i, x);
  }
}

// Digit counts of a sort's every pass, into c (control memory, zero).
// (At the end every block adds its counts to the same words, about 10 ns
// each: 16 elements per thread and at most 1,024 blocks keep that short.)
inline int hist_grid(int64_t n) {
  return static_cast<int>(std::max<int64_t>(1, std::min<int64_t>(n / (16 * kHistThreads), 1024)));
}
template <int KW, class In>
hipError_t histogram(In in, int64_t n, const Digits& d, const Control& c, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const int grid = hist_grid(n);
  hipLaunchKernelGGL((k_hist<KW, In>), dim3(grid), dim3(kHistThreads), 0, st, in, static_cast<uint32_t>(n), d,
                     c.hist(0));
  return hipGetLastError();
}

template <int KW, int W, class S, int kThreads, int kItems, class In, class Out>
hipError_t pass_as(In in, Out out, int64_t n, const Digits& d, int p, const Control& c, hipStream_t st) {
  const int64_t tiles = tiles_of(n);
  hipLaunchKernelGGL((k_pass<KW, W, S, kThreads, kItems, In, Out>), dim3(static_cast<unsigned>(tiles)), dim3(kThreads),
                     0, st, in, out, static_cast<uint32_t>(n), d.shift[p], d.bits[p], c.hist(p),
                     c.state<S>(p, tiles), c.ticket(p));
  return hipGetLastError();
}

// One pass (p of d) of n elements, in -> out.
template <int KW, int W, class In, class Out>
hipError_t pass(In in, Out out, int64_t n, const Digits& d, int p, const Control& c, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  if (n < kSmallN) return pass_as<KW, W, uint32_t, kThreadsS, kItemsS>(in, out, n, d, p, c, st);
  if (narrow(n)) return pass_as<KW, W, uint32_t, kThreadsL, kItemsL>(in, out, n, d, p, c, st);
  return pass_as<KW, W, unsigned long long, kThreadsL, kItemsL>(in, out, n, d, p, c, st);
}

// A sort of n elements whose digit counts are in c: pass 0 reads in, the last
// pass writes out; those between go through buf[0], buf[1] in turn (pass p
// writes buf[p & 1]).
template <int KW, int W, class In, class Out>
hipError_t passes(In in, Out out, const Soa<W> (&buf)[2], int64_t n, const Digits& d, const Control& c,
                  hipStream_t st) {
  for (int p = 0; p < d.passes; ++p) {
    const bool last = p + 1 == d.passes;
    hipError_t e;
    if (p == 0)
      e = last ? pass<KW, W>(in, out, n, d, p, c, st) : pass<KW, W>(in, buf[0], n, d, p, c, st);
    else
      e = last ? pass<KW, W>(buf[(p - 1) & 1], out, n, d, p, c, st)
               : pass<KW, W>(buf[(p - 1) & 1], buf[p & 1], n, d, p, c, st);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace radix
}  // namespace dbbc
