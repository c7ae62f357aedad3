// Device construction of the priority-ordered CSR pair (Definition 3 relabel,
// the paper's Phase 2 "global index" on one device) with the per-entry
// reverse positions that let a wedge walk start without a search, and the
// closed-form VP wedge count.  Everything is ordered by radix sorts (radix.h)
// whose passes read the input records and write the graph's arrays
// themselves; an entry is moved by sequential streams except where a
// position in the other CSR has to be stored (one 4-byte scatter).
//   1. last-wins dedup: records sorted by (u, v), stable, so the last record
//      of a run of equal pairs is the one kept.  Degrees are the run lengths
//      of the sorted keys: U's in the final order, V's in the order after the
//      passes over the v bits (or from a sort of the kept records' v alone
//      when there are duplicates), with no counters;
//   2. all vertices sorted by (degree desc, global id desc): global ranks.  A
//      side's rank is its place among its own vertices in that order, so one
//      sort and one scan give both sides' ranks, input ids and row offsets;
//   3. the kept records, moved row by row into U rank order (they are sorted
//      by u already), are sorted by the V rank alone: the V-side CSR, rows by
//      V rank and neighbours by U rank; those, sorted by the U rank alone,
//      are the U-side CSR.
// Measured on 50M records (5M x 2M vertices): the build 32.8 ms before
// (atomic degree counters 4.4, two sorts of 64-bit (rank, rank) keys formed
// and filled by random gathers 14.3, reverse positions 5.1, W_VP walked per
// entry 4.5).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <string>
#include <vector>

#include "build_dev.h"
#include "kernels.h"
#include "radix.h"
#include "scan.h"

namespace dbbc {
namespace {

constexpr int kThreads = 256;

int grid_for(int64_t n) {
  return static_cast<int>(std::max<int64_t>(1, std::min<int64_t>((n + kThreads - 1) / kThreads, 1 << 16)));
}

#define GRID_STRIDE(i, n)                                                                    \
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < (n); \
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)

// Bits needed for the values 0 .. n - 1 (at least 1).
int bits_for(int64_t n) {
  int b = 1;
  while ((int64_t{1} << b) < n) ++b;
  return b;
}

// ---- step 1: records to sorted pairs, degrees ----------------------------------

// A record as a sort element: key (u << vbits) | v, then (index << 1) | negative.
struct RecordIn {
  const int32_t* u;
  const int32_t* v;
  const int8_t* s;
  int vbits;
  __device__ __forceinline__ uint64_t key(int32_t a, int32_t b) const {
    return (static_cast<uint64_t>(static_cast<uint32_t>(a)) << vbits) | static_cast<uint32_t>(b);
  }
  __device__ __forceinline__ radix::Elt<3> load(uint32_t i) const {
    const uint64_t key = this->key(u[i], v[i]);
    return {{static_cast<uint32_t>(key), static_cast<uint32_t>(key >> 32), (i << 1) | (s[i] < 0 ? 1u : 0u)}};
  }
};

__device__ __forceinline__ uint64_t key_at(const radix::Soa<3>& a, uint32_t i) {
  return (static_cast<uint64_t>(a.p[1][i]) << 32) | a.p[0][i];
}

// The sort's digit counts, and the smallest bad record per kind: bad[0] an id
// out of range, bad[1] a sign other than +1 / -1.
__global__ __launch_bounds__(kThreads) void k_record_hist(RecordIn in, uint32_t m, int32_t n_u, int32_t n_v,
                                                          radix::Digits d, uint32_t* hist, unsigned long long* bad) {
  __shared__ uint32_t h[radix::kMaxPasses * radix::kDigits];
  radix::clear_counts(h, d);
  // four records' loads at a time
  const uint64_t stride = static_cast<uint64_t>(gridDim.x) * kThreads;
  for (uint64_t i = static_cast<uint64_t>(blockIdx.x) * kThreads + threadIdx.x; i < m; i += 4 * stride) {
    int32_t a[4], b[4];
    int8_t g[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint64_t j = i + k * stride;
      if (j < m) {
        a[k] = in.u[j];
        b[k] = in.v[j];
        g[k] = in.s[j];
      }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint64_t j = i + k * stride;
      if (j >= m) continue;
      if (a[k] < 0 || a[k] >= n_u || b[k] < 0 || b[k] >= n_v)
        atomicMin(&bad[0], static_cast<unsigned long long>(j));
      if (g[k] != 1 && g[k] != -1) atomicMin(&bad[1], static_cast<unsigned long long>(j));
      radix::count_digits(h, in.key(a[k], b[k]), d);
    }
  }
  radix::add_counts(h, d, hist);
}

// A vertex's run in a sorted order: its first position and the one past its
// last (both 0 for a vertex without records).
struct Runs {
  uint32_t* start;
  uint32_t* end;
  int32_t n;
  // position i holds vertex x; the neighbours' vertices differ where the flags say
  __device__ __forceinline__ void mark(uint32_t i, uint32_t x, bool head, bool tail) const {
    if (x >= static_cast<uint32_t>(n)) return;  // an unchecked record: the build ends in an error
    if (head) start[x] = i;
    if (tail) end[x] = i + 1;
  }
};

// Runs of equal v (the low vbits of the key's first word) of elements
// grouped by v.
__global__ void k_runs_v(const uint32_t* w0, uint32_t m, uint32_t vmask, Runs r) {
  GRID_STRIDE(i64, m) {
    const uint32_t i = static_cast<uint32_t>(i64);
    const uint32_t x = w0[i] & vmask;
    r.mark(i, x, i == 0 || (w0[i - 1] & vmask) != x, i + 1 == m || (w0[i + 1] & vmask) != x);
  }
}

// Runs of equal u of the sorted pairs, and the number of records that a
// later one of the same pair replaces.
__global__ __launch_bounds__(kThreads) void k_runs_u(radix::Soa<3> a, uint32_t m, int vbits, Runs r,
                                                     unsigned long long* dups) {
  unsigned long long d = 0;
  GRID_STRIDE(i64, m) {
    const uint32_t i = static_cast<uint32_t>(i64);
    const uint64_t k = key_at(a, i);
    const uint64_t prev = i > 0 ? key_at(a, i - 1) : 0, next = i + 1 < m ? key_at(a, i + 1) : 0;
    const uint32_t x = static_cast<uint32_t>(k >> vbits);
    r.mark(i, x, i == 0 || static_cast<uint32_t>(prev >> vbits) != x,
           i + 1 == m || static_cast<uint32_t>(next >> vbits) != x);
    d += (i + 1 < m && next == k) ? 1 : 0;
  }
#pragma unroll
  for (int w = 32; w > 0; w >>= 1) d += __shfl_xor(d, w, 64);
  if ((threadIdx.x & 63) == 0 && d) atomicAdd(dups, d);
}

// Duplicates dropped: the last record of each run of equal pairs moves to
// its place among the kept ones.  A block takes kKeepChunk records; pass 0
// counts each block's, pass 1 (after a scan of the counts) moves them.
constexpr uint32_t kKeepChunk = 8 * kThreads;

template <int kPass>
__global__ __launch_bounds__(kThreads) void k_keep(radix::Soa<3> a, uint32_t m, uint32_t* counts, radix::Soa<3> out) {
  __shared__ uint32_t sh[kThreads / 64];
  const uint32_t c0 = blockIdx.x * kKeepChunk;
  uint32_t done = 0;
  const uint32_t at = kPass ? counts[blockIdx.x] : 0u;
  for (uint32_t j = 0; j < kKeepChunk; j += kThreads) {
    const uint32_t i = c0 + j + threadIdx.x;
    const bool keep = i < m && (i + 1 == m || key_at(a, i) != key_at(a, i + 1));
    uint32_t all;
    const uint32_t before = block_excl<kThreads>(keep ? 1u : 0u, sh, all);
    if (kPass && keep) out.store(at + done + before, a.load(i));
    done += all;
  }
  if (!kPass && threadIdx.x == 0) counts[blockIdx.x] = done;
}

// The kept records' v as a keys-only sort's input (the key's low bits).
struct VertexIn {
  const uint32_t* w0;
  uint32_t mask;
  __device__ __forceinline__ radix::Elt<1> load(uint32_t i) const { return {{w0[i] & mask}}; }
};

// ---- step 2: ranks -------------------------------------------------------------

// Vertices in descending global id (x for U, n_u + y for V), keyed by the
// complement of their degree: a stable sort gives (degree desc, id desc).
struct RankIn {
  const uint32_t *su, *eu, *sv, *ev;  // run starts and ends per side
  uint32_t n_u, n, top;
  __device__ __forceinline__ radix::Elt<2> load(uint32_t i) const {
    const uint32_t gid = n - 1 - i;
    const uint32_t d = gid < n_u ? eu[gid] - su[gid] : ev[gid - n_u] - sv[gid - n_u];
    return {{top - d, gid}};
  }
};

// One block takes kRankChunk places of the global order.  Pass 0 sums each
// chunk's U vertices and both sides' degrees; pass 1 adds up the chunks
// before its own and writes, by side rank: input id, global rank and row
// offset; and the side rank of every input id.  (With one chunk, pass 1 is
// all.)
constexpr int kRankPer = 8;
constexpr uint32_t kRankChunk = kThreads * kRankPer;

struct RankSums {
  uint32_t nu, du, dv, pad;
};
struct RankOut {
  int32_t* ord[2];
  int32_t* sr[2];
  int32_t* grank[2];
  uint32_t* off[2];
};

__device__ __forceinline__ RankSums operator+(const RankSums& a, const RankSums& b) {
  return RankSums{a.nu + b.nu, a.du + b.du, a.dv + b.dv, 0};
}
__device__ __forceinline__ RankSums wave_up(const RankSums& a, int d) {
  return RankSums{__shfl_up(a.nu, d, 64), __shfl_up(a.du, d, 64), __shfl_up(a.dv, d, 64), 0};
}

template <int kPass>
__global__ __launch_bounds__(kThreads) void k_ranks(radix::Soa<2> sorted, uint32_t n, uint32_t n_u, uint32_t top,
                                                    uint32_t me, RankSums* chunks, RankOut o) {
  __shared__ RankSums sh[kThreads / 64 + 1];
  const int tid = static_cast<int>(threadIdx.x), lane = tid & 63, wave = tid >> 6;
  const uint32_t r0 = blockIdx.x * kRankChunk + tid * kRankPer;
  uint32_t deg[kRankPer], gid[kRankPer];
  RankSums t{0, 0, 0, 0};
#pragma unroll
  for (int j = 0; j < kRankPer; ++j) {
    const bool in = r0 + j < n;
    deg[j] = in ? top - sorted.p[0][r0 + j] : 0u;
    gid[j] = in ? sorted.p[1][r0 + j] : 0u;
    const bool is_u = in && gid[j] < n_u;
    t = t + RankSums{is_u ? 1u : 0u, is_u ? deg[j] : 0u, is_u ? 0u : deg[j], 0};
  }
  RankSums x = t;  // inclusive over the wavefront
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const RankSums up = wave_up(x, d);
    if (lane >= d) x = x + up;
  }
  if (lane == 63) sh[wave] = x;
  RankSums base{0, 0, 0, 0};
  if (kPass) {  // the chunks before this one
    RankSums c{0, 0, 0, 0};
    for (uint32_t i = tid; i < blockIdx.x; i += kThreads) c = c + chunks[i];
#pragma unroll
    for (int d = 32; d > 0; d >>= 1)
      c = c + RankSums{__shfl_xor(c.nu, d, 64), __shfl_xor(c.du, d, 64), __shfl_xor(c.dv, d, 64), 0};
    __shared__ RankSums before[kThreads / 64];
    if (lane == 0) before[wave] = c;
    __syncthreads();
    for (int w = 0; w < kThreads / 64; ++w) base = base + before[w];
  } else {
    __syncthreads();
  }
  if (!kPass) {
    if (tid == 0) {
      RankSums c{0, 0, 0, 0};
      for (int w = 0; w < kThreads / 64; ++w) c = c + sh[w];
      chunks[blockIdx.x] = c;
    }
    return;
  }
  for (int w = 0; w < wave; ++w) base = base + sh[w];
  RankSums run = base + RankSums{x.nu - t.nu, x.du - t.du, x.dv - t.dv, 0};
#pragma unroll
  for (int j = 0; j < kRankPer; ++j) {
    const uint32_t r = r0 + j;
    if (r >= n) break;
    if (gid[j] < n_u) {
      const uint32_t k = run.nu;
      o.ord[0][k] = static_cast<int32_t>(gid[j]);
      o.sr[0][gid[j]] = static_cast<int32_t>(k);
      o.grank[0][k] = static_cast<int32_t>(r);
      o.off[0][k] = run.du;
      ++run.nu;
      run.du += deg[j];
    } else {
      const uint32_t k = r - run.nu, y = gid[j] - n_u;
      o.ord[1][k] = static_cast<int32_t>(y);
      o.sr[1][y] = static_cast<int32_t>(k);
      o.grank[1][k] = static_cast<int32_t>(r);
      o.off[1][k] = run.dv;
      run.dv += deg[j];
    }
    if (r + 1 == n) {
      o.off[0][n_u] = me;
      o.off[1][n - n_u] = me;
    }
  }
}

// Digit counts of the entries' row ranks, from the row offsets: a pass's
// digit is constant over stretches of 2^shift rows, whose entries are a
// difference of two offsets.  Consecutive stretches have consecutive digits
// (no two lanes of an add share a counter).
__global__ __launch_bounds__(kThreads) void k_row_hist(const uint32_t* off, uint32_t n, radix::Digits d,
                                                       uint32_t* hist) {
  __shared__ uint32_t h[radix::kMaxPasses * radix::kDigits];
  radix::clear_counts(h, d);
  for (int p = 0; p < d.passes; ++p) {
    const int sh = d.shift[p];
    const int64_t stretches = static_cast<int64_t>((static_cast<uint64_t>(n) + (1ull << sh) - 1) >> sh);
    GRID_STRIDE(j, stretches) {
      const uint64_t lo = static_cast<uint64_t>(j) << sh;
      const uint64_t hi = min(static_cast<uint64_t>(n), lo + (1ull << sh));
      const uint32_t c = off[hi] - off[lo];
      if (c) atomicAdd(&h[p * radix::kDigits + (static_cast<uint32_t>(j) & ((1u << d.bits[p]) - 1u))], c);
    }
  }
  radix::add_counts(h, d, hist);
}

// ---- step 3: the two CSRs -------------------------------------------------------

// The kept records into U rank order: record i of vertex u, the j-th of its
// run, goes to place off[rank of u] + j, as (V rank, U rank, index | sign).
__global__ void k_place(radix::Soa<3> a, uint32_t me, int vbits, const uint32_t* start_u, const int32_t* sr_u,
                        const int32_t* sr_v, const uint32_t* off_u, radix::Soa<3> out) {
  const uint32_t vmask = (1u << vbits) - 1u;
  GRID_STRIDE(i64, me) {
    const uint32_t i = static_cast<uint32_t>(i64);
    const uint64_t k = key_at(a, i);
    const uint32_t u = static_cast<uint32_t>(k >> vbits);
    const uint32_t x = static_cast<uint32_t>(sr_u[u]);
    out.store(off_u[x] + (i - start_u[u]),
              radix::Elt<3>{{static_cast<uint32_t>(sr_v[static_cast<uint32_t>(k) & vmask]), x, a.p[2][i]}});
  }
}

// The V-side CSR from the sort by V rank: entry words, and what the next
// sort needs of every position (its row and record).
struct VOut {
  uint32_t* adj;
  uint32_t* row;
  uint32_t* rec;
  __device__ __forceinline__ void store(uint32_t q, const radix::Elt<3>& e) const {
    adj[q] = (e.w[1] << 1) | (e.w[2] & 1u);
    row[q] = e.w[0];
    rec[q] = e.w[2] >> 1;
  }
};

// ... read back as (U rank, V rank | sign, record, V position).
struct VIn {
  const uint32_t* adj;
  const uint32_t* row;
  const uint32_t* rec;
  __device__ __forceinline__ radix::Elt<4> load(uint32_t q) const {
    const uint32_t w = adj[q];
    return {{w >> 1, (row[q] << 1) | (w & 1u), rec[q], q}};
  }
};

// The U-side CSR from the sort by U rank, and both sides' reverse positions:
// an edge's place in the other side's row.
struct UOut {
  uint32_t* adj;
  uint32_t* rec;
  int32_t* rev_u;
  int32_t* rev_v;
  const uint32_t* off_u;
  const uint32_t* off_v;
  __device__ __forceinline__ void store(uint32_t k, const radix::Elt<4>& e) const {
    adj[k] = e.w[1];
    rec[k] = e.w[2];
    rev_u[k] = static_cast<int32_t>(e.w[3] - off_v[e.w[1] >> 1]);
    rev_v[e.w[3]] = static_cast<int32_t>(k - off_u[e.w[0]]);
  }
};

// Per row of both sides (side 0's rows first): cut[x], the neighbours of
// higher priority (a prefix of the row); the row's part of W_VP; whether x
// starts a wedge as a pivot; and, for rows x < 4096 of side 0, the entries of
// rank below 4096, 2048 and 1024 (the dense block's fill, which picks its
// default size).
//   W_VP: the wedges through mid y start at its higher-priority neighbours;
// the one at place j of row y walks the d(y) - 1 - j entries after it, so
// row y adds cut (d - 1) - cut (cut - 1) / 2, with no walk over entries.
//   A pivot x is active when some lower neighbour y has an entry after x.
// Row x is in priority order, so from the first lower neighbour of degree 1
// on there is none; a thread looks at a few entries, and the wavefront at
// the rest of a row that is still undecided.
// Results: [0] W_VP, [1] active pivots, [2..4] the block's entries, [5] and
// [6] the largest degrees.
struct RowSide {
  const uint32_t* off;
  const uint32_t* adj;
  const int32_t* rev;
  const int32_t* grank;
  int32_t* cut;
  int32_t n;
};
struct RowSides {
  RowSide s[2];
};
constexpr uint32_t kLook = 8;  // entries a thread looks at alone

__global__ __launch_bounds__(kThreads) void k_rows(RowSides S, unsigned long long* res) {
  const int lane = static_cast<int>(threadIdx.x) & 63;
  const int64_t n = static_cast<int64_t>(S.s[0].n) + S.s[1].n;
  const int64_t span = (n + 63) / 64 * 64;
  unsigned long long w_all = 0, active = 0;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < span;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const bool in = i < n;
    const int side = in && i >= S.s[0].n ? 1 : 0;
    const RowSide& P = S.s[side];
    const RowSide& O = S.s[1 - side];
    const int32_t x = in ? static_cast<int32_t>(side ? i - S.s[0].n : i) : 0;
    const uint32_t b = P.off[x], end = P.off[x + 1];
    uint32_t e = end;
    bool act = false, open = false;
    if (in) {
      uint32_t lo = b, hi = end;
      const int32_t gx = P.grank[x];
      while (lo < hi) {
        const uint32_t mid = lo + (hi - lo) / 2;
        if (O.grank[P.adj[mid] >> 1] < gx)
          lo = mid + 1;
        else
          hi = mid;
      }
      const uint64_t c = lo - b, d = end - b;
      P.cut[x] = static_cast<int32_t>(c);
      if (c) w_all += c * (d - 1) - c * (c - 1) / 2;
      if (x == 0) res[5 + side] = d;
      open = true;
      for (e = lo; e < end && e < lo + kLook; ++e) {
        const uint32_t y = P.adj[e] >> 1;
        const uint32_t dy = O.off[y + 1] - O.off[y];
        if (dy < 2 || static_cast<uint32_t>(P.rev[e]) + 1 < dy) {
          act = dy >= 2;
          open = false;
          break;
        }
      }
      open = open && e < end;
      if (side == 0 && x < 4096) {
        for (int k = 0; k < 3; ++k) {
          const int32_t T = 4096 >> k;
          if (x >= T) continue;
          uint32_t l = b, h = end;
          while (l < h) {
            const uint32_t mid = l + (h - l) / 2;
            if (P.adj[mid] < static_cast<uint32_t>(T) << 1)
              l = mid + 1;
            else
              h = mid;
          }
          if (l > b) atomicAdd(&res[2 + k], static_cast<unsigned long long>(l - b));
        }
      }
    }
    for (uint64_t left = __ballot(open); left; left &= left - 1) {
      const int j = __builtin_ctzll(left);
      const int sj = __shfl(side, j, 64);
      const uint32_t ej = __shfl(e, j, 64), endj = __shfl(end, j, 64);
      const RowSide& Q = S.s[sj];
      const RowSide& R = S.s[1 - sj];
      bool found = false;
      for (uint32_t q = ej; q < endj && !found; q += 64) {
        bool hit = false, stop = false;
        if (q + lane < endj) {
          const uint32_t y = Q.adj[q + lane] >> 1;
          const uint32_t dy = R.off[y + 1] - R.off[y];
          stop = dy < 2;
          hit = !stop && static_cast<uint32_t>(Q.rev[q + lane]) + 1 < dy;
        }
        found = __ballot(hit) != 0;
        if (__ballot(stop)) break;
      }
      if (lane == j) act = found;
    }
    active += act ? 1 : 0;
  }
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) {
    w_all += __shfl_xor(w_all, d, 64);
    active += __shfl_xor(active, d, 64);
  }
  __shared__ unsigned long long sh[2][kThreads / 64];
  if (lane == 0) {
    sh[0][threadIdx.x >> 6] = w_all;
    sh[1][threadIdx.x >> 6] = active;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    unsigned long long t = 0;
    for (int w = 0; w < kThreads / 64; ++w) t += sh[threadIdx.x][w];
    if (t) atomicAdd(&res[threadIdx.x], t);
  }
}

// Device memory of one build step, freed on scope exit (at least 16 bytes,
// so that even an empty array has an address).
struct Tmp : DevBuf {
  hipError_t alloc(size_t bytes) { return DevBuf::alloc(std::max<size_t>(bytes, 16)); }
};

struct Fail {
  int status;
  std::string msg;
};

#define DEV_TRY(expr)                                                                                   \
  do {                                                                                                  \
    hipError_t e_ = (expr);                                                                             \
    if (e_ != hipSuccess)                                                                               \
      throw Fail{e_ == hipErrorOutOfMemory ? DBBC_E_OOM : DBBC_E_DEVICE,                                \
                 std::string(#expr) + ": " + hipGetErrorString(e_)};                                    \
  } while (0)

template <class T>
void to_host(std::vector<T>& out, const void* src, size_t n, hipStream_t st) {
  out.resize(n);
  if (n) DEV_TRY(hipMemcpyAsync(out.data(), src, n * sizeof(T), hipMemcpyDeviceToHost, st));
}

#define LAUNCH(kernel, grid, threads, ...)                                             \
  do {                                                                                 \
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), 0, st, __VA_ARGS__);         \
    DEV_TRY(hipGetLastError());                                                        \
  } while (0)

void build(int32_t n_u, int32_t n_v, int64_t m, const int32_t* u_in, const int32_t* v_in, const int8_t* s_in,
           uint32_t flags, hipStream_t st, HostGraph& g, DeviceCsr& out) {
  const size_t M = static_cast<size_t>(m);
  // inputs on the device
  Tmp du, dv, ds;
  const int32_t* u = u_in;
  const int32_t* v = v_in;
  const int8_t* s = s_in;
  if (!(flags & DBBC_INPUT_DEVICE)) {
    DEV_TRY(du.alloc(M * 4));
    DEV_TRY(dv.alloc(M * 4));
    DEV_TRY(ds.alloc(M));
    if (m) {
      DEV_TRY(hipMemcpyAsync(du.p, u_in, M * 4, hipMemcpyHostToDevice, st));
      DEV_TRY(hipMemcpyAsync(dv.p, v_in, M * 4, hipMemcpyHostToDevice, st));
      DEV_TRY(hipMemcpyAsync(ds.p, s_in, M, hipMemcpyHostToDevice, st));
    }
    u = du.as<int32_t>();
    v = dv.as<int32_t>();
    s = ds.as<int8_t>();
  }
  const int32_t n[2] = {n_u, n_v};
  const int64_t nn = static_cast<int64_t>(n_u) + n_v;
  const int bits[2] = {bits_for(n_u), bits_for(n_v)};
  const int vbits = bits[1];
  radix::Digits dig_pair = radix::digits_of(0, vbits);  // the passes over v, then those over u
  const int v_passes = dig_pair.passes;
  radix::add_digits(dig_pair, vbits, vbits + bits[0]);
  const radix::Digits dig_side[2] = {radix::digits_of(0, bits[0]), radix::digits_of(0, bits[1])};
  // degrees are at most the other side's size
  const int deg_bits = bits_for(int64_t{std::max(n_u, n_v)} + 1);
  const radix::Digits dig_deg = radix::digits_of(0, deg_bits);
  const uint32_t top = static_cast<uint32_t>((uint64_t{1} << deg_bits) - 1);

  // Workspace: the result words (bad[2], replaced records, then k_rows'
  // seven), the vertices' runs and side ranks, chunk counts, the sorts'
  // control memory (one region: a sort's words are dead when its last pass
  // is done, in stream order), and eight record-sized arrays: two buffers of
  // three for the sorts of pairs and of V ranks, and two more where the sort
  // by U rank has more than two passes.  The rank sort's four vertex-sized
  // buffers lie in the second three record arrays, free at that time, where
  // they fit.
  constexpr int kResWords = 10;
  const size_t Mw = Carve::round(std::max<size_t>(M, 1)), Nw = Carve::round(static_cast<size_t>(nn));
  const size_t chunks_m = (M + kKeepChunk - 1) / kKeepChunk, chunks_n = (nn + kRankChunk - 1) / kRankChunk;
  const size_t ctl_words = std::max({radix::control_words(m, dig_pair), radix::control_words(nn, dig_deg),
                                     radix::control_bound(m, dig_side[0]), radix::control_bound(m, dig_side[1])});
  Tmp work;
  Carve cv;
  unsigned long long *words = nullptr, *ctl = nullptr;
  uint32_t *start[2], *end[2], *chunk = nullptr, *rank_buf = nullptr, *arr[8];
  int32_t* sr[2];
  for (int sizing = 1; sizing >= 0; --sizing) {
    if (!sizing) {
      DEV_TRY(work.alloc(cv.used * 4));
      cv = Carve{work.as<uint32_t>(), 0};
    }
    words = reinterpret_cast<unsigned long long*>(cv.take(2 * kResWords));
    for (int x = 0; x < 2; ++x) {  // cleared together with the words
      start[x] = cv.take(static_cast<size_t>(n[x]));
      end[x] = cv.take(static_cast<size_t>(n[x]));
    }
    for (int x = 0; x < 2; ++x) sr[x] = reinterpret_cast<int32_t*>(cv.take(static_cast<size_t>(n[x])));
    chunk = cv.take(std::max(chunks_m, 4 * chunks_n));
    ctl = reinterpret_cast<unsigned long long*>(cv.take(2 * ctl_words));
    for (int k = 0; k < 6; ++k) arr[k] = cv.take(Mw);
    for (int k = 6; k < 8; ++k) arr[k] = dig_side[0].passes > 2 ? cv.take(Mw) : nullptr;
    rank_buf = 4 * Nw <= 3 * Mw ? nullptr : cv.take(4 * Nw);
  }
  const size_t clear = static_cast<size_t>(reinterpret_cast<uint32_t*>(sr[0]) - reinterpret_cast<uint32_t*>(words));
  DEV_TRY(launch_fill_u64(words, 2, ~0ull, st));
  DEV_TRY(launch_fill_u64(words + 2, clear / 2 - 2, 0ull, st));
  const radix::Control cc{ctl};
  auto clear_control = [&](int64_t count, const radix::Digits& d) {
    DEV_TRY(launch_fill_u64(ctl, radix::control_words(count, d), 0ull, st));
  };

  // 1. records sorted by (u, v): after the passes over v, V's runs; in the
  // final order, U's runs and the records that later ones replace
  const radix::Soa<3> half[2] = {{{arr[0], arr[1], arr[2]}}, {{arr[3], arr[4], arr[5]}}};
  int cur = 1;  // the half that holds the sorted pairs
  const Runs runs[2] = {{start[0], end[0], n_u}, {start[1], end[1], n_v}};
  const uint32_t vmask = (1u << vbits) - 1u;
  unsigned long long head[3] = {~0ull, ~0ull, 0};
  if (m) {
    const RecordIn rin{u, v, s, vbits};
    const uint32_t m32 = static_cast<uint32_t>(m);
    clear_control(m, dig_pair);
    LAUNCH(k_record_hist, radix::hist_grid(m), kThreads, rin, m32, n_u, n_v, dig_pair, cc.hist(0), words);
    for (int p = 0; p < dig_pair.passes; ++p) {
      if (p == v_passes) LAUNCH(k_runs_v, grid_for(m), kThreads, half[cur].p[0], m32, vmask, runs[1]);
      if (p == 0)
        DEV_TRY((radix::pass<2, 3>(rin, half[0], m, dig_pair, p, cc, st)));
      else
        DEV_TRY((radix::pass<2, 3>(half[cur], half[1 - cur], m, dig_pair, p, cc, st)));
      cur = 1 - cur;
    }
    LAUNCH(k_runs_u, std::min(grid_for(m), 2048), kThreads, half[cur], m32, vbits, runs[0], words + 2);
    DEV_TRY(hipMemcpyAsync(head, words, sizeof(head), hipMemcpyDeviceToHost, st));
    DEV_TRY(hipStreamSynchronize(st));
  }
  if (head[0] != ~0ull || head[1] != ~0ull) {
    // the first bad record, ids checked before the sign
    if (head[0] <= head[1])
      throw Fail{DBBC_E_ID_RANGE, "edge " + std::to_string(head[0]) + " has a vertex id out of range"};
    int8_t sv = 0;
    DEV_TRY(hipMemcpyAsync(&sv, s + head[1], 1, hipMemcpyDeviceToHost, st));
    DEV_TRY(hipStreamSynchronize(st));
    throw Fail{DBBC_E_SIGN, "edge " + std::to_string(head[1]) + " has sign " + std::to_string(int(sv)) +
                                " (must be +1 or -1)"};
  }
  const int64_t dups = static_cast<int64_t>(head[2]), me = m - dups;
  if (dups && (flags & DBBC_DUP_REJECT)) throw Fail{DBBC_E_DUPLICATE, std::to_string(dups) + " duplicate (u, v) records"};
  g.n_u = n_u;
  g.n_v = n_v;
  g.m = me;
  g.m_in = m;
  g.dups_dropped = dups;
  const uint32_t me32 = static_cast<uint32_t>(me);
  if (dups) {
    // the kept records, and the runs over them: U's directly, V's from a
    // sort of their v (every vertex keeps a record, so every run is rewritten)
    const radix::Soa<3> from = half[cur], to = half[1 - cur];
    LAUNCH(k_keep<0>, static_cast<unsigned>(chunks_m), kThreads, from, static_cast<uint32_t>(m), chunk, to);
    DEV_TRY(scan_counts(chunk, static_cast<uint32_t>(chunks_m), nullptr, st));
    LAUNCH(k_keep<1>, static_cast<unsigned>(chunks_m), kThreads, from, static_cast<uint32_t>(m), chunk, to);
    LAUNCH(k_runs_u, std::min(grid_for(me), 2048), kThreads, to, me32, vbits, runs[0], words + 2);
    const VertexIn vin{to.p[0], vmask};
    const radix::Soa<1> vbuf[2] = {{{from.p[0]}}, {{from.p[1]}}};
    clear_control(me, dig_side[1]);
    DEV_TRY((radix::histogram<1>(vin, me, dig_side[1], cc, st)));
    DEV_TRY((radix::passes<1, 1>(vin, radix::Soa<1>{{from.p[2]}}, vbuf, me, dig_side[1], cc, st)));
    LAUNCH(k_runs_v, grid_for(me), kThreads, from.p[2], me32, ~0u, runs[1]);
    cur = 1 - cur;
  }

  // 2. the priority order of all vertices: ranks, input ids, row offsets
  Tmp off[2], adj[2];
  for (int x = 0; x < 2; ++x) {
    const size_t nx = static_cast<size_t>(n[x]);
    DEV_TRY(out.ord[x].alloc(nx * 4));
    DEV_TRY(out.grank[x].alloc(nx * 4));
    DEV_TRY(off[x].alloc((nx + 1) * 4));
    DEV_TRY(adj[x].alloc((static_cast<size_t>(me) + kAdjPad) * 4));
    DEV_TRY(out.rev[x].alloc(static_cast<size_t>(me) * 4));
    DEV_TRY(out.cut[x].alloc(nx * 4));
  }
  DEV_TRY(out.rec.alloc(static_cast<size_t>(me) * 4));
  {
    const uint32_t n32 = static_cast<uint32_t>(nn);
    const RankIn kin{start[0], end[0], start[1], end[1], static_cast<uint32_t>(n_u), n32, top};
    uint32_t* rb[4];
    for (size_t k = 0; k < 4; ++k)  // (three consecutive arrays of Mw words)
      rb[k] = (rank_buf ? rank_buf : arr[cur ? 0 : 3]) + k * Nw;
    const radix::Soa<2> rbuf[2] = {{{rb[0], rb[1]}}, {{rb[2], rb[3]}}};
    const radix::Soa<2>& sorted = rbuf[(dig_deg.passes - 1) & 1];
    clear_control(nn, dig_deg);
    DEV_TRY((radix::histogram<1>(kin, nn, dig_deg, cc, st)));
    DEV_TRY((radix::passes<1, 2>(kin, sorted, rbuf, nn, dig_deg, cc, st)));
    RankOut ro;
    for (int x = 0; x < 2; ++x) {
      ro.ord[x] = out.ord[x].as<int32_t>();
      ro.sr[x] = sr[x];
      ro.grank[x] = out.grank[x].as<int32_t>();
      ro.off[x] = off[x].as<uint32_t>();
    }
    RankSums* rc = reinterpret_cast<RankSums*>(chunk);
    const unsigned blocks = static_cast<unsigned>(chunks_n);
    if (blocks > 1)
      LAUNCH(k_ranks<0>, blocks, kThreads, sorted, n32, static_cast<uint32_t>(n_u), top, me32, rc, ro);
    LAUNCH(k_ranks<1>, blocks, kThreads, sorted, n32, static_cast<uint32_t>(n_u), top, me32, rc, ro);
  }

  // 3. the two CSRs
  for (int x = 0; x < 2; ++x) DEV_TRY(hipMemsetAsync(adj[x].as<uint32_t>() + me, 0, kAdjPad * 4, st));
  if (me) {
    const radix::Soa<3>&from = half[cur], &to = half[1 - cur];
    LAUNCH(k_place, grid_for(me), kThreads, from, me32, vbits, start[0], sr[0], sr[1], off[0].as<uint32_t>(), to);
    // by V rank: pass p reads `to` for even p, `from` for odd p; the last
    // pass also writes two arrays of the other buffer
    const radix::Digits& dv = dig_side[1];
    const radix::Soa<3> vbuf[2] = {from, to};
    const radix::Soa<3>& spare = dv.passes & 1 ? from : to;
    const radix::Soa<3>& spent = dv.passes & 1 ? to : from;
    const VOut vout{adj[1].as<uint32_t>(), spare.p[0], spare.p[1]};
    clear_control(me, dv);
    LAUNCH(k_row_hist, std::min(grid_for(n_v), 256), kThreads, off[1].as<uint32_t>(), static_cast<uint32_t>(n_v), dv,
           cc.hist(0));
    DEV_TRY((radix::passes<1, 3>(to, vout, vbuf, me, dv, cc, st)));
    // by U rank
    const radix::Digits& du = dig_side[0];
    const radix::Soa<4> ubuf[2] = {{{spare.p[2], spent.p[0], spent.p[1], spent.p[2]}},
                                   {{spare.p[0], spare.p[1], arr[6], arr[7]}}};
    const VIn uin{adj[1].as<uint32_t>(), spare.p[0], spare.p[1]};
    const UOut uout{adj[0].as<uint32_t>(), out.rec.as<uint32_t>(), out.rev[0].as<int32_t>(),
                    out.rev[1].as<int32_t>(), off[0].as<uint32_t>(), off[1].as<uint32_t>()};
    clear_control(me, du);
    LAUNCH(k_row_hist, std::min(grid_for(n_u), 256), kThreads, off[0].as<uint32_t>(), static_cast<uint32_t>(n_u), du,
           cc.hist(0));
    DEV_TRY((radix::passes<1, 4>(uin, uout, ubuf, me, du, cc, st)));
  }
  RowSides rows;
  for (int x = 0; x < 2; ++x)
    rows.s[x] = RowSide{off[x].as<uint32_t>(), adj[x].as<uint32_t>(), out.rev[x].as<int32_t>(),
                        out.grank[x].as<int32_t>(), out.cut[x].as<int32_t>(), n[x]};
  LAUNCH(k_rows, std::min(grid_for(nn), 2048), kThreads, rows, words + 3);

  // 4. the sizes the host keeps (the arrays stay on the device)
  unsigned long long sums[7];
  DEV_TRY(hipMemcpyAsync(sums, words + 3, sizeof(sums), hipMemcpyDeviceToHost, st));
  DEV_TRY(hipStreamSynchronize(st));
  for (int x = 0; x < 2; ++x) {
    HostSide& S = g.side[x];
    S = HostSide{};
    S.n = n[x];
    S.max_deg = static_cast<int64_t>(sums[5 + x]);
  }
  g.arrays = false;
  g.wedges_vp = static_cast<int64_t>(sums[0]);
  g.pivots_active = static_cast<int64_t>(sums[1]);
  for (int k = 0; k < 3; ++k) g.hub_nnz[k] = static_cast<int64_t>(sums[2 + k]);
  for (int x = 0; x < 2; ++x) {
    out.adj[x] = std::move(adj[x]);
    out.off[x] = std::move(off[x]);
  }
}

}  // namespace

int fetch_host_arrays(const DevGraphView& d, HostGraph& g, hipStream_t st, std::string& err) {
  if (g.arrays) return DBBC_OK;
  try {
    const size_t me = static_cast<size_t>(g.m);
    for (int x = 0; x < 2; ++x) {
      HostSide& S = g.side[x];
      const size_t n = static_cast<size_t>(S.n);
      to_host(S.off, d.off[x], n + 1, st);
      to_host(S.adj, d.adj[x], me, st);
      to_host(S.rev, d.rev[x], me, st);
      to_host(S.cut, d.cut[x], n, st);
      to_host(S.grank, d.grank[x], n, st);
      to_host(S.orig, d.ord[x], n, st);
    }
    to_host(g.side[0].rec, d.rec, me, st);
    g.side[1].rec.clear();
    DEV_TRY(hipStreamSynchronize(st));
  } catch (const Fail& f) {
    err = f.msg;
    (void)hipStreamSynchronize(st);
    return f.status;
  } catch (const std::bad_alloc&) {
    err = "host allocation failed while copying the graph";
    (void)hipStreamSynchronize(st);
    return DBBC_E_OOM;
  }
  g.arrays = true;
  return DBBC_OK;
}

int build_device_graph(int32_t n_u, int32_t n_v, int64_t m, const int32_t* u, const int32_t* v,
                       const int8_t* sign, uint32_t flags, hipStream_t st, HostGraph& g, DeviceCsr& out,
                       std::string& err) {
  if (n_u <= 0 || n_v <= 0 || m < 0) {
    err = "n_u and n_v must be positive and m non-negative";
    return DBBC_E_INVALID_ARG;
  }
  if (static_cast<int64_t>(n_u) + n_v >= (int64_t(1) << 30) || m >= (int64_t(1) << 31) - 1) {
    err = "graph too large: need n_u + n_v < 2^30 and m < 2^31 - 1";
    return DBBC_E_TOO_LARGE;
  }
  if (m > 0 && (!u || !v || !sign)) {
    err = "edge arrays must not be NULL";
    return DBBC_E_INVALID_ARG;
  }
  try {
    build(n_u, n_v, m, u, v, sign, flags, st, g, out);
  } catch (const Fail& f) {
    err = f.msg;
    (void)hipStreamSynchronize(st);
    return f.status;
  } catch (const std::bad_alloc&) {
    err = "host allocation failed while building the graph";
    (void)hipStreamSynchronize(st);
    return DBBC_E_OOM;
  }
  return DBBC_OK;
}

}  // namespace dbbc
