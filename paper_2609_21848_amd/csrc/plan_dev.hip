// Plans built on the device: the work split of make_plan (plan.cpp), for a
// count or for the per-vertex pass, computed from the device CSR with
// kernels, scans and sorts (the binning step of Algorithm 1 that sizes each
// pivot's work, Eq. 1, done per CSR entry instead of per pivot on the host).
//
// Per side s, every CSR entry e of row x, with mid y = adj[e] >> 1, yields at
// most one run of each kind:
//   F  forward: pivot x, the entries of row y below x in priority (from
//      rev[e] + 1 on), for e past x's higher-priority prefix cut[x]; a
//      window pivot (x < L) stops at the window, a hub pivot (x < T) with a
//      hub mid (y < T') starts past the dense block;
//   R  reverse (x >= L): the prefix of row y below both the reverse window
//      R and y's own higher-priority prefix cut[y];
//   M  reverse-mid (x >= L, R < L): the part of that prefix in [R, L);
//   H  per-vertex plans, hub pivots (x < T) through non-hub mids (y >= T'):
//      the part of the forward run below T (the hub pairs' sparse wedges,
//      tallied apart and completed by the dense block).
// Each (row, kind) is one candidate item, with its run count and work: sums
// over the row's entries.  Nothing is kept per entry.  A block takes a chunk
// of entries (of any rows), forms their run lengths, and leaves the chunk's
// run counts and wedges per kind, and the sums before every row that starts
// in it; a scan of the chunks' sums then gives every candidate's run count
// and work as differences.  The candidates are classified as make_plan
// classifies its items (skipped, small, hash, direct, reverse), counted per
// chunk of rows, and placed in their lists after a scan of those counts; a
// second pass over the entries forms the runs again and writes each at its
// item's place.  What a run needs of its mid is one 16-byte record per mid
// (one memory access per entry where six arrays were read).
//
// Measured on 50M records (5M x 2M vertices): a plan took 18.8 ms with
// per-entry lengths and their scans (11.6) and a scan of 64-byte counts per
// candidate (4.3), and takes 5.2: the two passes over the entries 1.5 and 1.6
// (bound by the random 16-byte record per entry), candidates 0.85, parts 0.6.
// On 2.2M records 1.90 -> 0.39 ms, on 20K 0.66 -> 0.15 ms (12 launches, 80
// before).
//
// Per-vertex plans also record every run's mid (flagged kMidWide where its
// credits may need two words) and first-edge position, and the owner of
// every small item; a direct item is cut into key windows that share its runs,
// or, past pv_part_work wedges, into parts that share its counters, and reverse endpoints with more than
// kReverseMaxSegs runs become direct items.
// Where the result differs from make_plan's, both are valid plans of the
// same wedges (the counts are the same):
//   - items and runs are listed in candidate order (row, then kind);
//   - small items are grouped greedily within chunks of kGroupChunk items;
//   - a split direct item starts a new part at every run that holds a
//     multiple of part_work in its wedge range (and every kPartMaxRuns
//     runs), so a part has at most part_work wedges plus its first run; the
//     hub pivots' tally items are cut the same way at kHubTallyPartWork.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <string>

#include "kernels.h"
#include "plan_dev.h"
#include "radix.h"
#include "scan.h"

namespace dbbc {
namespace {

constexpr int kThreads = 256;

enum : int { kF = 0, kR = 1, kM = 2, kH = 3 };  // run kinds (kH: per-vertex plans only)
enum : int { kSkip = 0, kSmallC = 1, kHashC = 2, kDirectC = 3, kRevC = 4, kHubC = 5 };  // item classes

constexpr uint32_t kPartMaxRuns = 65535;  // runs of a direct part (16-bit per-part counters)
constexpr int kGroupChunk = 256;          // small items grouped per chunk (one wavefront)

struct Fail {
  int status;
  std::string msg;
};

#define PD_TRY(expr)                                                                    \
  do {                                                                                  \
    hipError_t e_ = (expr);                                                             \
    if (e_ != hipSuccess)                                                               \
      throw Fail{e_ == hipErrorOutOfMemory ? DBBC_E_OOM : DBBC_E_DEVICE,                \
                 std::string(#expr) + ": " + hipGetErrorString(e_)};                    \
  } while (0)

int grid_for(int64_t n) {
  return static_cast<int>(std::max<int64_t>(1, std::min<int64_t>((n + kThreads - 1) / kThreads, 1 << 16)));
}

#define GRID_STRIDE(i, n)                                                                    \
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < (n); \
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)

// What the runs through a mid y need of it: its row, the row's entries of key
// rank below L, R and T, and those below L that rank above y itself (windows
// are at most 32,768 keys, so the counts fit 16 bits).  16 bytes, one access
// per entry; the largest key of its reverse runs is kept apart (rkey).
struct alignas(16) Mid {
  uint32_t off, end;
  uint16_t below_L, below_R, below_T, above_L;
};
static_assert(kPVWindowPacked <= 65535 && kMaxReverseL <= 65535, "window counts fit 16 bits");

constexpr int kPer = 4;  // entries per thread (8 take too many registers for four wavefronts a SIMD)
constexpr uint32_t kChunk = kThreads * kPer;
constexpr uint32_t kRowChunk = kThreads;  // rows per block where candidates are handled

// A place in a chunked sequence: the sums before it.  cnt: runs; sum: wedges.
struct PSide {
  const uint32_t* off;   // n + 1
  const uint32_t* adj;   // m
  const int32_t* rev;    // m
  const int32_t* cut;    // n
  const Mid* mids;       // per row of the other side
  const uint16_t* rkey;  // ... largest key of its reverse runs
  uint32_t* chunk_cnt[4];            // per kind: runs before each chunk of entries (chunks + 1)
  unsigned long long* chunk_sum[4];  // ... wedges
  uint32_t* row_cnt[4];              // per kind and row: runs of its chunk before it
  unsigned long long* row_sum[4];    // ... wedges
  int32_t* rmax;          // per row: largest key of its reverse runs
  uint32_t* parts;        // per candidate: parts of a split direct or a hub tally item
  uint32_t* part_pos;     // ... and its first part's place
  uint2* place;           // per candidate: see Place
  int32_t n, no, L, R, T, TO;
  int32_t nk;             // run kinds (candidates per row): 3, or 4 in per-vertex plans
  bool pv;                // a per-vertex plan
  bool wide_all;          // per-vertex plans: flag every run kMidWide
  unsigned long long max_deg;  // largest degree of the side (the wide-credit bound)
  unsigned long long max_mid;  // largest degree of the other side (a run's most entries)
  uint32_t m;
  uint32_t side;
  uint32_t chunks, row_chunks;
  uint32_t small_work;
  unsigned long long part_work;
};

struct PSides {
  PSide s[2];
};

struct Run {
  uint32_t start, len;
};

// The run of kind k at entry e (its reverse position rev) of row x through
// mid y; first_low: the row's first lower-priority entry.
__device__ __forceinline__ Run run_at(const PSide& P, int k, int32_t x, uint32_t e, uint32_t first_low, uint32_t y,
                                      int32_t rev, const Mid& mid) {
  if (k == kF || k == kH) {
    if (e < first_low) return Run{0, 0};
    uint32_t start = mid.off + static_cast<uint32_t>(rev) + 1, end;
    const bool hub = x < P.T && static_cast<int32_t>(y) < P.TO;
    if (k == kH) {  // hub pivot x through a non-hub mid: the run's keys below T
      if (x >= P.T || hub) return Run{0, 0};
      end = mid.off + mid.below_T;
    } else if (x < P.L) {
      end = mid.off + mid.below_L;
      if (hub) start = max(start, mid.off + mid.below_T);
    } else {
      end = mid.end;
    }
    return Run{start, end > start ? end - start : 0u};
  }
  if (x < P.L) return Run{0, 0};
  if (k == kR) return Run{mid.off, min(mid.below_R, mid.above_L)};
  if (P.R == P.L) return Run{0, 0};
  return Run{mid.off + mid.below_R, mid.above_L > mid.below_R ? mid.above_L - uint32_t{mid.below_R} : 0u};
}

__device__ __forceinline__ Mid load_mid(const Mid* mids, uint32_t y) {
  return __builtin_bit_cast(Mid, *reinterpret_cast<const uint4*>(mids + y));
}

// Runs and wedges of candidate (x, k).
__device__ __forceinline__ void row_totals(const PSide& P, int k, int32_t x, uint32_t& nseg, unsigned long long& work) {
  const uint32_t b = P.off[x], e = P.off[x + 1];
  nseg = 0;
  work = 0;
  if (b == e) return;
  // rows without entries come last: the entry after a row starts the next
  // row, or there is none
  const bool last = e == P.m;
  const uint32_t cb = b / kChunk, ce = last ? P.chunks : e / kChunk;
  nseg = P.chunk_cnt[k][ce] - P.chunk_cnt[k][cb] - P.row_cnt[k][x];
  work = P.chunk_sum[k][ce] - P.chunk_sum[k][cb] - P.row_sum[k][x];
  if (!last) {
    nseg += P.row_cnt[k][x + 1];
    work += P.row_sum[k][x + 1];
  }
}

struct Cand {
  int cls;
  uint32_t nseg;
  unsigned long long work;
  uint32_t nparts;  // reverse: parts (0 = a single item); direct: parts when split
  bool split;       // a direct item cut into parts
  int32_t key_lo, key_hi;
  uint32_t flags;
};

// Per-vertex plans: the key windows of a direct item (kPVWindowPacked keys
// with packed counters, see pv_packed; else kPVWindow keys).
__device__ bool pv_item_packed(const PSide& P, uint32_t nseg, uint32_t flags) {
  const int64_t deg_T = P.T < P.n ? static_cast<int64_t>(P.off[P.T + 1] - P.off[P.T]) : 0;
  return pv_packed(nseg, (flags & kItemHubPairs) != 0, deg_T);
}
__device__ uint32_t pv_window_count(int32_t key_lo, int32_t key_hi, bool packed) {
  const uint32_t win = static_cast<uint32_t>(packed ? kPVWindowPacked : kPVWindow);
  return (static_cast<uint32_t>(key_hi - key_lo) + win - 1) / win;
}
__device__ uint32_t pv_item_windows(const PSide& P, const Cand& c) {
  return pv_window_count(c.key_lo, c.key_hi, pv_item_packed(P, c.nseg, c.flags));
}

// Classify candidate (x, k) as make_plan's place() does.  With kParts, a
// split direct item's (and a hub tally item's) part count is read too.
template <bool kParts>
__device__ Cand classify(const PSide& P, int32_t x, int k) {
  Cand c{};
  c.cls = kSkip;
  if (k == kH) {  // a hub pivot's tally item (per-vertex plans): kept with one run
    if (x >= P.T) return c;
    row_totals(P, kH, x, c.nseg, c.work);
    if (c.nseg == 0) return c;
    c.cls = kHubC;
    c.key_lo = x + 1;
    c.key_hi = P.T;
    c.flags = kItemHubPairs;
    if (kParts) c.nparts = P.parts[static_cast<int64_t>(x) * P.nk + k];
    return c;
  }
  if (k != kF && (x < P.L || (k == kM && P.R == P.L))) return c;
  row_totals(P, k, x, c.nseg, c.work);
  const bool hub = k == kF && x < P.T;
  c.flags = hub ? kItemHubPairs : 0u;
  // one run: every pair of the item has at most one wedge, and adds nothing
  // unless the dense block completes the pair
  if (c.nseg == 0 || (c.nseg < 2 && !hub)) return c;
  const bool small = c.work <= P.small_work;
  if (k == kF) {
    c.key_lo = x + 1;
    c.key_hi = x < P.L ? P.L : P.n;
    c.cls = small ? kSmallC : (x < P.L ? kDirectC : kHashC);
  } else if (k == kR) {
    // rows are sorted by rank: the keys stop at the largest run end
    c.key_lo = 0;
    c.key_hi = min(P.R, max(P.rmax[x], 0) + 1);
    if (c.work <= static_cast<unsigned long long>(reverse_small_work(P.pv, P.small_work))) {
      c.cls = kSmallC;
      return c;
    }
    if (P.pv) {  // no parts: one reverse item, or a direct item past kReverseMaxSegs runs
      c.cls = c.nseg > kReverseMaxSegs ? kDirectC : kRevC;
      return c;
    }
    c.cls = kRevC;
    c.nparts = c.nseg <= kReverseCountMaxSegs ? 0u : (c.nseg + kReverseCountMaxSegs - 1) / kReverseCountMaxSegs;
  } else {
    c.key_lo = P.R;
    c.key_hi = P.L;
    c.cls = small ? kSmallC : kDirectC;
  }
  if (c.cls == kDirectC && (c.work > P.part_work || (!P.pv && c.nseg > kPartMaxRuns))) {
    c.split = true;
    if (kParts) c.nparts = P.parts[static_cast<int64_t>(x) * P.nk + k];
  }
  return c;
}

// ---- kernels ------------------------------------------------------------------

// The mids' records of both sides: side s's runs go through the rows y of the
// other side.
struct MidArgs {
  const uint32_t* off;
  const uint32_t* adj;
  const int32_t* cut;
  Mid* out;
  uint16_t* rkey;
  int32_t n;        // rows y
  int32_t L, R, T;  // windows of the keys' side
};

__global__ __launch_bounds__(kThreads) void k_mids(MidArgs a0, MidArgs a1) {
  GRID_STRIDE(i, static_cast<int64_t>(a0.n) + a1.n) {
    const MidArgs& a = i < a0.n ? a0 : a1;
    const int64_t y = i < a0.n ? i : i - a0.n;
    const uint32_t b = a.off[y], e = a.off[y + 1];
    // entries of rank below k (rows are sorted by rank; an entry is
    // (rank << 1) | negative), looked for up to `to`
    auto below = [&](int32_t k, uint32_t to) {
      const uint32_t key = static_cast<uint32_t>(k) << 1;
      uint32_t lo = b, hi = to;
      while (lo < hi) {
        const uint32_t mid = lo + (hi - lo) / 2;
        if (a.adj[mid] < key)
          lo = mid + 1;
        else
          hi = mid;
      }
      return lo;
    };
    Mid m;
    m.off = b;
    m.end = e;
    const uint32_t l = below(a.L, e), r = a.R == a.L ? l : below(a.R, l);  // R <= L
    m.below_L = static_cast<uint16_t>(l - b);
    m.below_R = static_cast<uint16_t>(r - b);
    m.below_T = static_cast<uint16_t>(a.T ? below(a.T, l) - b : 0u);  // T <= L
    m.above_L = static_cast<uint16_t>(min(l - b, static_cast<uint32_t>(a.cut[y])));
    *reinterpret_cast<uint4*>(a.out + y) = __builtin_bit_cast(uint4, m);
    const uint32_t rl = min(m.below_R, m.above_L);
    a.rkey[y] = static_cast<uint16_t>(rl ? a.adj[b + rl - 1] >> 1 : 0u);
  }
}

// The row of entry e: the last x with off[x] <= e (rows without entries come
// last), found by one wavefront, 64 probes a step.
__device__ __forceinline__ int32_t row_of(const uint32_t* off, int32_t n, uint32_t e) {
  const int lane = static_cast<int>(threadIdx.x) & 63;
  int64_t lo = 0, hi = n;  // off[lo] <= e, and off[x] > e for x >= hi (off[n] = m > e)
  while (hi - lo > 1) {
    const int64_t step = (hi - lo + 63) / 64;
    const int64_t x = lo + (lane + 1) * step;
    const uint64_t le = __ballot(x < hi && off[x < hi ? x : lo] <= e);
    const int k = __popcll(le);  // probes at or before the row (a prefix)
    const int64_t nlo = lo + static_cast<int64_t>(k) * step;
    hi = min(hi, nlo + step);
    lo = nlo;
  }
  return static_cast<int32_t>(lo);
}

// One block's chunk of entries of a side: each thread's kPer consecutive
// entries and their rows.
struct ChunkShared {
  uint32_t head[kChunk];  // the row that starts at an entry of the chunk, or 0
  uint32_t wmax[kThreads / 64];
  int32_t r0;
};
struct ChunkRows {
  uint32_t c0, c1;        // the chunk's entries
  int32_t r0;             // row of the first
  uint32_t e0;            // the thread's first entry
  int32_t row[kPer];
};

__device__ __forceinline__ ChunkRows chunk_rows(const PSide& P, uint32_t chunk, ChunkShared& sh) {
  const int tid = static_cast<int>(threadIdx.x), lane = tid & 63, wave = tid >> 6;
  ChunkRows c;
  c.c0 = chunk * kChunk;
  c.c1 = min(P.m, c.c0 + kChunk);
  if (wave == 0) {
    const int32_t r = row_of(P.off, P.n, c.c0);
    if (lane == 0) sh.r0 = r;
  }
  for (uint32_t i = tid; i < kChunk; i += kThreads) sh.head[i] = 0;
  __syncthreads();
  c.r0 = sh.r0;
  for (int64_t x = static_cast<int64_t>(c.r0) + 1 + tid; x < P.n; x += kThreads) {
    const uint32_t b = P.off[x];
    if (b >= c.c1) break;
    sh.head[b - c.c0] = static_cast<uint32_t>(x);
  }
  __syncthreads();
  c.e0 = c.c0 + tid * kPer;
  uint32_t mx = 0;
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    mx = max(mx, sh.head[tid * kPer + j]);
    c.row[j] = static_cast<int32_t>(mx);
  }
  uint32_t x = mx;  // rows grow along the entries: a running maximum
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t up = __shfl_up(x, d, 64);
    if (lane >= d) x = max(x, up);
  }
  if (lane == 63) sh.wmax[wave] = x;
  uint32_t before = __shfl_up(x, 1, 64);
  if (lane == 0) before = 0;
  __syncthreads();
  for (int w = 0; w < wave; ++w) before = max(before, sh.wmax[w]);
  before = max(before, static_cast<uint32_t>(c.r0));
#pragma unroll
  for (int j = 0; j < kPer; ++j) c.row[j] = max(c.row[j], static_cast<int32_t>(before));
  return c;
}

// Exclusive sums over the block's threads of nv 64-bit values, and totals.
template <int kNv, int kT = kThreads>
__device__ __forceinline__ void block_excl64(unsigned long long (&v)[kNv], unsigned long long (&total)[kNv],
                                             unsigned long long (*sh)[kNv]) {
  const int lane = static_cast<int>(threadIdx.x) & 63, wave = static_cast<int>(threadIdx.x) >> 6;
  unsigned long long x[kNv];
#pragma unroll
  for (int k = 0; k < kNv; ++k) x[k] = v[k];
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
#pragma unroll
    for (int k = 0; k < kNv; ++k) {
      const unsigned long long up = __shfl_up(x[k], d, 64);
      if (lane >= d) x[k] += up;
    }
  }
  __syncthreads();
  if (lane == 63)
#pragma unroll
    for (int k = 0; k < kNv; ++k) sh[wave][k] = x[k];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kNv; ++k) {
    unsigned long long before = 0, all = 0;
    for (int w = 0; w < kT / 64; ++w) {
      before += w < wave ? sh[w][k] : 0ull;
      all += sh[w][k];
    }
    v[k] = before + x[k] - v[k];
    total[k] = all;
  }
}

// Run counts of the four kinds of at most kChunk entries, in one word.
__device__ __forceinline__ unsigned long long one_run(int k) { return 1ull << (16 * k); }
__device__ __forceinline__ uint32_t runs_of(unsigned long long w, int k) {
  return static_cast<uint32_t>(w >> (16 * k)) & 0xffffu;
}

// Pass over the entries: each chunk's runs and wedges per kind, the sums
// before each row that starts in it, and each row's largest reverse key.
template <int kNk>
__global__ __launch_bounds__(kThreads, 4) void k_entries(PSides S) {
  __shared__ ChunkShared sh;
  __shared__ int32_t rm[kChunk + 1];  // largest reverse key + 1 of the rows from r0 on
  __shared__ unsigned long long scan[kThreads / 64][kNk + 1];
  const PSide& P = blockIdx.x < S.s[0].chunks ? S.s[0] : S.s[1];
  const uint32_t chunk = blockIdx.x < S.s[0].chunks ? blockIdx.x : blockIdx.x - S.s[0].chunks;
  const int tid = static_cast<int>(threadIdx.x);
  for (uint32_t i = tid; i <= kChunk; i += kThreads) rm[i] = 0;
  const ChunkRows c = chunk_rows(P, chunk, sh);
  uint32_t w[kPer];
  int32_t rev[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const uint32_t e = c.e0 + j;
    w[j] = e < c.c1 ? P.adj[e] : 0u;
    rev[j] = e < c.c1 ? P.rev[e] : 0;
  }
  uint32_t len[kPer][kNk];
  unsigned long long v[kNk + 1] = {};  // packed run counts, then wedges per kind
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const uint32_t e = c.e0 + j;
    const bool in = e < c.c1;
    const uint32_t y = w[j] >> 1;
    const Mid mid = load_mid(P.mids, y);
    const int32_t x = c.row[j];
    const uint32_t low = P.off[x] + static_cast<uint32_t>(P.cut[x]);
#pragma unroll
    for (int k = 0; k < kNk; ++k) {
      const uint32_t l = in ? run_at(P, k, x, e, low, y, rev[j], mid).len : 0u;
      len[j][k] = l;
      if (l) v[0] += one_run(k);
      v[1 + k] += l;
    }
    if (len[j][kR]) atomicMax(&rm[x - c.r0], P.rkey[y] + 1);
  }
  unsigned long long total[kNk + 1];
  block_excl64<kNk + 1>(v, total, scan);
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const uint32_t e = c.e0 + j;
    if (e < c.c1 && e == P.off[c.row[j]]) {
#pragma unroll
      for (int k = 0; k < kNk; ++k) {
        P.row_cnt[k][c.row[j]] = runs_of(v[0], k);
        P.row_sum[k][c.row[j]] = v[1 + k];
      }
    }
#pragma unroll
    for (int k = 0; k < kNk; ++k) {
      if (len[j][k]) v[0] += one_run(k);
      v[1 + k] += len[j][k];
    }
  }
  if (tid < kNk) {
    unsigned long long t = 0;
#pragma unroll
    for (int k = 0; k < kNk; ++k) t = tid == k ? total[1 + k] : t;
    P.chunk_cnt[tid][chunk] = runs_of(total[0], tid);
    P.chunk_sum[tid][chunk] = t;
  }
  __syncthreads();
  // rows inside the chunk are stored, those that cross its ends joined
  for (uint32_t i = tid; i <= kChunk; i += kThreads) {
    if (rm[i] == 0) continue;
    const int32_t x = c.r0 + static_cast<int32_t>(i);
    if (P.off[x] >= c.c0 && P.off[x + 1] <= c.c1)
      P.rmax[x] = rm[i] - 1;
    else
      atomicMax(&P.rmax[x], rm[i] - 1);
  }
}

// scan_block, with the total after the last element.
template <class T>
__device__ __forceinline__ T scan_with_total(T* p, uint32_t n) {
  const T all = scan_block(p, n);
  if (threadIdx.x == 0) p[n] = all;
  return all;
}

// The chunks' runs (blocks [0, 2 nk)) and wedges (the rest) per side and kind.
__global__ __launch_bounds__(kScanThreads) void k_scan_chunks(PSides S) {
  const int nk = S.s[0].nk;
  const int b = static_cast<int>(blockIdx.x) % (2 * nk), side = b / nk, k = b % nk;
  const PSide& P = S.s[side];
  if (static_cast<int>(blockIdx.x) < 2 * nk)
    scan_with_total(P.chunk_cnt[k], P.chunks);
  else
    scan_with_total(P.chunk_sum[k], P.chunks);
}

// ---- parts ---------------------------------------------------------------------
//
// Split direct items (kinds F and M) and the hub pivots' tally items (kind H)
// start a part at the first run, at every kPartMaxRuns-th run
// and at every run whose wedge range [pex, pex + len) of the item holds a
// multiple of the part budget (part_work, or kHubTallyPartWork).  Such items
// are few and large: they are listed (k_find_parts), and a block walks the
// entries of one.

// A listed candidate: row, kind | side << 2.
__global__ __launch_bounds__(kThreads) void k_find_parts(PSides S, uint2* list, uint32_t max_list, uint32_t* n_list) {
  GRID_STRIDE(i, static_cast<int64_t>(S.s[0].n) + S.s[1].n) {
    const bool side0 = i < S.s[0].n;
    const PSide& P = side0 ? S.s[0] : S.s[1];
    const int32_t x = static_cast<int32_t>(side0 ? i : i - S.s[0].n);
    const unsigned long long d = P.off[x + 1] - P.off[x];
    if (!(P.pv && x < P.T) && d <= kPartMaxRuns && d * P.max_mid <= P.part_work) continue;
    for (int k = 0; k < P.nk; ++k) {
      if (k == kR) continue;
      const Cand c = classify<false>(P, x, k);
      if (!c.split && c.cls != kHubC) continue;
      const uint32_t at = atomicAdd(n_list, 1u);
      if (at < max_list) list[at] = make_uint2(static_cast<uint32_t>(x), static_cast<uint32_t>(k) | (P.side << 2));
    }
  }
}

// What a part's item needs: its first run (index in the item) and the item's
// wedges before it.
struct PartStart {
  unsigned long long wedges;
  uint32_t run, pad;
};

constexpr int kPartThreads = 1024;
template <int kPass>
__global__ __launch_bounds__(kPartThreads) void k_parts(PSides S, const uint2* list, const uint32_t* n_list,
                                                    PartStart* direct, PartStart* hub) {
  __shared__ unsigned long long scan[kPartThreads / 64][2];
  __shared__ uint32_t sh[kPartThreads / 64];
  const int tid = static_cast<int>(threadIdx.x);
  for (uint32_t q = blockIdx.x; q < *n_list; q += gridDim.x) {
    const int32_t x = static_cast<int32_t>(list[q].x);
    const int k = static_cast<int>(list[q].y & 3u);
    const PSide& P = S.s[list[q].y >> 2];
    const uint32_t b = P.off[x], end = P.off[x + 1], low = b + static_cast<uint32_t>(P.cut[x]);
    const int64_t cand = static_cast<int64_t>(x) * P.nk + k;
    const unsigned long long pw = k == kH ? static_cast<unsigned long long>(kHubTallyPartWork) : P.part_work;
    PartStart* out = kPass ? (k == kH ? hub : direct) + P.part_pos[cand] : nullptr;
    unsigned long long runs = 0, wedges = 0;
    uint32_t parts = 0;
    for (uint32_t t0 = b; t0 < end; t0 += kPartThreads * kPer) {
      uint32_t len[kPer];
      unsigned long long v[2] = {0, 0}, total[2];
#pragma unroll
      for (int j = 0; j < kPer; ++j) {
        const uint32_t e = t0 + tid * kPer + j;
        len[j] = 0;
        if (e >= t0 && e < end) {
          const uint32_t y = P.adj[e] >> 1;
          len[j] = run_at(P, k, x, e, low, y, P.rev[e], load_mid(P.mids, y)).len;
        }
        v[0] += len[j] ? 1 : 0;
        v[1] += len[j];
      }
      block_excl64<2, kPartThreads>(v, total, scan);
      uint32_t mine = 0, flag = 0;
      unsigned long long r = runs + v[0], w = wedges + v[1];
#pragma unroll
      for (int j = 0; j < kPer; ++j) {
        if (!len[j]) continue;
        if (r % kPartMaxRuns == 0 || (w + len[j] - 1) / pw != (w - 1) / pw) {
          flag |= 1u << j;
          ++mine;
        }
        ++r;
        w += len[j];
      }
      uint32_t all;
      uint32_t at = parts + block_excl<kPartThreads>(mine, sh, all);
      if (kPass) {
        r = runs + v[0];
        w = wedges + v[1];
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
          if (!len[j]) continue;
          if (flag >> j & 1u) out[at++] = PartStart{w, static_cast<uint32_t>(r), 0u};
          ++r;
          w += len[j];
        }
      }
      parts += all;
      runs += total[0];
      wedges += total[1];
    }
    if (!kPass && tid == 0) P.parts[cand] = parts;
    __syncthreads();
  }
}

// ---- candidates ------------------------------------------------------------------

// What the candidates add to each list (scanned into list positions), then
// the plan's statistics: wedges and runs per kernel (direct, small, hash,
// reverse), the sparse and the skipped wedges (summed only).
enum : int {
  kBigRuns = 0,    // runs in segs (hash, direct and reverse items)
  kSmallRuns,      // runs in small_segs
  kHubRuns,        // runs in hub_segs (per-vertex plans)
  kSmallItems,
  kHashItems,
  kDirect,
  kDirectParts,    // parts of split direct items
  kDirectSplit,
  kWindows,        // per-vertex plans: key windows of the direct items
  kRev,
  kRevReduces,
  kRevAcc,
  kHubParts,
  kLists,
  kStWedges = kLists,
  kStRuns = kStWedges + 4,
  kStSparse = kStRuns + 4,
  kStSkipped,
  kCounters
};

// Add candidate c's list counts to q.
__device__ __forceinline__ void add_lists(const PSide& P, const Cand& c, unsigned long long* q) {
  switch (c.cls) {
    case kSmallC:
      q[kSmallRuns] += c.nseg;
      q[kSmallItems] += 1;
      break;
    case kHashC:
      q[kBigRuns] += c.nseg;
      q[kHashItems] += 1;
      break;
    case kDirectC: {
      const uint32_t nw = P.pv ? pv_item_windows(P, c) : 1u;
      q[kBigRuns] += c.nseg;
      q[kDirect] += 1;
      if (c.split) {  // every window in the same parts
        q[kDirectParts] += nw * c.nparts;
        q[kDirectSplit] += nw;
      } else if (P.pv) {
        q[kWindows] += nw;
      }
      break;
    }
    case kRevC:
      q[kBigRuns] += c.nseg;
      q[kRev] += c.nparts ? c.nparts : 1;
      if (c.nparts) {
        q[kRevReduces] += 1;
        q[kRevAcc] += c.nparts;
      }
      break;
    case kHubC:  // the dense block's sparse wedges: not in the kernels' statistics
      q[kHubRuns] += c.nseg;
      q[kHubParts] += c.nparts;
      break;
    default:
      break;
  }
}

// A block's rows of a side (side 0's blocks first), one per thread; the
// row's candidates.
struct RowCands {
  int side;
  int32_t x;  // may be past the side's last row: no candidates
  Cand c[4];
};
template <int kNk>
__device__ __forceinline__ RowCands row_cands(const PSides& S) {
  RowCands r;
  r.side = blockIdx.x < S.s[0].row_chunks ? 0 : 1;
  const PSide& P = S.s[r.side];
  const uint32_t chunk = r.side ? blockIdx.x - S.s[0].row_chunks : blockIdx.x;
  const int64_t x = static_cast<int64_t>(chunk) * kRowChunk + threadIdx.x;
  r.x = static_cast<int32_t>(x);
#pragma unroll
  for (int k = 0; k < kNk; ++k) {
    r.c[k] = Cand{};
    r.c[k].cls = kSkip;
    if (x < P.n) r.c[k] = classify<true>(P, r.x, k);
  }
  return r;
}

// Each block of rows: its candidates' list counts and statistics
// (counts[q * stride + block]).
template <int kNk>
__global__ __launch_bounds__(kThreads) void k_count(PSides S, unsigned long long* counts, uint32_t stride,
                                                    unsigned long long* max_direct) {
  __shared__ unsigned long long sh[kThreads / 64][kCounters];
  const RowCands r = row_cands<kNk>(S);
  const PSide& P = S.s[r.side];
  unsigned long long q[kCounters] = {};
  unsigned long long heaviest = 0;  // direct item (a split one: about its parts' budget)
#pragma unroll
  for (int k = 0; k < kNk; ++k) {
    const Cand& c = r.c[k];
    add_lists(P, c, q);
    if (c.cls == kDirectC) heaviest = max(heaviest, c.split ? min(c.work, P.part_work) : c.work);
    if (c.cls == kSkip) q[kStSkipped] += c.work;
    if (c.cls == kSkip || c.cls == kHubC) continue;
    const int slot = c.cls == kSmallC ? 1 : c.cls == kHashC ? 2 : c.cls == kDirectC ? 0 : 3;
    unsigned long long mult = 1;
    if (P.pv && slot == 0)  // the windows share the runs
      mult = pv_item_windows(P, c);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      q[kStWedges + t] += t == slot ? c.work * mult : 0ull;
      q[kStRuns + t] += t == slot ? c.nseg * mult : 0ull;
    }
    q[kStSparse] += c.work;
  }
#pragma unroll
  for (int t = 0; t < kCounters; ++t) {
    unsigned long long v = q[t];
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6][t] = v;
  }
  if (__ballot(heaviest != 0)) {  // (few wavefronts have direct items)
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) heaviest = max(heaviest, __shfl_xor(heaviest, d, 64));
    if ((threadIdx.x & 63) == 0) atomicMax(max_direct, heaviest);
  }
  __syncthreads();
  if (threadIdx.x < kCounters) {
    unsigned long long v = 0;
    for (int w = 0; w < kThreads / 64; ++w) v += sh[w][threadIdx.x];
    counts[static_cast<size_t>(threadIdx.x) * stride + blockIdx.x] = v;
  }
}

// Scan of the row chunks' counts, one block per counter: the totals go to
// out[q], the sums before side 1's first chunk to out[kCounters + q].
__global__ __launch_bounds__(kScanThreads) void k_scan_rows(unsigned long long* counts, uint32_t stride, uint32_t n,
                                                            uint32_t side1, unsigned long long* out) {
  unsigned long long* c = counts + static_cast<size_t>(blockIdx.x) * stride;
  const unsigned long long all = scan_with_total(c, n);
  __syncthreads();
  if (threadIdx.x == 0) {
    out[blockIdx.x] = all;
    out[kCounters + blockIdx.x] = c[side1];  // (side1 <= n)
  }
}

__device__ uint32_t dsat32(unsigned long long w) { return w > 0xffffffffull ? 0xffffffffu : static_cast<uint32_t>(w); }

// Where a candidate's runs go: run number c of its kind (over the whole side)
// goes to x + c; y says which list: kNowhere, a list with the top bit set, or
// the index of a small item.
constexpr uint32_t kNowhere = 0xffffffffu, kToSegs = 0x80000000u, kToHub = 0x80000001u;

// The order of hash and direct items: heaviest first, by the work's exponent
// and its nine bits after the leading one (a 16-bit key: two sort passes).
__device__ __forceinline__ uint32_t work_key(unsigned long long work) {
  uint32_t f = 0;
  if (work) {
    const int e = 63 - __builtin_clzll(work);
    f = (static_cast<uint32_t>(e) << 9) | (static_cast<uint32_t>(e >= 9 ? work >> (e - 9) : work << (9 - e)) & 0x1ffu);
  }
  return 0x7fffu - f;
}

// A count's direct items and parts (see direct_order_work).
__device__ __forceinline__ uint32_t direct_key(unsigned long long work, uint32_t runs) {
  return work_key(direct_order_work(work, runs));
}

struct ItemOut {
  // small items (grouped later): work | hub pivot << 30 | side << 31, first run, owner
  uint32_t* small_key;
  uint32_t* small_seg;
  int32_t* small_owner;
  Item* hash;          // hash items, unordered
  uint32_t* hash_key;
  Item* direct;        // direct items that are not split (per-vertex plans: their key windows), unordered
  uint32_t* direct_key;
  Item* split;         // split direct items
  uint32_t* split_part;  // ... the first part's place
  Item* rev;           // reverse items (final)
  Reduce* reduces;     // reverse reduces first
};

// Every candidate's item into its list, and its runs' place.
template <int kNk>
__global__ __launch_bounds__(kThreads) void k_items(PSides S, const unsigned long long* counts, uint32_t stride,
                                                    ItemOut o) {
  __shared__ unsigned long long sh[kThreads / 64][kLists];
  const RowCands rc = row_cands<kNk>(S);
  const PSide& P = S.s[rc.side];
  unsigned long long q[kLists] = {}, total[kLists];
#pragma unroll
  for (int k = 0; k < kNk; ++k) add_lists(P, rc.c[k], q);
  block_excl64<kLists>(q, total, sh);
#pragma unroll
  for (int t = 0; t < kLists; ++t) q[t] += counts[static_cast<size_t>(t) * stride + blockIdx.x];
  const int32_t x = rc.x;
  if (x >= P.n) return;
#pragma unroll
  for (int k = 0; k < kNk; ++k) {
    const Cand& c = rc.c[k];
    const int64_t cand = static_cast<int64_t>(x) * kNk + k;
    uint2 place = make_uint2(0u, kNowhere);
    Item it{};
    it.seg_count = c.nseg;
    it.owner = x;
    it.key_lo = c.key_lo;
    it.key_hi = c.key_hi;
    it.acc_slot = -1;
    it.flags = c.flags;
    it.side = P.side;
    it.work = dsat32(c.work);
    it.graph = 0;
    if (c.cls == kSmallC) {
      it.seg_begin = static_cast<uint32_t>(q[kSmallRuns]);
      place = make_uint2(it.seg_begin, static_cast<uint32_t>(q[kSmallItems]));
      o.small_key[q[kSmallItems]] = it.work | ((c.flags & kItemHubPairs) ? 1u << 30 : 0u) | (P.side << 31);
      o.small_seg[q[kSmallItems]] = it.seg_begin;
      o.small_owner[q[kSmallItems]] = x;
    } else if (c.cls == kHubC) {
      place = make_uint2(static_cast<uint32_t>(q[kHubRuns]), kToHub);
      P.part_pos[cand] = static_cast<uint32_t>(q[kHubParts]);
    } else if (c.cls != kSkip) {
      it.seg_begin = static_cast<uint32_t>(q[kBigRuns]);
      place = make_uint2(it.seg_begin, kToSegs);
      if (c.cls == kHashC) {
        o.hash[q[kHashItems]] = it;
        o.hash_key[q[kHashItems]] = work_key(c.work);
      } else if (c.cls == kDirectC) {
        if (c.split) P.part_pos[cand] = static_cast<uint32_t>(q[kDirectParts]);
        if (kNk == 4) {  // key windows that share the runs
          const bool packed = pv_item_packed(P, c.nseg, c.flags);
          const uint32_t nw = pv_window_count(c.key_lo, c.key_hi, packed);
          const int32_t win = packed ? kPVWindowPacked : kPVWindow;
          if (packed) it.flags |= kItemPacked;
          for (uint32_t w = 0; w < nw; ++w) {
            it.key_lo = c.key_lo + static_cast<int32_t>(w) * win;
            it.key_hi = min(c.key_hi, it.key_lo + win);
            if (c.split) {
              it.work = w;
              o.split[q[kDirectSplit] + w] = it;
              o.split_part[q[kDirectSplit] + w] = static_cast<uint32_t>(q[kDirectParts]) + w * c.nparts;
            } else {
              o.direct[q[kWindows] + w] = it;
              o.direct_key[q[kWindows] + w] = work_key(c.work);
            }
          }
        } else if (c.split) {
          o.split[q[kDirectSplit]] = it;
          o.split_part[q[kDirectSplit]] = static_cast<uint32_t>(q[kDirectParts]);
        } else {
          o.direct[q[kDirect] - q[kDirectSplit]] = it;
          o.direct_key[q[kDirect] - q[kDirectSplit]] = direct_key(c.work, c.nseg);
        }
      } else if (c.nparts == 0) {
        o.rev[q[kRev]] = it;
      } else {
        // parts of kReverseCountMaxSegs runs (their work is summed once the
        // runs are written), reduced into one accumulator slot each
        for (uint32_t p = 0; p < c.nparts; ++p) {
          Item part = it;
          part.seg_begin = it.seg_begin + p * kReverseCountMaxSegs;
          part.seg_count = min(kReverseCountMaxSegs, c.nseg - p * kReverseCountMaxSegs);
          part.flags |= kItemMultiPart;
          part.acc_slot = static_cast<int32_t>(q[kRevAcc] + p);
          part.work = 0;
          o.rev[q[kRev] + p] = part;
        }
        Reduce r{};
        r.acc_slot = static_cast<int32_t>(q[kRevAcc]);
        r.n_parts = static_cast<int32_t>(c.nparts);
        r.owner = x;
        r.key_lo = c.key_lo;
        r.key_hi = c.key_hi;
        r.flags = c.flags;
        r.side = P.side;
        r.graph = 0;
        o.reduces[q[kRevReduces]] = r;
      }
    }
    // runs are numbered per kind over the side: those before the row
    if (place.y != kNowhere) place.x -= P.chunk_cnt[k][P.off[x] / kChunk] + P.row_cnt[k][x];
    P.place[cand] = place;
    add_lists(P, c, q);
  }
}

// Small items into groups of at most kSmallGroupWork wedges that one
// wavefront counts in one hash table: greedy in list order within each chunk
// of kGroupChunk items.  A group holds items of one side, at most
// min(kSmallMaxItems, 2^(32 - key_bits) - 1) of them (the group's hash key is
// (index in group << key_bits) | key), and an item whose hub-pair counts go
// to the dense path stays alone.  A wavefront takes a chunk: each item's
// lanes find where a group that starts at it would end (a search over the
// work's prefix sums, up to the next item that may not join), the chain of
// starts from the chunk's first item is followed by lane reads (a few cycles
// a group), and the groups are written by their first items' lanes.
// Pass 0 counts each chunk's groups; pass 1 writes them and each item's index
// in its group.
struct SmallList {
  const uint32_t* key;  // work | hub pivot << 30 | side << 31
  const uint32_t* seg;  // first run (the next item's ends it)
  const int32_t* owner;
  uint32_t n, n_runs;
  int32_t kb0, kb1;     // key bits per side
  bool pv;
};

// v of a lane that every lane names.
__device__ __forceinline__ uint32_t lane_word(uint32_t v, uint32_t lane) {
  return static_cast<uint32_t>(__builtin_amdgcn_readlane(
      static_cast<int>(v), __builtin_amdgcn_readfirstlane(static_cast<int>(lane))));
}

template <int kPass>
__global__ __launch_bounds__(kThreads) void k_group(SmallList s, uint32_t* chunk_groups, Item* groups,
                                                    uint32_t* local_of) {
  constexpr uint32_t kHub = 1u << 30, kSide = 1u << 31;
  constexpr int kT = kGroupChunk / 64;
  __shared__ uint32_t sums[kThreads / 64][kGroupChunk + 1];  // work before each item of the chunk
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t n_chunks = (s.n + kGroupChunk - 1) / kGroupChunk;
  const uint32_t wave = threadIdx.x >> 6;
  const uint32_t ch = blockIdx.x * (kThreads / 64) + wave;
  if (ch >= n_chunks) return;
  const uint32_t c0 = ch * kGroupChunk, cnt = min(s.n - c0, static_cast<uint32_t>(kGroupChunk));
  uint32_t* P = sums[wave];
  uint32_t key[kT];
#pragma unroll
  for (int t = 0; t < kT; ++t) key[t] = t * 64 + lane < cnt ? s.key[c0 + t * 64 + lane] : 0u;
  uint32_t run = 0;
  uint64_t stop[kT];  // items that may not join the one before
  uint32_t last_kind = 0;
#pragma unroll
  for (int t = 0; t < kT; ++t) {
    uint32_t w = key[t] & (kHub - 1), x = w;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t up = __shfl_up(x, d, 64);
      if (lane >= static_cast<uint32_t>(d)) x += up;
    }
    P[t * 64 + lane] = run + x - w;
    run += lane_word(x, 63);
    uint32_t before = __shfl_up(key[t], 1, 64);
    if (lane == 0) before = last_kind;
    stop[t] = __ballot((key[t] & kHub) || (before & kHub) || ((before ^ key[t]) & kSide));
    last_kind = lane_word(key[t], 63);
  }
  if (lane == 0) P[kGroupChunk] = run;
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  uint32_t nx[kT];  // where a group that starts here ends
#pragma unroll
  for (int t = 0; t < kT; ++t) {
    const uint32_t i = t * 64 + lane;
    const uint32_t max_items = min(kSmallMaxItems, (1u << (32 - ((key[t] & kSide) ? s.kb1 : s.kb0))) - 1u);
    uint32_t hi = min(cnt, i + max_items);  // the end is in (i, hi]
#pragma unroll
    for (int q = kT - 1; q >= 0; --q) {  // ... and no later than the next stop
      const uint64_t m = q < t ? 0 : q > t ? stop[q] : lane == 63 ? 0 : stop[q] & ~((2ull << lane) - 1ull);
      if (m) hi = min(hi, static_cast<uint32_t>(q * 64 + __builtin_ctzll(m)));
    }
    uint32_t lo = i + 1;
    const uint32_t limit = P[i] + kSmallGroupWork;
    while (lo < hi) {  // the last end whose wedges fit (an item alone always does)
      const uint32_t mid = (lo + hi + 1) / 2;
      if (P[mid] <= limit)
        lo = mid;
      else
        hi = mid - 1;
    }
    nx[t] = lo;
  }
  uint64_t starts[kT] = {};
  uint32_t pos = 0;
#pragma unroll
  for (int t = 0; t < kT; ++t) {
    while (pos < min(cnt, static_cast<uint32_t>(t + 1) * 64)) {
      starts[t] |= 1ull << (pos & 63u);
      pos = lane_word(nx[t], pos & 63u);
    }
  }
  uint32_t g = kPass ? chunk_groups[ch] : 0u;
  uint32_t first = 0;  // the group that is open at a batch's start
#pragma unroll
  for (int t = 0; t < kT; ++t) {
    if (kPass && t * 64 + lane < cnt) {
      const uint32_t i = t * 64 + lane;
      const uint64_t upto = starts[t] & ((2ull << lane) - 1ull);
      const uint32_t mine = upto ? t * 64 + 63u - static_cast<uint32_t>(__clzll(static_cast<long long>(upto))) : first;
      local_of[c0 + i] = i - mine;
      if (mine == i) {
        const uint32_t end = nx[t];
        Item grp{};
        grp.seg_begin = s.seg[c0 + i];
        grp.seg_count = (c0 + end < s.n ? s.seg[c0 + end] : s.n_runs) - grp.seg_begin;
        grp.owner = s.owner[c0 + i];
        grp.key_hi = static_cast<int32_t>(end - i);
        grp.acc_slot = s.pv ? static_cast<int32_t>(c0 + i) : -1;  // per-vertex plans: owners are listed per item
        grp.flags = (key[t] & kHub) ? kItemHubPairs : 0u;
        grp.side = key[t] >> 31;
        grp.work = P[end] - P[i];
        groups[g + __popcll(upto) - 1] = grp;
      }
    }
    if (starts[t]) first = t * 64 + 63u - static_cast<uint32_t>(__clzll(static_cast<long long>(starts[t])));
    g += static_cast<uint32_t>(__popcll(starts[t]));
  }
  if (!kPass && lane == 0) chunk_groups[ch] = g;
}

struct RunOut {
  Segment* segs;
  Segment* small_segs;
  const uint32_t* local_of;  // small item -> index in its group
  // per-vertex plans
  uint32_t* seg_mid;         // each run's mid (| kMidWide), and its first edge's position
  uint32_t* seg_edge;
  uint32_t* small_seg_mid;
  uint32_t* small_seg_edge;
  Segment* hub_segs;         // the hub pivots' tally runs
  uint32_t* any_wide;        // set when some run is flagged kMidWide
};

// Second pass over the entries: every run into its item's place,
// segs[item's first + j] for the j-th run of the item, or small_segs tagged
// with the item's index in its group.
template <int kNk>
__global__ __launch_bounds__(kThreads, 4) void k_runs(PSides S, RunOut o) {
  __shared__ ChunkShared sh;
  __shared__ unsigned long long scan[kThreads / 64][1];
  const PSide& P = blockIdx.x < S.s[0].chunks ? S.s[0] : S.s[1];
  const uint32_t chunk = blockIdx.x < S.s[0].chunks ? blockIdx.x : blockIdx.x - S.s[0].chunks;
  const ChunkRows c = chunk_rows(P, chunk, sh);
  uint32_t w[kPer];
  int32_t rev[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const uint32_t e = c.e0 + j;
    w[j] = e < c.c1 ? P.adj[e] : 0u;
    rev[j] = e < c.c1 ? P.rev[e] : 0;
  }
  Run run[kPer][kNk];
  bool wide[kPer];
  unsigned long long v[1] = {0}, total[1];
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const uint32_t e = c.e0 + j;
    const uint32_t y = w[j] >> 1;
    const Mid mid = load_mid(P.mids, y);
    const int32_t x = c.row[j];
    const uint32_t low = P.off[x] + static_cast<uint32_t>(P.cut[x]);
    // per-vertex plans: flagged when the run's credits may reach 2^32 (the
    // mid's degree times the side's largest degree)
    wide[j] = kNk == 4 && (P.wide_all || static_cast<unsigned long long>(mid.end - mid.off) * P.max_deg >= (1ull << 32));
#pragma unroll
    for (int k = 0; k < kNk; ++k) {
      run[j][k] = run_at(P, k, x, e, low, y, rev[j], mid);
      if (e >= c.c1) run[j][k].len = 0;
      if (run[j][k].len) v[0] += one_run(k);
    }
  }
  block_excl64<1>(v, total, scan);
  uint32_t before[kNk];
#pragma unroll
  for (int k = 0; k < kNk; ++k) before[k] = P.chunk_cnt[k][chunk] + runs_of(v[0], k);
  bool any_wide = false;
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const uint32_t e = c.e0 + j;
#pragma unroll
    for (int k = 0; k < kNk; ++k) {
      const Run r = run[j][k];
      if (r.len == 0) continue;
      const uint2 place = P.place[static_cast<int64_t>(c.row[j]) * kNk + k];
      const uint32_t at = place.x + before[k]++;
      if (place.y == kNowhere) continue;
      const uint32_t len_g = (r.len << 1) | (w[j] & 1u);
      if (place.y == kToHub) {
        o.hub_segs[at] = Segment{r.start, len_g};
        continue;
      }
      const uint32_t mid = (w[j] >> 1) | (wide[j] ? kMidWide : 0u);
      any_wide = any_wide || wide[j];
      if (place.y == kToSegs) {
        o.segs[at] = Segment{r.start, len_g};
        if (kNk == 4) {
          o.seg_mid[at] = mid;
          o.seg_edge[at] = e;
        }
      } else {
        o.small_segs[at] = Segment{r.start, (o.local_of[place.y] << 16) | len_g};
        if (kNk == 4) {
          o.small_seg_mid[at] = mid;
          o.small_seg_edge[at] = e;
        }
      }
    }
  }
  if (kNk == 4 && __ballot(any_wide) && (threadIdx.x & 63) == 0 &&
      *reinterpret_cast<volatile uint32_t*>(o.any_wide) == 0)
    atomicOr(o.any_wide, 1u);
}

// The work of every reverse part (at most kReverseCountMaxSegs runs).
__global__ void k_rev_part_work(Item* rev, int64_t n, const Segment* segs) {
  GRID_STRIDE(i, n) {
    Item& it = rev[i];
    if (!(it.flags & kItemMultiPart)) continue;
    uint32_t w = 0;
    for (uint32_t j = 0; j < it.seg_count; ++j) w += segs[it.seg_begin + j].len_g >> 1;
    it.work = w;
  }
}

// A part of an item: runs [p.run, the next part's first) of its seg_count.
__device__ __forceinline__ Item part_of(Item it, uint32_t seg_begin, uint32_t seg_count, unsigned long long work,
                                        const PartStart* parts, uint32_t p, uint32_t n) {
  const PartStart s = parts[p];
  const uint32_t run_end = p + 1 < n ? parts[p + 1].run : seg_count;
  const unsigned long long w_end = p + 1 < n ? parts[p + 1].wedges : work;
  it.seg_begin = seg_begin + s.run;
  it.seg_count = run_end - s.run;
  it.work = dsat32(w_end - s.wedges);
  return it;
}

// The hub pivots' tally items (per-vertex plans), one per part of each
// pivot's hub runs.
__global__ __launch_bounds__(kThreads) void k_hub_parts(PSides S, const PartStart* parts, Item* out) {
  GRID_STRIDE(i, static_cast<int64_t>(S.s[0].T) + S.s[1].T) {
    const PSide& P = i < S.s[0].T ? S.s[0] : S.s[1];
    const int32_t x = static_cast<int32_t>(i < S.s[0].T ? i : i - S.s[0].T);
    const Cand c = classify<true>(P, x, kH);
    if (c.cls != kHubC) continue;
    const int64_t cand = static_cast<int64_t>(x) * P.nk + kH;
    const uint32_t first = P.place[cand].x + P.chunk_cnt[kH][P.off[x] / kChunk] + P.row_cnt[kH][x];
    const uint32_t at = P.part_pos[cand];
    Item it{};
    it.owner = x;
    it.key_lo = c.key_lo;
    it.key_hi = c.key_hi;
    it.acc_slot = -1;
    it.flags = c.flags;
    it.side = P.side;
    for (uint32_t p = 0; p < c.nparts; ++p) out[at + p] = part_of(it, first, c.nseg, c.work, parts + at, p, c.nparts);
  }
}

// Hash and direct items in order: a sort of (key, index) whose last pass
// moves the items themselves.
struct OrderIn {
  const uint32_t* key;
  __device__ __forceinline__ radix::Elt<2> load(uint32_t i) const { return {{key[i], i}}; }
};
struct GatherOut {
  const Item* in;
  Item* out;
  __device__ __forceinline__ void store(uint32_t pos, const radix::Elt<2>& e) const { out[pos] = in[e.w[1]]; }
};
// The parts of split direct items, and (count plans) their reduces.
struct SplitOut {
  Item* items;
  uint32_t* key;        // count plans: the parts' place in the order of all direct items
  Reduce* reduces;
  uint32_t acc0;        // count plans: first accumulator slot of the direct parts (one each)
  bool pv;              // per-vertex plans: an item's parts share an accumulator
};

__global__ void k_split_parts(PSides S, const Item* split, const uint32_t* part_at, uint32_t n, uint32_t n_parts,
                              const PartStart* parts, SplitOut o) {
  GRID_STRIDE(i, n) {
    const Item it = split[i];
    const PSide& P = S.s[it.side];
    const uint32_t at = part_at[i], np = (i + 1 < n ? part_at[i + 1] : n_parts) - at;
    // the item's kind: an owner below the window is counted forward (F)
    uint32_t nseg;
    unsigned long long work;
    row_totals(P, it.owner < P.L ? kF : kM, it.owner, nseg, work);
    const PartStart* first = parts + at - (o.pv ? it.work * np : 0u);  // (pv: work is the item's window)
    for (uint32_t p = 0; p < np; ++p) {
      Item part = part_of(it, it.seg_begin, nseg, work, first, p, np);
      part.flags |= kItemMultiPart;
      part.acc_slot = static_cast<int32_t>(o.pv ? i : o.acc0 + at + p);
      if (o.pv)
        part.work = (p << 16) | np;
      else
        o.key[at + p] = direct_key(part.work, part.seg_count);
      o.items[at + p] = part;
    }
    if (o.pv) continue;
    Reduce r{};
    r.acc_slot = static_cast<int32_t>(o.acc0 + at);
    r.n_parts = static_cast<int32_t>(np);
    r.owner = it.owner;
    r.key_lo = it.key_lo;
    r.key_hi = it.key_hi;
    r.flags = it.flags;
    r.side = it.side;
    r.graph = 0;
    o.reduces[i] = r;
  }
}

// The dense block's signs: B[x][y] for x < T, y < T' (rows of K bytes), and
// Bm keeps those of mids above x in the global order.
// (pos, per-vertex plans: the CSR position of every hub edge)
// One wavefront per row: its entries of rank below T' come first.
__global__ __launch_bounds__(kThreads) void k_hub_signs(const uint32_t* off, const uint32_t* adj,
                                                        const int32_t* grank_s, const int32_t* grank_o, int32_t T,
                                                        int32_t TO, int32_t K, int8_t* B, int8_t* Bm, int32_t* pos) {
  const int32_t x = static_cast<int32_t>((blockIdx.x * kThreads + threadIdx.x) >> 6);
  if (x >= T) return;
  const uint32_t end = off[x + 1];
  const int32_t gx = grank_s[x];
  for (uint32_t e = off[x] + (threadIdx.x & 63); e < end; e += 64) {
    const uint32_t y = adj[e] >> 1;
    if (static_cast<int32_t>(y) >= TO) break;
    const int8_t sg = (adj[e] & 1u) ? int8_t(-1) : int8_t(1);
    const size_t at = static_cast<size_t>(x) * K + y;
    B[at] = sg;
    if (grank_o[y] > gx) Bm[at] = sg;
    if (pos) pos[at] = static_cast<int32_t>(e);
  }
}

// The transposes of B and Bm (K x T): Bt[y][x] = B[x][y].
__global__ void k_hub_transpose(const int8_t* B, const int8_t* Bm, int32_t T, int32_t K, int8_t* Bt, int8_t* Bmt) {
  const int64_t n = static_cast<int64_t>(T) * K;
  GRID_STRIDE(i, n) {  // i = y T + x: coalesced writes
    const int64_t y = i / T, x = i % T;
    Bt[i] = B[x * K + y];
    Bmt[i] = Bm[x * K + y];
  }
}

// Per column y: Zc[x][y] = #{w > x : B[w][y] != 0} and
// Zc'[w][y] = #{x < w : Bm[x][y] != 0} (T x K each), in chunks of
// kColChunk rows: the nonzeros of every (column, chunk), then per (column,
// chunk) the counts of the chunks below (above) it and a walk of its rows.
constexpr int32_t kColChunk = 128;

__global__ void k_hub_chunk_counts(const int8_t* B, const int8_t* Bm, int32_t T, int32_t K, uint32_t* cB,
                                   uint32_t* cBm) {
  const int32_t nch = (T + kColChunk - 1) / kColChunk;
  const int64_t n = static_cast<int64_t>(nch) * K;
  GRID_STRIDE(i, n) {  // i = c K + y: coalesced reads of row x
    const int32_t c = static_cast<int32_t>(i / K), y = static_cast<int32_t>(i % K);
    uint32_t nb = 0, nbm = 0;
    for (int32_t x = c * kColChunk; x < min(T, (c + 1) * kColChunk); ++x) {
      nb += B[static_cast<size_t>(x) * K + y] != 0;
      nbm += Bm[static_cast<size_t>(x) * K + y] != 0;
    }
    cB[i] = nb;
    cBm[i] = nbm;
  }
}

__global__ void k_hub_col_counts(const int8_t* B, const int8_t* Bm, int32_t T, int32_t K, const uint32_t* cB,
                                 const uint32_t* cBm, int32_t* Zc, int32_t* Zcp) {
  const int32_t nch = (T + kColChunk - 1) / kColChunk;
  const int64_t n = static_cast<int64_t>(nch) * K;
  GRID_STRIDE(i, n) {
    const int32_t c = static_cast<int32_t>(i / K), y = static_cast<int32_t>(i % K);
    int32_t below = 0, above = 0;
    for (int32_t d = c + 1; d < nch; ++d) below += static_cast<int32_t>(cB[static_cast<size_t>(d) * K + y]);
    for (int32_t d = 0; d < c; ++d) above += static_cast<int32_t>(cBm[static_cast<size_t>(d) * K + y]);
    const int32_t x0 = c * kColChunk, x1 = min(T, (c + 1) * kColChunk);
    for (int32_t x = x1 - 1; x >= x0; --x) {
      Zc[static_cast<size_t>(x) * K + y] = below;
      below += B[static_cast<size_t>(x) * K + y] != 0;
    }
    for (int32_t w = x0; w < x1; ++w) {
      Zcp[static_cast<size_t>(w) * K + y] = above;
      above += Bm[static_cast<size_t>(w) * K + y] != 0;
    }
  }
}

// U-CSR position k -> V-CSR position of the same edge: row y = adj_u[k] >> 1
// of V, at the entry's reverse position.
__global__ void k_edge_positions(const uint32_t* adj_u, const int32_t* rev_u, const uint32_t* off_v, int64_t m,
                                 uint32_t* out) {
  GRID_STRIDE(k, m) out[k] = off_v[adj_u[k] >> 1] + static_cast<uint32_t>(rev_u[k]);
}

// ---- host side ------------------------------------------------------------------

template <class T>
T* alloc_n(DevBuf& b, int64_t n) {
  PD_TRY(b.alloc(static_cast<size_t>(std::max<int64_t>(n, 1)) * sizeof(T)));
  return b.as<T>();
}

#define LAUNCH(kernel, grid, threads, ...)                                             \
  do {                                                                                 \
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), 0, st, __VA_ARGS__);         \
    PD_TRY(hipGetLastError());                                                         \
  } while (0)

// The planner's scratch memory, carved out of one allocation.
struct Scratch {
  Carve c;
  template <class T>
  T* take(int64_t n) {
    return reinterpret_cast<T*>(c.take((static_cast<size_t>(std::max<int64_t>(n, 1)) * sizeof(T) + 3) / 4));
  }
};

// Items in work order.
void order_items(const uint32_t* key, int64_t n, uint32_t* buf, unsigned long long* ctl, const Item* in, Item* out,
                 hipStream_t st) {
  if (n == 0) return;
  const radix::Digits d = radix::digits_of(0, 16);
  const size_t w = Carve::round(static_cast<size_t>(n));
  const radix::Soa<2> bufs[2] = {{{buf, buf + w}}, {{nullptr, nullptr}}};  // two passes: the second is not used
  const radix::Control cc{ctl};
  PD_TRY(launch_fill_u64(ctl, radix::control_words(n, d), 0ull, st));
  PD_TRY((radix::histogram<1>(OrderIn{key}, n, d, cc, st)));
  PD_TRY((radix::passes<1, 2>(OrderIn{key}, GatherOut{in, out}, bufs, n, d, cc, st)));
}

void plan(const DevGraphView& g, const PlanParams& p, hipStream_t st, HostPlan& hp, DevPlanLists& out) {
  PSides S{};
  MidArgs ma[2];
  const int nk = p.per_vertex ? 4 : 3;
  const int64_t nn = static_cast<int64_t>(g.n[0]) + g.n[1];
  // a direct item can be split only past these
  const int64_t part_work = p.per_vertex ? p.pv_part_work : p.part_work;
  const bool parts = g.wedges > part_work || (p.per_vertex ? hp.T[0] > 0
                                                           : std::max(g.max_deg[0], g.max_deg[1]) > kPartMaxRuns);
  DevBuf scratch_b;
  unsigned long long *counts = nullptr, *totals_d = nullptr;
  // listed candidates, any wide run; then (64 bits each) the number of small
  // groups and the heaviest direct item
  uint32_t* words = nullptr;
  size_t clear_words = 0;
  uint2* part_list = nullptr;
  // candidates that can have parts: the hub pivots, or those of more than
  // part_work wedges or kPartMaxRuns runs (a kind has at most W_VP wedges
  // and m runs per side)
  const int64_t max_list =
      std::min<int64_t>(nk * nn, int64_t{hp.T[0]} + hp.T[1] +
                                     4 * (g.wedges / std::max<int64_t>(part_work, 1) + g.m / kPartMaxRuns) + 8);
  const uint32_t row_chunks[2] = {static_cast<uint32_t>((g.n[0] + int64_t{kRowChunk} - 1) / kRowChunk),
                                  static_cast<uint32_t>((g.n[1] + int64_t{kRowChunk} - 1) / kRowChunk)};
  const uint32_t all_row_chunks = row_chunks[0] + row_chunks[1], stride = all_row_chunks + 1;
  Scratch sc;
  for (int sizing = 1; sizing >= 0; --sizing) {
    if (!sizing) {
      PD_TRY(scratch_b.alloc(sc.c.used * 4));
      sc.c = Carve{scratch_b.as<uint32_t>(), 0};
    }
    // cleared together: the words, then both sides' largest keys
    words = sc.take<uint32_t>(6);
    for (int s = 0; s < 2; ++s) S.s[s].rmax = sc.take<int32_t>(g.n[s]);
    clear_words = sc.c.used;
    for (int s = 0; s < 2; ++s) {
      const int o = 1 - s;
      PSide& P = S.s[s];
      P.off = g.off[s];
      P.adj = g.adj[s];
      P.rev = g.rev[s];
      P.cut = g.cut[s];
      P.n = g.n[s];
      P.no = g.n[o];
      P.L = hp.L[s];
      P.R = hp.R[s];
      P.T = hp.T[s];
      P.TO = hp.T[o];
      P.m = static_cast<uint32_t>(g.m);
      P.side = static_cast<uint32_t>(s);
      P.pv = p.per_vertex;
      P.nk = nk;
      P.wide_all = p.wide_all;
      P.max_deg = static_cast<unsigned long long>(g.max_deg[s]);
      P.max_mid = static_cast<unsigned long long>(g.max_deg[o]);
      P.small_work = static_cast<uint32_t>(p.small_work);
      P.part_work = static_cast<unsigned long long>(part_work);
      P.chunks = static_cast<uint32_t>((g.m + kChunk - 1) / kChunk);
      P.row_chunks = row_chunks[s];
      Mid* mids = sc.take<Mid>(P.no);
      P.mids = mids;
      uint16_t* rkey = sc.take<uint16_t>(P.no);
      P.rkey = rkey;
      ma[s] = MidArgs{g.off[o], g.adj[o], g.cut[o], mids, rkey, P.no, P.L, P.R, P.T};
      for (int k = 0; k < nk; ++k) {
        P.chunk_cnt[k] = sc.take<uint32_t>(int64_t{P.chunks} + 1);
        P.chunk_sum[k] = sc.take<unsigned long long>(int64_t{P.chunks} + 1);
        P.row_cnt[k] = sc.take<uint32_t>(P.n);
        P.row_sum[k] = sc.take<unsigned long long>(P.n);
      }
      P.parts = parts ? sc.take<uint32_t>(int64_t{nk} * P.n) : nullptr;
      P.part_pos = parts ? sc.take<uint32_t>(int64_t{nk} * P.n) : nullptr;
      P.place = sc.take<uint2>(int64_t{nk} * P.n);
    }
    part_list = parts ? sc.take<uint2>(max_list) : nullptr;
    counts = sc.take<unsigned long long>(int64_t{kCounters} * stride);
    totals_d = sc.take<unsigned long long>(2 * kCounters);
  }
  PD_TRY(launch_fill_u64(reinterpret_cast<unsigned long long*>(words), clear_words / 2, 0ull, st));
  unsigned long long* n_groups_d = reinterpret_cast<unsigned long long*>(words + 2);
  unsigned long long* max_direct_d = reinterpret_cast<unsigned long long*>(words + 4);
  LAUNCH(k_mids, grid_for(nn), kThreads, ma[0], ma[1]);
  const uint32_t entry_blocks = S.s[0].chunks + S.s[1].chunks;
  if (g.m > 0) {
    if (nk == 4)
      LAUNCH(k_entries<4>, entry_blocks, kThreads, S);
    else
      LAUNCH(k_entries<3>, entry_blocks, kThreads, S);
  }
  LAUNCH(k_scan_chunks, 4 * nk, kScanThreads, S);
  unsigned long long tot[2 * kCounters];  // the totals, and the sums before side 1's first candidate
  for (PlanParams q = p;;) {
    if (parts) {
      LAUNCH(k_find_parts, grid_for(nn), kThreads, S, part_list, static_cast<uint32_t>(max_list), words);
      LAUNCH(k_parts<0>, 512, kPartThreads, S, part_list, words, nullptr, nullptr);
    }
    if (nk == 4)
      LAUNCH(k_count<4>, all_row_chunks, kThreads, S, counts, stride, max_direct_d);
    else
      LAUNCH(k_count<3>, all_row_chunks, kThreads, S, counts, stride, max_direct_d);
    LAUNCH(k_scan_rows, kCounters, kScanThreads, counts, stride, all_row_chunks, row_chunks[0], totals_d);
    PD_TRY(hipMemcpyAsync(tot, totals_d, sizeof(tot), hipMemcpyDeviceToHost, st));
    PD_TRY(hipStreamSynchronize(st));
    // per-vertex plans: a split item's parts share its windows' counters
    const unsigned long long slots = tot[kRevAcc] + (p.per_vertex ? tot[kDirectSplit] : tot[kDirectParts]);
    if (!larger_parts(q, static_cast<int64_t>(slots) * hp.acc_width * 4)) break;
    for (PSide& P : S.s) P.part_work = static_cast<unsigned long long>(p.per_vertex ? q.pv_part_work : q.part_work);
    PD_TRY(launch_fill_u64(reinterpret_cast<unsigned long long*>(words), 3, 0ull, st));
  }
  const unsigned long long* at1 = tot + kCounters;
  {
    PlanSizes z{};
    z.runs = std::max({tot[kBigRuns], tot[kSmallRuns], tot[kHubRuns]});
    z.items = std::max<uint64_t>({tot[kSmallItems], tot[kHashItems], tot[kRev], tot[kHubParts],
                                  tot[kDirectParts] +
                                      (p.per_vertex ? tot[kWindows] : tot[kDirect] - tot[kDirectSplit])});
    z.reduces = tot[kRevReduces] + tot[kDirectSplit];
    z.acc_slots = tot[kRevAcc] + tot[kDirectParts];
    std::string err;
    const int rc = check_plan_sizes(z, err);
    if (rc != DBBC_OK) throw Fail{rc, err};
  }
  const int64_t n_small = static_cast<int64_t>(tot[kSmallItems]), n_hash = static_cast<int64_t>(tot[kHashItems]);
  const int64_t n_rev = static_cast<int64_t>(tot[kRev]), n_split = static_cast<int64_t>(tot[kDirectSplit]);
  // direct items that are ordered, and all of them (the split items' parts)
  const int64_t n_direct = static_cast<int64_t>(p.per_vertex ? tot[kWindows] : tot[kDirect] - tot[kDirectSplit]);
  const int64_t n_dir_items = n_direct + static_cast<int64_t>(tot[kDirectParts]);
  const int64_t n_reduces = static_cast<int64_t>(tot[kRevReduces]) + (p.per_vertex ? 0 : n_split);
  const int64_t acc_slots = static_cast<int64_t>(tot[kRevAcc] + (p.per_vertex ? tot[kDirectSplit] : tot[kDirectParts]));

  // items
  DevBuf scratch2_b;
  ItemOut io{};
  Item* groups = nullptr;  // at most one per small item
  uint32_t *group_cnt = nullptr, *local_of = nullptr, *order_buf = nullptr;
  unsigned long long* ctl = nullptr;
  PartStart *dir_parts = nullptr, *hub_parts = nullptr;
  const uint32_t n_chunks = static_cast<uint32_t>((n_small + kGroupChunk - 1) / kGroupChunk);
  const int64_t n_direct_key = p.per_vertex ? n_direct : n_dir_items;  // direct items that are ordered
  const int64_t n_order = std::max(n_hash, n_direct_key);
  sc = Scratch{};
  for (int sizing = 1; sizing >= 0; --sizing) {
    if (!sizing) {
      PD_TRY(scratch2_b.alloc(sc.c.used * 4));
      sc.c = Carve{scratch2_b.as<uint32_t>(), 0};
    }
    io.small_key = sc.take<uint32_t>(n_small);
    io.small_seg = sc.take<uint32_t>(n_small);
    io.small_owner = sc.take<int32_t>(p.per_vertex ? 0 : n_small);
    groups = sc.take<Item>(n_small);
    group_cnt = sc.take<uint32_t>(n_chunks);
    local_of = sc.take<uint32_t>(n_small);
    io.hash = sc.take<Item>(n_hash);
    io.hash_key = sc.take<uint32_t>(n_hash);
    io.direct = sc.take<Item>(n_direct_key);
    io.direct_key = sc.take<uint32_t>(n_direct_key);
    io.split = sc.take<Item>(n_split);
    io.split_part = sc.take<uint32_t>(n_split);
    order_buf = sc.take<uint32_t>(2 * static_cast<int64_t>(Carve::round(static_cast<size_t>(n_order))));
    ctl = sc.take<unsigned long long>(static_cast<int64_t>(radix::control_bound(n_order, radix::digits_of(0, 16))));
    dir_parts = sc.take<PartStart>(static_cast<int64_t>(tot[kDirectParts]));
    hub_parts = sc.take<PartStart>(static_cast<int64_t>(tot[kHubParts]));
  }
  io.rev = alloc_n<Item>(out.reverse_items, n_rev);
  io.reduces = alloc_n<Reduce>(out.reduces, n_reduces);
  if (p.per_vertex) io.small_owner = alloc_n<int32_t>(out.small_owner, n_small);
  if (nk == 4)
    LAUNCH(k_items<4>, all_row_chunks, kThreads, S, counts, stride, io);
  else
    LAUNCH(k_items<3>, all_row_chunks, kThreads, S, counts, stride, io);
  if (tot[kDirectParts] + tot[kHubParts] > 0)
    LAUNCH(k_parts<1>, 512, kPartThreads, S, part_list, words, dir_parts, hub_parts);

  // small groups
  for (int s = 0; s < 2; ++s) {
    int32_t kb = 1;
    while ((int64_t{1} << kb) < g.n[s]) ++kb;
    hp.key_bits[s] = kb;
  }
  if (n_chunks > 0) {
    const uint32_t blocks = (n_chunks + kThreads / 64 - 1) / (kThreads / 64);
    const SmallList sl{io.small_key, io.small_seg, io.small_owner, static_cast<uint32_t>(n_small),
                       static_cast<uint32_t>(tot[kSmallRuns]), hp.key_bits[0], hp.key_bits[1], p.per_vertex};
    LAUNCH(k_group<0>, blocks, kThreads, sl, group_cnt, nullptr, nullptr);
    PD_TRY(scan_counts(group_cnt, n_chunks, n_groups_d, st));
    LAUNCH(k_group<1>, blocks, kThreads, sl, group_cnt, groups, local_of);
  }

  // runs
  RunOut ro{};
  ro.segs = alloc_n<Segment>(out.segs, static_cast<int64_t>(tot[kBigRuns]));
  ro.small_segs = alloc_n<Segment>(out.small_segs, static_cast<int64_t>(tot[kSmallRuns]));
  ro.local_of = local_of;
  ro.any_wide = words + 1;
  if (p.per_vertex) {
    ro.seg_mid = alloc_n<uint32_t>(out.seg_mid, static_cast<int64_t>(tot[kBigRuns]));
    ro.seg_edge = alloc_n<uint32_t>(out.seg_edge, static_cast<int64_t>(tot[kBigRuns]));
    ro.small_seg_mid = alloc_n<uint32_t>(out.small_seg_mid, static_cast<int64_t>(tot[kSmallRuns]));
    ro.small_seg_edge = alloc_n<uint32_t>(out.small_seg_edge, static_cast<int64_t>(tot[kSmallRuns]));
    ro.hub_segs = alloc_n<Segment>(out.hub_segs, static_cast<int64_t>(tot[kHubRuns]));
  }
  if (g.m > 0) {
    if (nk == 4)
      LAUNCH(k_runs<4>, entry_blocks, kThreads, S, ro);
    else
      LAUNCH(k_runs<3>, entry_blocks, kThreads, S, ro);
  }
  if (tot[kRevReduces] > 0) LAUNCH(k_rev_part_work, grid_for(n_rev), kThreads, io.rev, n_rev, ro.segs);
  if (p.per_vertex) {  // the hub pivots' tally items, side 0 first
    Item* hub_items = alloc_n<Item>(out.hub_items, static_cast<int64_t>(tot[kHubParts]));
    if (tot[kHubParts] > 0)
      LAUNCH(k_hub_parts, grid_for(int64_t{hp.T[0]} + hp.T[1]), kThreads, S, hub_parts, hub_items);
  }

  // hash items, heaviest first
  Item* hash = alloc_n<Item>(out.hash_items, n_hash);
  order_items(io.hash_key, n_hash, order_buf, ctl, io.hash, hash, st);
  // direct items, heaviest first (per-vertex plans: the parts of split items, then
  // the others: parts are tallied by a launch of their own)
  Item* direct = alloc_n<Item>(out.direct_items, n_dir_items);
  if (n_split > 0)
    LAUNCH(k_split_parts, grid_for(n_split), kThreads, S, io.split, io.split_part, static_cast<uint32_t>(n_split),
           static_cast<uint32_t>(tot[kDirectParts]), dir_parts,
           SplitOut{p.per_vertex ? direct : io.direct + n_direct, io.direct_key + n_direct, io.reduces + tot[kRevReduces], static_cast<uint32_t>(tot[kRevAcc]), p.per_vertex});
  order_items(io.direct_key, n_direct_key, order_buf, ctl, io.direct, direct + (p.per_vertex ? tot[kDirectParts] : 0), st);
  PD_TRY(out.acc.alloc(std::max<size_t>(static_cast<size_t>(acc_slots) * hp.acc_width * sizeof(uint32_t), 16)));

  // the dense block's signs
  for (int s = 0; s < 2; ++s) {
    out.hub_K[s] = 0;
    const int32_t T = hp.T[s], TO = hp.T[1 - s];
    if (T == 0) continue;
    const int32_t K = (TO + kHubKPad - 1) / kHubKPad * kHubKPad;
    const size_t TK = static_cast<size_t>(T) * K;
    int8_t* Bs = alloc_n<int8_t>(out.hub_B[s], static_cast<int64_t>(TK));
    int8_t* Bm = alloc_n<int8_t>(out.hub_Bm[s], static_cast<int64_t>(TK));
    PD_TRY(launch_fill_u64(reinterpret_cast<unsigned long long*>(Bs), TK / 8, 0ull, st));
    PD_TRY(launch_fill_u64(reinterpret_cast<unsigned long long*>(Bm), TK / 8, 0ull, st));
    int32_t* hpos = nullptr;
    if (p.per_vertex) {  // T K is a multiple of 128 kHubKPad: whole words
      hpos = alloc_n<int32_t>(out.hub_pos[s], static_cast<int64_t>(TK));
      PD_TRY(launch_fill_u64(reinterpret_cast<unsigned long long*>(hpos), TK / 2, ~0ull, st));
    }
    LAUNCH(k_hub_signs, (T + kThreads / 64 - 1) / (kThreads / 64), kThreads, g.off[s], g.adj[s], g.grank[s],
           g.grank[1 - s], T, TO, K, Bs, Bm, hpos);
    if (p.per_vertex) {  // the credit products' constants
      int8_t* Bt = alloc_n<int8_t>(out.hub_Bt[s], static_cast<int64_t>(TK));
      int8_t* Bmt = alloc_n<int8_t>(out.hub_Bmt[s], static_cast<int64_t>(TK));
      int32_t* Zc = alloc_n<int32_t>(out.hub_Zc[s], static_cast<int64_t>(TK));
      int32_t* Zcp = alloc_n<int32_t>(out.hub_Zcp[s], static_cast<int64_t>(TK));
      hipLaunchKernelGGL(k_hub_transpose, dim3(grid_for(static_cast<int64_t>(TK))), dim3(kThreads), 0, st, Bs, Bm,
                         T, K, Bt, Bmt);
      PD_TRY(hipGetLastError());
      const int64_t ncol = static_cast<int64_t>((T + kColChunk - 1) / kColChunk) * K;
      DevBuf cb_b, cbm_b;
      uint32_t* cB = alloc_n<uint32_t>(cb_b, ncol);
      uint32_t* cBm = alloc_n<uint32_t>(cbm_b, ncol);
      hipLaunchKernelGGL(k_hub_chunk_counts, dim3(grid_for(ncol)), dim3(kThreads), 0, st, Bs, Bm, T, K, cB, cBm);
      PD_TRY(hipGetLastError());
      hipLaunchKernelGGL(k_hub_col_counts, dim3(grid_for(ncol)), dim3(kThreads), 0, st, Bs, Bm, T, K, cB, cBm, Zc,
                         Zcp);
      PD_TRY(hipGetLastError());
      PD_TRY(hipStreamSynchronize(st));  // cb_b, cbm_b leave scope
    }
    out.hub_K[s] = K;
  }
  uint32_t words_h[6];
  PD_TRY(hipMemcpyAsync(words_h, words, sizeof(words_h), hipMemcpyDeviceToHost, st));
  PD_TRY(hipStreamSynchronize(st));
  out.any_wide = words_h[1] != 0;
  const uint32_t n_groups = words_h[2];  // at most the small items
  Item* groups_out = alloc_n<Item>(out.small_groups, n_groups);
  if (n_groups > 0)
    PD_TRY(hipMemcpyAsync(groups_out, groups, static_cast<size_t>(n_groups) * sizeof(Item), hipMemcpyDeviceToDevice,
                          st));

  hp.direct_max_work = words_h[4] | (static_cast<uint64_t>(words_h[5]) << 32);
  hp.acc_slots = static_cast<int32_t>(acc_slots);
  hp.n_reverse_side0 = static_cast<int32_t>(at1[kRev]);
  if (p.per_vertex) {
    hp.n_hub_side0 = static_cast<int32_t>(at1[kHubParts]);
    hp.n_heavy = static_cast<int32_t>(tot[kDirectParts]);
  }
  hp.n_items_kept[0] = static_cast<int32_t>(n_dir_items);
  hp.n_items_kept[1] = static_cast<int32_t>(n_rev);
  hp.n_items_kept[2] = static_cast<int32_t>(n_groups);
  hp.n_items_kept[3] = static_cast<int32_t>(n_hash);
  hp.n_items_kept[4] = static_cast<int32_t>(n_reduces);
  for (int j = 0; j < 4; ++j) {
    hp.k_wedges[j] = static_cast<int64_t>(tot[kStWedges + j]);
    hp.k_segs[j] = static_cast<int64_t>(tot[kStRuns + j]);
  }
  hp.w_sparse = static_cast<int64_t>(tot[kStSparse]);
  hp.w_skipped = static_cast<int64_t>(tot[kStSkipped]);
}

}  // namespace

int make_plan_device(const DevGraphView& g, const PlanParams& p, hipStream_t st, HostPlan& hp, DevPlanLists& out,
                     std::string& err) {
  int rc = check_plan_params(p, err);
  if (rc != DBBC_OK) return rc;
  // candidates and entries (plus one) are counted in 31 bits
  if ((p.per_vertex ? 4 : 3) * (static_cast<int64_t>(g.n[0]) + g.n[1]) + 1 > INT32_MAX || g.m + 1 > INT32_MAX) {
    err = "graph too large for the device planner";
    return DBBC_E_TOO_LARGE;
  }
  hp = HostPlan();
  hp.p = p;
  plan_windows(g.n, p, hp);
  try {
    plan(g, p, st, hp, out);
  } catch (const Fail& f) {
    err = f.msg;
    (void)hipStreamSynchronize(st);
    return f.status;
  } catch (const std::bad_alloc&) {
    err = "host allocation failed while planning";
    (void)hipStreamSynchronize(st);
    return DBBC_E_OOM;
  }
  return DBBC_OK;
}

}  // namespace dbbc

namespace dbbc {

int edge_positions_device(const DevGraphView& g, uint32_t* out, hipStream_t st, std::string& err) {
  if (g.m == 0) return DBBC_OK;
  hipLaunchKernelGGL(k_edge_positions, dim3(grid_for(g.m)), dim3(kThreads), 0, st, g.adj[0], g.rev[0], g.off[1], g.m,
                     out);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    err = std::string("edge positions: ") + hipGetErrorString(e);
    return DBBC_E_DEVICE;
  }
  return DBBC_OK;
}

}  // namespace dbbc
