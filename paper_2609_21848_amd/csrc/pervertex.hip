// HIP kernels (gfx950) of the per-vertex pass: for every vertex, the number
// of balanced and unbalanced butterflies that contain it (the vertex measure
// of Section I's applications).
//
// Each butterfly is counted once, at the pair (x, w) that owns it under the
// vertex priority (Algorithm 1, Phase 5): x and w are its two same-side
// vertices and its two mids are wedge mids of the pair.  With the pair's
// symmetric and asymmetric wedge counts p and n (Lemma 1):
//   - x and w each lie in C(p,2) + C(n,2) balanced and p n unbalanced
//     butterflies of the pair;
//   - the mid of a symmetric wedge lies in p - 1 balanced ones (paired with
//     each other symmetric mid) and n unbalanced ones, the mid of an
//     asymmetric wedge in n - 1 balanced and p unbalanced ones.
// So every item is walked twice: a tally of p and n per key as in the count
// pass, then a credit walk that reads each wedge's final p and n and adds
// the mid's share; the sweep credits the key vertices and, summed, the
// item's owner.  Every pair's counts are complete inside one item -- except
// those of heavy direct items, cut into parts whose counters meet in an
// accumulator before the parts credit from it (k_pv_heavy_tally), and the hub
// pairs of a dense block, whose completed counts the block's products leave in
// hub_xy (hubpv.hip) before these kernels run.
//
// Mid credits are summed per run (a run has one mid) in registers, then per
// batch in a per-wavefront LDS slot of the run's lane, and reach HBM as one
// 64-bit atomic per run; key and owner credits are one atomic per nonzero
// pair and per item.  Walk tags here are (item index in group << 7) |
// (run lane << 1) | g.
//
// Per-edge counts (the edge measure of the same section, kEdge): a wedge's
// share (p - 1 and n, or n - 1 and p) is also the number of butterflies of
// the pair that contain each of its two edges, since such a butterfly is the
// union of this wedge and one other wedge of the pair.  The run's first edge
// takes the run's summed share in the mid's place (the pass has no per-vertex
// output: 2M edges 1.63 -> 1.16 ms, 20M 24.3 -> 19.6 ms without the vertices'
// credits, their sums and the fills); the walked entry's edge takes
// its wedge's share at its position in the other side's CSR, one 64-bit
// atomic per wedge with both values packed (two for runs flagged kMidWide).
// The credit walk then reads long runs lane-major, so that the atomics of a
// wavefront hit consecutive positions.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "internal.h"
#include "kernels.h"
#include "walk.h"

namespace dbbc {
namespace dev {

// The runs k0 + stride * lane (< k1) of a batch with per-vertex tags, and
// each lane's mid (and, with kEdge, the position of its first edge).
struct RunEnds {
  uint32_t mid = 0, edge = 0, wide = 0;
};

template <bool kTagged, bool kEdge>
__device__ __forceinline__ SegReg load_seg_pv(const Segment* __restrict__ segs,
                                              const uint32_t* __restrict__ mids,
                                              const uint32_t* __restrict__ edges, uint32_t k0, uint32_t k1,
                                              RunEnds& re, uint32_t stride = 1) {
  SegReg r = load_seg<kTagged>(segs, k0, k1, stride);
  const uint32_t lane = static_cast<uint32_t>(lane_id());
  const uint32_t g = r.tag & 1u;
  r.tag = kTagged ? (((r.tag >> 1) << 7) | (lane << 1) | g) : ((lane << 1) | g);
  const uint32_t k = k0 + stride * lane;
  const bool in = k < k1;
  const uint32_t m = in ? as_global(mids)[k] : 0u;
  re.mid = m & ~kMidWide;
  if (kEdge) {
    re.edge = in ? as_global(edges)[k] : 0u;
    re.wide = m & kMidWide;
  }
  return r;
}

// Credit walk: Look(e, tag, p, n) gives the pair counts of a wedge's key
// (false: the key is not counted by this item or pass).  Credits of the
// lane's current run are kept in registers and added to the run's LDS slot
// when the lane moves to another run; with kEdge every wedge's share is
// also added to the walked entry's edge (by entry position: packed in ep,
// or in wb and wu for a wide run: bit j of `wide` for the run of lane j).
// Non-returning 64-bit add to global memory (device scope).
__device__ __forceinline__ void add_global(global_t<unsigned long long>* p, unsigned long long v) {
  __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <class Look, bool kEdge, class Acc, bool kPack = false>
struct Credit {
  Look look;
  Acc* cb;  // per-wavefront LDS: balanced credit per run lane (kPack: both,
            // balanced in the low and unbalanced in the high 32 bits)
  Acc* cu;  // unbalanced (unused with kPack)
  global_t<unsigned long long>* ep;
  global_t<unsigned long long>* wb;
  global_t<unsigned long long>* wu;
  uint64_t wide = 0;  // runs (by lane) whose credits take two words
  uint32_t cur = 0xffffffffu;  // the run of the chunk slots summed in sb, su (wave-uniform)
  Acc sb = 0, su = 0;
  // the wedge's shares: balanced b and unbalanced u (false: not a wedge of
  // this item or pass)
  __device__ __forceinline__ bool share(uint32_t e, uint32_t tag, bool valid, uint32_t& b, uint32_t& u) {
    uint32_t p, n;
    if (!valid || !look(e, tag, p, n)) return false;
    const bool sym = ((e ^ tag) & 1u) == 0;
    b = sym ? p - 1u : n - 1u;
    u = sym ? n : p;
    return true;
  }
  __device__ __forceinline__ void edge(uint32_t j, uint32_t pos, uint32_t b, uint32_t u) {
    if (kEdge) {
      if ((wide >> j) & 1u) {
        if (b) add_global(wb + pos, b);
        if (u) add_global(wu + pos, u);
      } else if (b | u) {
        add_global(ep + pos, (static_cast<unsigned long long>(u) << 32) | b);
      }
    }
  }
  // a run's LDS slot takes b and u: one 64-bit add with kPack (each half
  // stays below 2^32: the caller's runs bound their credits)
  __device__ __forceinline__ void slot_add(uint32_t j, Acc b, Acc u) {
    if constexpr (kPack) {
      if (b | u) atomicAdd(&cb[j], (u << 32) | b);
    } else {
      if (b) atomicAdd(&cb[j], b);
      if (u) atomicAdd(&cu[j], u);
    }
  }
  __device__ __forceinline__ void put() {
    if (cur != 0xffffffffu) slot_add(cur, sb, su);
    sb = su = 0;
  }
  // a staged position (lanes in different runs): its shares straight to its
  // run's LDS slot
  __device__ __forceinline__ void add(uint32_t e, uint32_t tag, bool valid, uint32_t pos) {
    uint32_t b, u;
    if (!share(e, tag, valid, b, u)) return;
    const uint32_t j = (tag >> 1) & 63u;
    slot_add(j, b, u);
    edge(j, pos, b, u);
  }
  // a chunk slot (every lane in the chunk's run): summed in registers until
  // the run changes (a wave-uniform test)
  __device__ __forceinline__ void add_chunk(uint32_t e, uint32_t tag, bool valid, uint32_t pos) {
    const uint32_t j = (tag >> 1) & 63u;
    if (j != cur) {
      put();
      cur = j;
    }
    uint32_t b, u;
    if (!share(e, tag, valid, b, u)) return;
    sb += b;
    su += u;
    edge(j, pos, b, u);
  }
  __device__ __forceinline__ void flush() {
    put();
    cur = 0xffffffffu;
  }
};

template <bool kEdge, bool kPack = false, class Look, class Acc>
__device__ __forceinline__ Credit<Look, kEdge, Acc, kPack> credit(Look l, Acc* cb, Acc* cu, const DevSideConst& sc,
                                                                  const RunEnds& re) {
  static_assert(!kPack || sizeof(Acc) == 8, "packed slots are 64-bit");
  Credit<Look, kEdge, Acc, kPack> c{l, cb, cu, as_global(sc.epack_o), as_global(sc.ewb_o), as_global(sc.ewu_o)};
  if (kEdge) c.wide = __ballot(re.wide != 0);
  return c;
}

// A run's credits b and u: to its mid (id: its input id), or with kEdge to its
// first edge (the per-edge pass has no per-vertex output).
template <bool kEdge, class Id>
__device__ __forceinline__ void run_credits_out(unsigned long long b, unsigned long long u, RunEnds re, Id id,
                                                const DevSideConst& sc) {
  if constexpr (!kEdge) {
    const int32_t mid = id();
    if (b) atomicAdd(&sc.bal_mid[mid], b);
    if (u) atomicAdd(&sc.unb_mid[mid], u);
  } else if (re.wide) {
    if (b) add_global(as_global(sc.ewb) + re.edge, b);
    if (u) add_global(as_global(sc.ewu) + re.edge, u);
  } else {  // the run's credits are below 2^32 (no wide flag)
    add_global(as_global(sc.epack) + re.edge, (u << 32) | b);
  }
}

// A batch's run credits to their mids (per-vertex; lane: its run's b, u and its
// mid's input id; every lane takes part).  The adds of a pair sit side by side and
// go out from two lanes of one instruction: an add costs its 64-byte line, 23 - 27 G
// of them a second whatever they hold, so two arrays would cost two lines a run
// (50M edges: direct 9.40 -> 8.74, reverse 15.13 -> 14.67 ms).
__device__ __forceinline__ void mid_pairs_out(uint32_t b, uint32_t u, uint32_t id, const DevSideConst& sc) {
  const uint64_t any = __ballot((b | u) != 0);
  const uint32_t lane = static_cast<uint32_t>(lane_id());
#pragma unroll
  for (uint32_t h = 0; h < 2; ++h) {
    if (static_cast<uint32_t>(any >> (32 * h)) == 0) continue;
    const uint32_t src = 32 * h + (lane >> 1);
    const uint32_t vb = bpermute(b, src), vu = bpermute(u, src), vi = bpermute(id, src);
    const uint32_t v = lane & 1u ? vu : vb;
    if (v) add_global(as_global(sc.mid_pairs) + 2 * static_cast<size_t>(vi) + (lane & 1u), v);
  }
}

// After a batch's credit walk: each lane puts its run's credits out.
template <bool kEdge, class Acc>
__device__ __forceinline__ void flush_mid_credits(Acc* cb, Acc* cu, RunEnds re, const DevSideConst& sc) {
  wave_sync_lds();
  const int lane = lane_id();
  const unsigned long long b = cb[lane], u = cu[lane];
  if (b | u) {
    cb[lane] = 0;
    cu[lane] = 0;
    run_credits_out<kEdge>(b, u, re, [&] { return sc.orig_mid[re.mid]; }, sc);
  }
  wave_sync_lds();
}

// The same for packed slots (balanced | unbalanced << 32).
template <bool kEdge>
__device__ __forceinline__ void flush_mid_credits_packed(unsigned long long* cbu, RunEnds re,
                                                         const DevSideConst& sc) {
  wave_sync_lds();
  const int lane = lane_id();
  const unsigned long long v = cbu[lane];
  if (v) {
    cbu[lane] = 0;
    run_credits_out<kEdge>(v & 0xffffffffull, v >> 32, re, [&] { return sc.orig_mid[re.mid]; }, sc);
  }
  wave_sync_lds();
}

// Completed counts of the hub pair (x, key) (dense block of the pass): the
// block's products store X = p + n and Y = p - n in hub_xy.
__device__ __forceinline__ void hub_counts(const DevSideConst& sc, uint32_t x, uint32_t key, uint32_t& p,
                                           uint32_t& n) {
  const size_t T = static_cast<size_t>(sc.T);
  const global_t<int32_t>* h = as_global(sc.hub_xy) + x * T + key;
  const int32_t X = h[0], Y = h[T * T];
  p = static_cast<uint32_t>((X + Y) / 2);
  n = static_cast<uint32_t>((X - Y) / 2);
}

// Key credits of one pair (p, n) at key vertex `key` of side s (with kEdge, the
// global sums alone).
template <bool kEdge>
struct PairCredit {
  int64_t c = 0, x = 0;  // owner sums
  __device__ __forceinline__ void add(const DevSideConst& sc, uint32_t key, uint32_t p, uint32_t n, Sums& s) {
    s.add(p, n);
    if (kEdge) return;
    const int64_t P = p, N = n;
    const int64_t cb = P * (P - 1) / 2 + N * (N - 1) / 2, cx = P * N;
    if (cb) atomicAdd(&sc.bal[sc.orig[key]], static_cast<unsigned long long>(cb));
    if (cx) atomicAdd(&sc.unb[sc.orig[key]], static_cast<unsigned long long>(cx));
    c += cb;
    x += cx;
  }
  // The wavefront's owner sums to `owner` (one atomic per wavefront).
  __device__ __forceinline__ void to_owner(const DevSideConst& sc, int32_t owner) {
    if (kEdge) return;
    const int64_t c2 = wave_sum64(c), x2 = wave_sum64(x);
    if (lane_id() == 0) {
      if (c2) atomicAdd(&sc.bal[sc.orig[owner]], static_cast<unsigned long long>(c2));
      if (x2) atomicAdd(&sc.unb[sc.orig[owner]], static_cast<unsigned long long>(x2));
    }
    c = x = 0;
  }
};

// ---------------------------------------------------------------------------
// Direct items: one workgroup per item, p and n counters over the item's
// key window, 32-bit each (at most kPVWindow keys) or, for items with fewer
// than 2^16 runs (kItemPacked), 16|16 bits in one word (at most
// kPVWindowPacked keys, the whole window of the count pass, so a pivot's
// runs are walked once per walk); windows of one pivot share their runs and
// skip the keys of the others.  The walks stage short runs in the run-table
// form (a 64-entry table per wavefront), which leaves the LDS to the
// counters.  Key credits are global atomics (the keys that many items
// share, a side's top vertices, are the dense block's when it is on).
// An item is two walks with dependent loads before each, and its wedges' credits
// were 20 instructions and an LDS round trip each.  So the next item's
// descriptor and first runs are loaded under the sweep and serve both walks; a
// packed item's counters are indexed by key and its credits take four words at a
// time (PackedCredit); and a hub pivot's completed pair counts are copied into
// its counter words, where they fit 16 bits (a plane read per wedge before).
// 50M edges, both sides: 15.6 -> 9.3 ms (without the key credits 7.8, without
// the mids' 8.0, without the credit walk 5.2).
constexpr int kPVDirectThreads = 1024;
constexpr int kPVDirectWaves = kPVDirectThreads / kWave;

// An item's wedges into C: packed 16|16-bit words by key (one window, every key
// of the item below kPVWindowPacked; masked slots go to the lane's dummy word),
// or P | N halves by the key's place in the window.  The wavefronts take the
// item's runs interleaved, so that each gets a similar mix of long and short
// ones; `first` is the wavefront's first batch.
__device__ __forceinline__ void pv_direct_tally(const Item& it, const DevSideConst& sc, uint32_t long_len,
                                                const Marks<uint8_t>& mk, SegReg first, uint32_t* C,
                                                uint32_t* dummy, bool packed) {
  const uint32_t lo = static_cast<uint32_t>(it.key_lo), hi = static_cast<uint32_t>(it.key_hi);
  const uint32_t seg_end = it.seg_begin + it.seg_count;
  uint32_t* const P = C;
  uint32_t* const N = C + kPVWindow;
  for (uint32_t k0 = it.seg_begin + threadIdx.x / kWave; k0 < seg_end;) {
    if (packed)
      walk_regs<8, false, true>(first, sc.other_adj, mk, long_len, DirectTallyBF<kPVWindowPacked>{C, dummy});
    else
      walk_regs<4, false, true>(first, sc.other_adj, mk, long_len, hash_tally([&](uint32_t e, uint32_t tag) {
                                  const uint32_t key = e >> 1;
                                  if (key >= lo && key < hi) atomicAdd(((e ^ tag) & 1u) ? &N[key - lo] : &P[key - lo], 1u);
                                }));
    k0 += kPVDirectThreads;
    if (k0 < seg_end) first = load_seg<false>(sc.segs, k0, seg_end, kPVDirectWaves);
  }
}

// Credit walk of a packed item's batch.  A wedge's shares are its key's counter
// word, turned so that its own sign's count is the low half, less 1 (its own
// wedge): balanced | unbalanced << 16.  A chunk's four words are read before any
// is used, and its run's sums stay in registers until the run ends; then the
// run's lane takes the wavefront's sums.  Staged shares that are not zero go to
// their run's LDS slot.
template <bool kEdge>
struct PackedCredit {
  static constexpr bool kStaged = true, kChunk4 = true;
  // a run has at most one entry per key of the window, p and n are below 2^16
  static_assert(uint64_t{kPVWindowPacked} * 65535 < (uint64_t{1} << 32), "a run's credits fit 32 bits");
  const uint32_t* C;
  unsigned long long* cbu;           // per run lane: balanced | unbalanced << 32
  global_t<unsigned long long>* ep;  // per-edge credits, as in Credit
  global_t<unsigned long long>* wb;
  global_t<unsigned long long>* wu;
  uint64_t wide = 0;
  uint32_t cur = kNoRun, sb = 0, su = 0, slots = 0;  // the chunks' run (wavefront-uniform), its sums and slots per lane
  uint32_t mb = 0, mu = 0;                           // this lane's run: the chunks' credits
  static constexpr uint32_t kNoRun = 0xffffffffu;
  __device__ __forceinline__ uint32_t word(uint32_t e) const { return C[(e >> 1) & (kPVWindowPacked - 1)]; }
  // own sign's count | other sign's << 16
  static __device__ __forceinline__ uint32_t counts(uint32_t w, uint32_t e, uint32_t g) {
    return __builtin_amdgcn_alignbit(w, w, ((e << 4) + (g << 4)) & 31u);
  }
  __device__ __forceinline__ void edge(uint32_t j, uint32_t pos, uint32_t s) const {
    if (!kEdge || s == 0) return;
    const uint32_t b = s & 0xffffu, u = s >> 16;
    if ((wide >> j) & 1u) {
      if (b) add_global(wb + pos, b);
      if (u) add_global(wu + pos, u);
    } else {
      add_global(ep + pos, (static_cast<unsigned long long>(u) << 32) | b);
    }
  }
  __device__ __forceinline__ void put() {
    if (cur == kNoRun) return;
    const uint32_t b = wave_sum32(sb - slots), u = wave_sum32(su);
    sb = su = slots = 0;
    const bool own = static_cast<uint32_t>(lane_id()) == cur;
    mb += own ? b : 0u;
    mu += own ? u : 0u;
  }
  __device__ __forceinline__ void add_chunk4(const uint32_t (&e)[4], uint32_t tag, uint32_t rem,
                                             const uint32_t (&off)[4], uint32_t pos) {
    const uint32_t j = (tag >> 1) & 63u, g = tag & 1u;
    if (j != cur) {
      put();
      cur = j;
    }
    uint32_t w[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) w[q] = word(e[q]);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t c = off[q] < rem ? counts(w[q], e[q], g) : 1u;
      sb += c & 0xffffu;
      su += c >> 16;
      edge(j, pos + off[q], c - 1u);
    }
    slots += 4;
  }
  __device__ __forceinline__ void add_staged(const Staged& s) {
    uint32_t w[kStageU];
#pragma unroll
    for (int q = 0; q < kStageU; ++q) w[q] = word(s.valid[q] ? s.e[q] : 0u);
#pragma unroll
    for (int q = 0; q < kStageU; ++q) {
      if (!s.valid[q]) continue;
      const uint32_t c = counts(w[q], s.e[q], s.tag[q] & 1u) - 1u;
      if (c != 0) {
        const uint32_t j = (s.tag[q] >> 1) & 63u;
        atomicAdd(&cbu[j], (static_cast<unsigned long long>(c >> 16) << 32) | (c & 0xffffu));
        edge(j, s.pos[q], c);
      }
    }
  }
};

// Heavy items.  An item runs on one CU, so a pivot with more than a CU's
// share of the wedges would outlast its launch (2M edges, per-edge pass:
// 1.14 ms for one item of 0.95M wedges, the others' work 0.3 ms).  Such items
// are cut into parts: this launch tallies the parts and adds their counters
// into the accumulator of the item's key window (consecutive keys, a few cache
// lines per instruction; unpacked: p, then n from the next 16-byte piece); the
// main launch's parts load the whole counters, credit their own runs' wedges,
// and sweep a slice of the keys.
__device__ __forceinline__ uint32_t pv_acc_half(uint32_t keys) { return (keys + 3u) & ~3u; }

__global__ __launch_bounds__(kPVDirectThreads) void k_pv_heavy_tally(DirectArgs a) {
  __shared__ uint32_t C[kPVWindowPacked];
  __shared__ __attribute__((aligned(16))) uint32_t mtab[kPVDirectWaves][2 * kWave];
  __shared__ uint8_t mflag[kPVDirectWaves][kGather];
  __shared__ uint32_t dummies[kPVDirectThreads];
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  for (int i = tid; i < kPVWindowPacked; i += kPVDirectThreads) C[i] = 0;
  for (int i = tid; i < kPVDirectWaves * static_cast<int>(kGather); i += kPVDirectThreads) (&mflag[0][0])[i] = 0;
  __syncthreads();
  for (int32_t i = blockIdx.x; i < a.n_items; i += gridDim.x) {
    const Item it = load_const(a.items, i);
    const DevSideConst sc = load_const(a.sides, 2 * it.graph + it.side);
    const bool packed = (it.flags & kItemPacked) != 0;
    pv_direct_tally(it, sc, a.long_len, Marks<uint8_t>{mtab[wave], mflag[wave]},
                    load_seg<false>(sc.segs, it.seg_begin + wave, it.seg_begin + it.seg_count, kPVDirectWaves), C,
                    &dummies[tid], packed);
    __syncthreads();
    global_t<uint32_t>* to = as_global(sc.acc) + static_cast<size_t>(it.acc_slot) * sc.acc_width;
    // packed: words by key; unpacked: by the key's place in the window
    const uint32_t lo = packed ? static_cast<uint32_t>(it.key_lo) : 0u;
    const uint32_t keys = static_cast<uint32_t>(packed ? it.key_hi : it.key_hi - it.key_lo);
    for (int h = 0; h < (packed ? 1 : 2); ++h) {
      uint32_t* const from = C + h * kPVWindow;
      for (uint32_t k = lo + tid; k < keys; k += kPVDirectThreads) {
        const uint32_t v = from[k];
        if (v) {
          from[k] = 0;
          __hip_atomic_fetch_add(to + h * pv_acc_half(keys) + k, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
    }
    __syncthreads();
  }
}

template <bool kEdge>
__global__ __launch_bounds__(kPVDirectThreads) void k_pv_direct(DirectArgs a) {
  a.res = own_copy(a.res, a.res_mask);
  __shared__ uint32_t C[kPVWindowPacked];  // P | N, or packed words
  __shared__ __attribute__((aligned(16))) uint32_t mtab[kPVDirectWaves][2 * kWave];
  __shared__ uint8_t mflag[kPVDirectWaves][kGather];
  // cu: unpacked items' unbalanced slots; a packed item's tally takes them for
  // dummy words
  __shared__ unsigned long long cb[kPVDirectWaves][kWave], cu[kPVDirectWaves][kWave];
  __shared__ int32_t item_sh;
  static_assert(2 * kPVWindow == kPVWindowPacked, "P | N halves fill the packed window");
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int lane = lane_id();
  for (int i = tid; i < kPVWindowPacked; i += kPVDirectThreads) C[i] = 0;
  uint32_t* const P = C;
  uint32_t* const N = C + kPVWindow;
  for (int i = tid; i < kPVDirectWaves * static_cast<int>(kGather); i += kPVDirectThreads) (&mflag[0][0])[i] = 0;
  cb[wave][lane] = 0;
  const Marks<uint8_t> mk{mtab[wave], mflag[wave]};
  int64_t tot_b = 0, tot_u = 0;  // this lane's pairs of the current graph
  uint32_t graph = kNoGraph;
  constexpr int kItemWords = sizeof(Item) / 4;
  // the words of item i, one per lane
  auto fetch = [&](int32_t i) {
    return i < a.n_items && lane < kItemWords
               ? as_global(reinterpret_cast<const uint32_t*>(a.items))[static_cast<size_t>(i) * kItemWords + lane]
               : 0u;
  };
  auto unpack = [&](uint32_t w) {
    Item it;
    uint32_t* o = reinterpret_cast<uint32_t*>(&it);
#pragma unroll
    for (int k = 0; k < kItemWords; ++k) o[k] = readlane(w, k);
    return it;
  };
  auto load_runs = [&](const Item& it, const DevSideConst& sc, uint32_t k0, RunEnds& re) {
    return load_seg_pv<false, kEdge>(sc.segs, sc.seg_mid, sc.seg_edge, k0, it.seg_begin + it.seg_count, re,
                                     kPVDirectWaves);
  };
  if (tid == 0) item_sh = static_cast<int32_t>(atomicAdd(a.queue, 1u));
  __syncthreads();
  int32_t i = __builtin_amdgcn_readfirstlane(item_sh);
  Item it{};
  DevSideConst sc{};
  RunEnds fre;
  SegReg first{0, 0, 0};
  if (i < a.n_items) {
    it = unpack(fetch(i));
    sc = load_const(a.sides, 2 * it.graph + it.side);
    first = load_runs(it, sc, it.seg_begin + wave, fre);
    graph = it.graph;
  }
  while (i < a.n_items) {
    if (it.graph != graph) {
      flush_sums(Sums{tot_b, tot_u}, a.res + static_cast<size_t>(graph) * kResStride);
      tot_b = tot_u = 0;
      graph = it.graph;
    }
    const uint32_t lo = static_cast<uint32_t>(it.key_lo), hi = static_cast<uint32_t>(it.key_hi);
    const uint32_t seg_end = it.seg_begin + it.seg_count;
    const bool packed = (it.flags & kItemPacked) != 0;
    // a hub pivot's keys below T are hub pairs: their completed counts come
    // from the dense block and their key credits were given there
    const uint32_t hubT = (it.flags & kItemHubPairs) ? static_cast<uint32_t>(sc.T) : 0u;
    const bool part = (it.flags & kItemMultiPart) != 0;
    if (part) {
      // a part of a heavy item: the tally launch before this one left the
      // item's whole counts in its accumulator (packed: by key, zeros below lo)
      const u32x4* from = reinterpret_cast<const u32x4*>(sc.acc + static_cast<size_t>(it.acc_slot) * sc.acc_width);
      const uint32_t k_begin = packed ? lo & ~3u : 0u, k_end = packed ? hi : hi - lo;
      for (uint32_t k = k_begin + 4 * tid; k < k_end; k += 4 * kPVDirectThreads) {
        *reinterpret_cast<u32x4*>(&C[k]) = *as_global(from + k / 4);
        if (!packed) *reinterpret_cast<u32x4*>(&N[k]) = *as_global(from + (pv_acc_half(hi - lo) + k) / 4);
      }
    } else {
      pv_direct_tally(it, sc, a.long_len, mk, first, C, reinterpret_cast<uint32_t*>(&cu[wave][lane]), packed);
    }
    __syncthreads();
    // the hub pairs' counts take their words, unless one has 2^16 wedges or more
    bool fast = packed;
    if (packed && hubT > lo) {
      const size_t TT = static_cast<size_t>(sc.T) * sc.T;
      const global_t<int32_t>* xy = as_global(sc.hub_xy) + static_cast<size_t>(it.owner) * sc.T;
      int32_t big = 0;
      for (uint32_t k = lo + tid; k < hubT; k += kPVDirectThreads) {
        const int32_t X = xy[k], Y = xy[TT + k];
        big |= X >> 16;
        C[k] = static_cast<uint32_t>((X + Y) / 2) | (static_cast<uint32_t>((X - Y) / 2) << 16);
      }
      fast = __syncthreads_or(big) == 0;
    }
    // credit the mids
    uint32_t ticket = 0;
    SegReg sr = first;
    RunEnds re = fre;
    if (!fast) cu[wave][lane] = 0;
    for (uint32_t k0 = it.seg_begin + wave;;) {
      const bool last = k0 >= seg_end || seg_end - k0 <= kPVDirectThreads;
      if (last && tid == 0) ticket = atomicAdd(a.queue, 1u);
      if (k0 < seg_end) {
        if (fast) {
          PackedCredit<kEdge> c{C, cb[wave], as_global(sc.epack_o), as_global(sc.ewb_o), as_global(sc.ewu_o)};
          if (kEdge) c.wide = __ballot(re.wide != 0);
          walk_regs<kEdge ? 4 : 8, kEdge, true>(sr, sc.other_adj, mk, a.long_len, c);
          c.put();
          wave_sync_lds();
          const unsigned long long v = cb[wave][lane];
          const uint32_t b = c.mb + static_cast<uint32_t>(v), u = c.mu + static_cast<uint32_t>(v >> 32);
          if (v) cb[wave][lane] = 0;
          if constexpr (kEdge) {
            if (b | u) run_credits_out<kEdge>(b, u, re, [] { return 0; }, sc);
          } else {
            mid_pairs_out(b, u, b | u ? static_cast<uint32_t>(as_global(sc.orig_mid)[re.mid]) : 0u, sc);
          }
          wave_sync_lds();
        } else {
          auto c = credit<kEdge>(
              [&](uint32_t e, uint32_t, uint32_t& p, uint32_t& n) {
                const uint32_t key = e >> 1;
                if (key < lo || key >= hi) return false;
                if (key < hubT) {
                  hub_counts(sc, static_cast<uint32_t>(it.owner), key, p, n);
                  return true;
                }
                if (packed) {
                  const uint32_t v = C[key];
                  p = v & 0xffffu;
                  n = v >> 16;
                } else {
                  p = P[key - lo];
                  n = N[key - lo];
                }
                return true;
              },
              cb[wave], cu[wave], sc, re);
          walk_regs<4, kEdge, true>(sr, sc.other_adj, mk, a.long_len, c);
          c.flush();
          flush_mid_credits<kEdge>(cb[wave], cu[wave], re, sc);
        }
      }
      if (last) break;
      k0 += kPVDirectThreads;
      sr = load_runs(it, sc, k0, re);
    }
    if (tid == 0) item_sh = static_cast<int32_t>(ticket);
    __syncthreads();
    i = __builtin_amdgcn_readfirstlane(item_sh);
    const uint32_t next_words = fetch(i);
    // credit the keys and the owner (packed counts: p + n < 2^16, so a
    // key's credits fit 32 bits).  Key credits go to the rank-indexed sums
    // (the threads' keys are consecutive: one instruction's atomics touch a
    // few cache lines, where input-id order would scatter them over 64).
    // A part sweeps its slice of the keys, and clears them all.
    PairCredit<kEdge> pc;
    uint32_t k_lo = lo, k_hi = hi;
    if (part) {
      const uint32_t idx = it.work >> 16, n = it.work & 0xffffu, step = (hi - lo + n - 1) / n;
      k_lo = min(hi, lo + idx * step);
      k_hi = min(hi, k_lo + step);
    }
    k_lo = max(k_lo, hubT);  // hub pairs are credited by the dense block
    if (packed) {
      for (uint32_t k = lo + tid; k < hi; k += kPVDirectThreads) {
        const uint32_t v = C[k];
        if (v == 0) continue;
        C[k] = 0;
        if (k < k_lo || k >= k_hi) continue;
        const uint32_t p = v & 0xffffu, n = v >> 16;
        const uint32_t cb2 = (mul24(p, p - 1u) + mul24(n, n - 1u)) >> 1, cx = mul24(p, n);
        if (!kEdge && cb2) atomicAdd(&sc.key_bal[k], static_cast<unsigned long long>(cb2));
        if (!kEdge && cx) atomicAdd(&sc.key_unb[k], static_cast<unsigned long long>(cx));
        pc.c += cb2;
        pc.x += cx;
      }
    } else {
      for (uint32_t k = lo + tid; k < hi; k += kPVDirectThreads) {
        const int64_t p = P[k - lo], n = N[k - lo];
        if ((p | n) == 0) continue;
        P[k - lo] = N[k - lo] = 0;
        if (k < k_lo || k >= k_hi) continue;
        const int64_t cb2 = p * (p - 1) / 2 + n * (n - 1) / 2, cx = p * n;
        if (!kEdge && cb2) atomicAdd(&sc.key_bal[k], static_cast<unsigned long long>(cb2));
        if (!kEdge && cx) atomicAdd(&sc.key_unb[k], static_cast<unsigned long long>(cx));
        pc.c += cb2;
        pc.x += cx;
      }
    }
    tot_b += pc.c;
    tot_u += pc.x;
    pc.to_owner(sc, it.owner);
    if (i < a.n_items) {
      it = unpack(next_words);
      sc = load_const(a.sides, 2 * it.graph + it.side);
      first = load_runs(it, sc, it.seg_begin + wave, fre);
    }
    __syncthreads();
  }
  __shared__ WaveSums wsum[kPVDirectWaves];
  flush_block_end(wave_sum64(tot_b), wave_sum64(tot_u), graph, wsum, kPVDirectWaves, a.res);
}

// The direct items' key credits of both sides (blockIdx.y; by rank, ranks below
// n, zero past a side's window) into the per-vertex outputs (input-id order).
__global__ void k_pv_key_flush(const DevSideConst* sides, int32_t n) {
  const DevSideConst sc = load_const(sides, blockIdx.y);
  for (int32_t k = blockIdx.x * blockDim.x + threadIdx.x; k < n; k += gridDim.x * blockDim.x) {
    const unsigned long long b = sc.key_bal[k], u = sc.key_unb[k];
    if (b | u) {
      const int32_t id = sc.orig[k];
      if (b) atomicAdd(&sc.bal[id], b);
      if (u) atomicAdd(&sc.unb[id], u);
    }
  }
}

__global__ void k_vertex_out(VertexOutArgs a) {
  const int32_t first = static_cast<int32_t>(blockIdx.x * blockDim.x + threadIdx.x);
  const int32_t step = static_cast<int32_t>(gridDim.x * blockDim.x);
  for (int s = 0; s < 2; ++s)
    for (int32_t i = first; i < a.n[s]; i += step) {
      const ulonglong2 mid = reinterpret_cast<const ulonglong2*>(a.mid[s])[i];
      if (a.out[s][0]) a.out[s][0][i] = a.acc[s][0][i] + mid.x;
      if (a.out[s][1]) a.out[s][1][i] = a.acc[s][1][i] + mid.y;
    }
  for (int32_t i = first; i < a.words; i += step) a.to[i] = a.from[i];
}

// ---------------------------------------------------------------------------
// Reverse items (at most kReverseMaxSegs runs): one wavefront per item, 8-bit
// p and n per key over the reverse window, two keys per 32-bit word.  The
// keys are the reverse window's vertices, shared by every item of a side, so
// their credits are summed per workgroup in LDS and reach HBM once per
// workgroup at the end (a launch holds the items of one side).  A pair's
// credit is below 2^15 (p + n <= 255), so the workgroup's 32-bit key sums
// hold up to kPVReverseBlockItems items (the launch sizes its grid for that).
// Bound by instruction issue at the 12 wavefronts per CU that the LDS holds
// (VALU busy half of the time) and by an item's chain of dependent loads.  So the
// next item's descriptor, first runs and mids are loaded under the current item
// and serve both walks; the tally's first staging rounds stay in registers for
// the credit walk; that walk takes a wedge's shares out of a counter word with
// one byte permutation; and the item's totals are half its runs' credits.
// 50M edges, both sides: 22.4 -> 15.6 ms (the loads 18.6, the credit walk 16.5,
// the sweep's test of whole words 15.6); 2M edges, per-edge: 0.53 -> 0.41 ms.
constexpr int kPVReverseWaves = 12;
constexpr int kPVReverseThreads = kPVReverseWaves * kWave;
constexpr int kPVReverseWords = kMaxReverseL / 2;
constexpr int64_t kPVReverseBlockItems = int64_t{1} << 16;
// (wavefronts take items in turn: one more each at most)
static_assert((kPVReverseBlockItems + kPVReverseWaves) * (kReverseMaxSegs * (kReverseMaxSegs - 1) / 2) <
                  (int64_t{1} << 32),
              "a workgroup's key credits fit 32 bits");
// staging rounds whose entries stay in registers from the tally to the credits
// (50M edges, per-vertex, side U: 10.9 ms with none, 10.5 with 1 or 2, 10.6 with 3,
// 11.0 with 4, which spill; per-edge 20M: 6.69, 6.62, 7.02 ms with 0, 1, 2)
constexpr int pv_reverse_kept(bool edge) { return edge ? 1 : 2; }

// Credit walk of a reverse batch.  A wedge's shares are one byte permutation of
// its key's counter word: byte p | n << 8 of the key's half, as own sign's count
// | other's << 16; less 1 (its own wedge), that is its balanced | unbalanced << 16.
// A chunk's four counter words are read before any is used, and its run's sums
// stay in registers until the run ends; then the run's lane takes the wavefront's
// sums.  Staged shares that are not zero go to their run's LDS slot.
template <bool kEdge>
struct ReverseCredit {
  static constexpr bool kStaged = true, kChunk4 = true;
  // ... the keys of the reverse window, and p, n are at most the item's runs
  static_assert(uint64_t{kMaxReverseL} * kReverseMaxSegs < (uint64_t{1} << 32), "a run's credits fit 32 bits");
  uint32_t base;             // LDS address of the counter words, aligned to their size
  unsigned long long* cbu;   // per run lane: balanced | unbalanced << 32
  global_t<unsigned long long>* ep;  // per-edge credits, as in Credit
  global_t<unsigned long long>* wb;
  global_t<unsigned long long>* wu;
  uint64_t wide = 0;
  uint32_t cur = kNoRun, sb = 0, su = 0, slots = 0;  // the chunks' run (wavefront-uniform), its sums and slots per lane
  uint32_t mb = 0, mu = 0;         // this lane's run: the chunks' credits
  static constexpr uint32_t kNoRun = 0xffffffffu;
  __device__ __forceinline__ uint32_t word(uint32_t e) const {
    return *(const lds_u32*)static_cast<uintptr_t>(base | (e & (4 * kPVReverseWords - 4)));
  }
  // own sign's count | other sign's << 16
  static __device__ __forceinline__ uint32_t counts(uint32_t w, uint32_t e, uint32_t g) {
    const uint32_t t = (e ^ g) & 3u;  // g is 0 or 1: key parity, asymmetric
    return __builtin_amdgcn_perm(w, w, 0x0c010c00u ^ (t | (t << 16)));
  }
  __device__ __forceinline__ void edge(uint32_t j, uint32_t pos, uint32_t s) const {
    if (!kEdge || s == 0) return;
    const uint32_t b = s & 0xffffu, u = s >> 16;
    if ((wide >> j) & 1u) {
      if (b) add_global(wb + pos, b);
      if (u) add_global(wu + pos, u);
    } else {
      add_global(ep + pos, (static_cast<unsigned long long>(u) << 32) | b);
    }
  }
  __device__ __forceinline__ void put() {
    if (cur == kNoRun) return;
    const uint32_t b = wave_sum32(sb - slots), u = wave_sum32(su);
    sb = su = slots = 0;
    const bool own = static_cast<uint32_t>(lane_id()) == cur;
    mb += own ? b : 0u;
    mu += own ? u : 0u;
  }
  __device__ __forceinline__ void add_chunk4(const uint32_t (&e)[4], uint32_t tag, uint32_t rem,
                                             const uint32_t (&off)[4], uint32_t pos) {
    const uint32_t j = (tag >> 1) & 63u, g = tag & 1u;
    if (j != cur) {
      put();
      cur = j;
    }
    uint32_t w[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) w[q] = word(e[q]);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t c = off[q] < rem ? counts(w[q], e[q], g) : 1u;
      const u16x2 h = __builtin_bit_cast(u16x2, c);
      sb = __builtin_amdgcn_udot2(h, u16x2{1, 0}, sb, false);
      su = __builtin_amdgcn_udot2(h, u16x2{0, 1}, su, false);
      edge(j, pos + off[q], c - 1u);
    }
    slots += 4;
  }
  __device__ __forceinline__ void add_staged(const Staged& s) {
    uint32_t w[kStageU];
#pragma unroll
    for (int q = 0; q < kStageU; ++q) w[q] = word(s.valid[q] ? s.e[q] : 0u);
#pragma unroll
    for (int q = 0; q < kStageU; ++q) {
      const uint32_t c = counts(w[q], s.e[q], s.tag[q] & 1u) - 1u;
      if (s.valid[q] && c != 0) {
        const uint32_t j = (s.tag[q] >> 1) & 63u;
        atomicAdd(&cbu[j], (static_cast<unsigned long long>(c >> 16) << 32) | (c & 0xffffu));
        edge(j, s.pos[q], c);
      }
    }
  }
};

template <bool kEdge>
__global__ __launch_bounds__(kPVReverseThreads) void k_pv_reverse(SmallArgs a) {
  a.res = own_copy(a.res, a.res_mask);
  // counters, each wavefront's array aligned to its size (the tally's
  // AND-OR addresses); one dummy word per lane
  __shared__ __attribute__((aligned(kPVReverseWords * 4))) uint32_t cnt[kPVReverseWaves][kPVReverseWords];
  __shared__ uint32_t dummies[kPVReverseWaves][kWave];
  __shared__ __attribute__((aligned(16))) uint32_t mtab[kPVReverseWaves][kGather];
  __shared__ uint8_t mflag[kPVReverseWaves][kGather];
  // a run's mid credits of staged wedges, balanced | unbalanced << 32: each at
  // most the run's length (at most 4096) times 255
  __shared__ unsigned long long cbu[kPVReverseWaves][kWave];
  // the workgroup's key credits, balanced | unbalanced << 32
  __shared__ unsigned long long ksum[kEdge ? 1 : kMaxReverseL];
  // chunk slots in flight per walk: as many as the registers allow (the
  // per-edge walks keep positions too)
  constexpr int kU = kEdge ? 4 : 6;
  // wave index, known to the compiler as wavefront-uniform
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWave);
  const int lane = lane_id();
  uint32_t* C = cnt[wave];
  if (lane == 0 && (lds_addr(C) & (kPVReverseWords * 4 - 1)) != 0) atomicOr(a.err, kErrLdsLayout);
  for (int i = threadIdx.x; i < (kEdge ? 1 : kMaxReverseL); i += kPVReverseThreads) ksum[i] = 0;
  for (int i = lane; i < kPVReverseWords; i += kWave) C[i] = 0;
  for (int i = lane; i < static_cast<int>(kGather); i += kWave) mflag[wave][i] = 0;
  cbu[wave][lane] = 0;
  wave_sync_lds();
  const Marks<uint8_t> mk{mtab[wave], mflag[wave]};
  int64_t tot_b = 0, tot_u = 0;  // the pass's global counts (wavefront-uniform)
  uint32_t graph = kNoGraph;
  const int32_t n = a.n_items, stride = static_cast<int32_t>(gridDim.x) * kPVReverseWaves;
  int32_t i = static_cast<int32_t>(blockIdx.x) * kPVReverseWaves + wave;
  // The next item's descriptor and first 64 runs are loaded under the current
  // item; both walks of an item's first runs share one load.
  const auto first_runs = [&](const Item& t, const DevSideConst& sc, RunEnds& re) {
    const uint32_t e = t.seg_begin + t.seg_count;
    return load_seg_pv<false, kEdge>(sc.segs, sc.seg_mid, sc.seg_edge, t.seg_begin,
                                     t.seg_begin + kWave < e ? t.seg_begin + kWave : e, re);
  };
  Item nxt{};
  SegReg nseg{0, 0, 0};
  RunEnds nre;
  Item cur{};
  if (i < n) {
    cur = load_const(a.items, i);
    nseg = first_runs(cur, load_const(a.sides, 2 * cur.graph + cur.side), nre);
  }
  if (i + stride < n) nxt = load_const(a.items, i + stride);
  for (; i < n; i += stride) {
    const Item it = cur;
    if (it.graph != graph) {
      if (graph != kNoGraph && lane == 0) {
        unsigned long long* res = a.res + static_cast<size_t>(graph) * kResStride;
        if (tot_b) atomicAdd(res + kResBalanced, static_cast<unsigned long long>(tot_b));
        if (tot_u) atomicAdd(res + kResUnbalanced, static_cast<unsigned long long>(tot_u));
      }
      tot_b = tot_u = 0;
      graph = it.graph;
    }
    const DevSideConst sc = load_const(a.sides, 2 * it.graph + it.side);
    SegReg sr = nseg;
    RunEnds re = nre;
    // where the item's credits go, known before they are
    const int32_t owner_id = kEdge ? 0 : *(const const_t<int32_t>*)(sc.orig + it.owner);
    int32_t mid_id = kEdge ? 0 : as_global(sc.orig_mid)[re.mid];
    if (i + stride < n) nseg = first_runs(nxt, load_const(a.sides, 2 * nxt.graph + nxt.side), nre);
    cur = nxt;
    if (i + 2 * stride < n) nxt = load_const(a.items, i + 2 * stride);
    const uint32_t seg_end = it.seg_begin + it.seg_count;
    const auto load_runs = [&](uint32_t k) {
      sr = load_seg_pv<false, kEdge>(sc.segs, sc.seg_mid, sc.seg_edge, k, k + kWave < seg_end ? k + kWave : seg_end, re);
      if (!kEdge) mid_id = as_global(sc.orig_mid)[re.mid];
    };
    // tally
    KeptRounds<pv_reverse_kept(kEdge), kEdge> kept;
    uint32_t k0 = it.seg_begin;
    for (;;) {
      walk_regs<kU, false, true>(sr, sc.other_adj, mk, a.long_len,
                                 PairTallyBF<kPVReverseWords>{lds_addr(C), lds_addr(&dummies[wave][lane])}, kept);
      if (k0 + kWave >= seg_end) break;
      k0 += kWave;
      load_runs(k0);
    }
    wave_sync_lds();
    // credits, the last batch first: its runs are at hand, and its first
    // staging rounds are kept
    uint32_t cb = 0, cu = 0;  // the credits of this lane's runs
    for (bool replay = true;; replay = false) {
      ReverseCredit<kEdge> c{lds_addr(C), cbu[wave], as_global(sc.epack_o), as_global(sc.ewb_o), as_global(sc.ewu_o)};
      if (kEdge) c.wide = __ballot(re.wide != 0);
      walk_regs<kU, kEdge, false, true>(sr, sc.other_adj, mk, a.long_len, c, kept, replay);
      c.put();
      wave_sync_lds();
      const unsigned long long v = cbu[wave][lane];
      cbu[wave][lane] = 0;
      const uint32_t b = c.mb + static_cast<uint32_t>(v), u = c.mu + static_cast<uint32_t>(v >> 32);
      if constexpr (kEdge) {
        if (b | u) run_credits_out<kEdge>(b, u, re, [] { return 0; }, sc);
      } else {
        mid_pairs_out(b, u, static_cast<uint32_t>(mid_id), sc);
      }
      cb += b;
      cu += u;
      wave_sync_lds();
      if (k0 == it.seg_begin) break;
      k0 -= kWave;
      load_runs(k0);
    }
    // The keys' credits, two 16-byte pieces of counter words per lane and step
    // (words past the item's keys are zero).  A pair with one wedge adds nothing
    // to its key: a word is looked at if one of its bytes is 2 or more, or both
    // of a key's are 1.
    auto local = [&](uint32_t key, uint32_t c) {  // c = p | n << 8
      const uint32_t p = c & 0xffu, n = c >> 8;
      const uint32_t cb2 = (__builtin_amdgcn_udot4(c, c, 0u, false) - p - n) >> 1, cx = mul24(p, n);
      atomicAdd(&ksum[key], (static_cast<unsigned long long>(cx) << 32) | cb2);
    };
    const uint32_t w_hi = static_cast<uint32_t>(it.key_hi + 1) >> 1;
    for (uint32_t w0 = 0; w0 < w_hi; w0 += 8 * kWave) {
      uint32_t cw[8], hit[8];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        uint4* at = reinterpret_cast<uint4*>(&C[w0 + static_cast<uint32_t>(4 * (h * kWave + lane))]);
        const uint4 c4 = *at;
        *at = make_uint4(0, 0, 0, 0);
        if (kEdge) continue;  // no per-vertex output
        cw[4 * h] = c4.x, cw[4 * h + 1] = c4.y, cw[4 * h + 2] = c4.z, cw[4 * h + 3] = c4.w;
      }
      if (kEdge) continue;
#pragma unroll
      for (int q = 0; q < 8; ++q) hit[q] = (cw[q] & 0xfefefefeu) | (cw[q] & (cw[q] >> 8) & 0x00010001u);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if ((hit[4 * h] | hit[4 * h + 1] | hit[4 * h + 2] | hit[4 * h + 3]) == 0) continue;
#pragma unroll
        for (int q = 4 * h; q < 4 * h + 4; ++q) {
          if (hit[q] == 0) continue;
          const uint32_t key = 2 * (w0 + static_cast<uint32_t>(4 * (h * kWave + lane) + q - 4 * h));
          local(key, cw[q] & 0xffffu);
          local(key + 1, cw[q] >> 16);
        }
      }
    }
    // The owner's credits, and the pass's totals: a butterfly of the item
    // credits its two mids.
    static_assert(uint64_t{kReverseMaxSegs} * kMaxReverseL * kReverseMaxSegs < (uint64_t{1} << 32),
                  "an item's credits fit 32 bits");
    const uint32_t item_b = wave_sum32(cb) / 2, item_u = wave_sum32(cu) / 2;
    tot_b += item_b;
    tot_u += item_u;
    if (!kEdge && lane == 0) {
      if (item_b) add_global(as_global(sc.bal) + owner_id, item_b);
      if (item_u) add_global(as_global(sc.unb) + owner_id, item_u);
    }
    wave_sync_lds();
  }
  __shared__ WaveSums wsum[kPVReverseWaves];
  flush_block_end(tot_b, tot_u, graph, wsum, kPVReverseWaves, a.res);
  if (kEdge) return;
  // the workgroup's key credits (all items of a launch are of one side)
  __syncthreads();
  if (a.n_items > 0) {
    const Item i0 = load_const(a.items, 0);
    const DevSideConst sc = load_const(a.sides, 2 * i0.graph + i0.side);
    const int32_t nkeys = sc.R < kMaxReverseL ? sc.R : kMaxReverseL;
    for (int k = threadIdx.x; k < nkeys; k += kPVReverseThreads) {
      const unsigned long long v = ksum[k], b = v & 0xffffffffull, u = v >> 32;
      if (b) atomicAdd(&sc.bal[sc.orig[k]], b);
      if (u) atomicAdd(&sc.unb[sc.orig[k]], u);
    }
  }
}

// ---------------------------------------------------------------------------
// Small-item groups: one wavefront per group, the group hash of the count
// pass; owners come from the group's owner list.
constexpr int kPVSmallThreads = 256;
constexpr int kPVSmallWaves = kPVSmallThreads / kWave;
constexpr int kPVSmallSlots = 2 * kSmallGroupWork;

// kTeam wavefronts take a group together, as in the count pass (small_team).
template <bool kEdge, int kTeam>
__global__ __launch_bounds__(kPVSmallThreads) void k_pv_small(SmallArgs a) {
  a.res = own_copy(a.res, a.res_mask);
  __shared__ uint32_t keys[kPVSmallWaves / kTeam][kPVSmallSlots];
  __shared__ uint32_t vals[kPVSmallWaves / kTeam][kPVSmallSlots];
  __shared__ __attribute__((aligned(16))) uint32_t mtab[kPVSmallWaves][kGather];
  __shared__ uint32_t mflag[kPVSmallWaves][kGather];
  __shared__ unsigned long long cb[kPVSmallWaves][kWave], cu[kPVSmallWaves][kWave];
  // wave index, known to the compiler as wavefront-uniform
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWave);
  const int lane = lane_id();
  const int member = wave % kTeam;
  uint32_t* K = keys[wave / kTeam];
  uint32_t* V = vals[wave / kTeam];
  const auto team_sync = [] {
    if (kTeam == 1)
      wave_sync_lds();
    else
      __syncthreads();
  };
  static_assert(kTeam == 1 || kTeam == kPVSmallWaves, "a team's barrier is the workgroup's");
  for (int i = member * kWave + lane; i < kPVSmallSlots; i += kTeam * kWave) {
    K[i] = kEmpty;
    V[i] = 0;
  }
  for (int i = lane; i < static_cast<int>(kGather); i += kWave) mflag[wave][i] = 0;
  cb[wave][lane] = 0;
  cu[wave][lane] = 0;
  team_sync();
  const Marks<uint32_t> mk{mtab[wave], mflag[wave]};
  Sums sums;
  uint32_t graph = kNoGraph;
  constexpr int kTeams = kPVSmallWaves / kTeam;
  const int32_t stride = static_cast<int32_t>(gridDim.x) * kTeams;
  for (int32_t i = static_cast<int32_t>(blockIdx.x) * kTeams + wave / kTeam; i < a.n_items; i += stride) {
    const Item it = load_const(a.items, i);
    if (it.graph != graph) {
      if (graph != kNoGraph) flush_sums(sums, a.res + static_cast<size_t>(graph) * kResStride);
      sums = Sums{};
      graph = it.graph;
    }
    const DevSideConst sc = load_const(a.sides, 2 * it.graph + it.side);
    const uint32_t kb = static_cast<uint32_t>(sc.key_bits);
    uint32_t size = 64;
    while (size < 2 * it.work) size <<= 1;
    const uint32_t mask = size - 1;
    const uint32_t seg_end = it.seg_begin + it.seg_count;
    auto hkey = [&](uint32_t e, uint32_t tag) { return (((tag & ~kMidWide) >> 7) << kb) | (e >> 1); };
    // a hub pivot's group (alone in it): keys below T as in k_pv_direct
    const uint32_t hubT = (it.flags & kItemHubPairs) ? static_cast<uint32_t>(sc.T) : 0u;
    for (uint32_t k0 = it.seg_begin + member; k0 < seg_end; k0 += kTeam * kWave) {
      const uint32_t k1 = k0 + kTeam * kWave < seg_end ? k0 + kTeam * kWave : seg_end;
      RunEnds re;
      walk_regs<4>(load_seg_pv<true, kEdge>(sc.small_segs, sc.small_seg_mid, sc.small_seg_edge, k0, k1, re, kTeam), sc.other_adj, mk,
                   a.long_len, hash_tally([&](uint32_t e, uint32_t tag) {
                     const uint32_t key = hkey(e, tag);
                     const uint32_t inc = ((e ^ tag) & 1u) ? 0x10000u : 1u;
                     uint32_t h = mix32(key) & mask;
                     const uint32_t st = probe_step(key, mask);
                     for (uint32_t probe = 0;; ++probe) {
                       if (probe > mask) {  // full table: cannot happen at load <= 1/2
                         atomicOr(a.err, kErrHashFull);
                         break;
                       }
                       // one compare-and-swap per probe (claims an empty slot)
                       const uint32_t c = atomicCAS(&K[h], kEmpty, key);
                       if (c == kEmpty || c == key) {
                         atomicAdd(&V[h], inc);
                         break;
                       }
                       h = (h + st) & mask;
                     }
                   }));
    }
    team_sync();
    for (uint32_t k0 = it.seg_begin + member; k0 < seg_end; k0 += kTeam * kWave) {
      const uint32_t k1 = k0 + kTeam * kWave < seg_end ? k0 + kTeam * kWave : seg_end;
      RunEnds re;
      const SegReg sr = load_seg_pv<true, kEdge>(sc.small_segs, sc.small_seg_mid, sc.small_seg_edge, k0, k1, re, kTeam);
      if (hubT == 0) {
        // a plain group has at most kSmallGroupWork wedges: a run's credits
        // stay below 2^18, so one packed LDS word per run
        auto c = credit<kEdge, true>(
            [&](uint32_t e, uint32_t tag, uint32_t& p, uint32_t& n) {
              const uint32_t key = hkey(e, tag);
              uint32_t h = mix32(key) & mask;
              const uint32_t st = probe_step(key, mask);
              for (uint32_t probe = 0; probe <= mask; ++probe) {
                if (K[h] == key) {
                  const uint32_t v = V[h];
                  p = v & 0xffffu;
                  n = v >> 16;
                  return true;
                }
                h = (h + st) & mask;
              }
              atomicOr(a.err, kErrHashFull);  // a tallied key must be there
              return false;
            },
            cb[wave], static_cast<unsigned long long*>(nullptr), sc, re);
        walk_regs<4, kEdge>(sr, sc.other_adj, mk, a.long_len, c);
        c.flush();
        flush_mid_credits_packed<kEdge>(cb[wave], re, sc);
        continue;
      }
      auto c = credit<kEdge>(
          [&](uint32_t e, uint32_t tag, uint32_t& p, uint32_t& n) {
            if ((e >> 1) < hubT) {
              hub_counts(sc, static_cast<uint32_t>(it.owner), e >> 1, p, n);
              return true;
            }
            const uint32_t key = hkey(e, tag);
            uint32_t h = mix32(key) & mask;
            const uint32_t st = probe_step(key, mask);
            for (uint32_t probe = 0; probe <= mask; ++probe) {
              if (K[h] == key) {
                const uint32_t v = V[h];
                p = v & 0xffffu;
                n = v >> 16;
                return true;
              }
              h = (h + st) & mask;
            }
            atomicOr(a.err, kErrHashFull);  // a tallied key must be there
            return false;
          },
          cb[wave], cu[wave], sc, re);
      walk_regs<4, kEdge>(sr, sc.other_adj, mk, a.long_len, c);
      c.flush();
      flush_mid_credits<kEdge>(cb[wave], cu[wave], re, sc);
    }
    if (kTeam > 1) __syncthreads();
    const uint32_t kmask = (1u << kb) - 1u;
    for (uint32_t h = member * kWave + lane; h < size; h += kTeam * kWave) {
      const uint32_t key = K[h];
      if (key == kEmpty) continue;
      const uint32_t v = V[h];
      K[h] = kEmpty;
      V[h] = 0;
      if ((key & kmask) < hubT) continue;  // a hub pair: credited by the dense block
      PairCredit<kEdge> pc;
      pc.add(sc, key & kmask, v & 0xffffu, v >> 16, sums);
      if (pc.c | pc.x) {  // a pair with one wedge credits nothing
        const int32_t id = sc.orig[sc.small_owner[it.acc_slot + static_cast<int32_t>(key >> kb)]];
        if (pc.c) atomicAdd(&sc.bal[id], static_cast<unsigned long long>(pc.c));
        if (pc.x) atomicAdd(&sc.unb[id], static_cast<unsigned long long>(pc.x));
      }
    }
    team_sync();
  }
  __shared__ WaveSums wsum[kPVSmallWaves];
  flush_block_end(sums, graph, wsum, kPVSmallWaves, a.res);
}

// ---------------------------------------------------------------------------
// Hash items (large pivots below the window): one workgroup per item, a
// shared hash with 32-bit p and n; items with many endpoints are done in
// passes over a partition of the keys, each pass tallying, crediting and
// sweeping its keys.
constexpr int kPVHashThreads = 512;
constexpr int kPVHashWaves = kPVHashThreads / kWave;
constexpr int kPVHashSlots = 8192;

template <bool kEdge>
__global__ __launch_bounds__(kPVHashThreads) void k_pv_hash(HashArgs a) {
  a.res = own_copy(a.res, a.res_mask);
  __shared__ uint32_t keys[kPVHashSlots];
  __shared__ unsigned long long vals[kPVHashSlots];
  __shared__ __attribute__((aligned(16))) uint32_t mtab[kPVHashWaves][kGather];
  __shared__ uint32_t mflag[kPVHashWaves][kGather];
  __shared__ unsigned long long cb[kPVHashWaves][kWave], cu[kPVHashWaves][kWave];
  __shared__ int32_t item_sh;
  __shared__ uint32_t work_sh;
  const int tid = threadIdx.x;
  const int wave = tid / kWave;
  const int lane = lane_id();
  for (int i = tid; i < kPVHashSlots; i += kPVHashThreads) {
    keys[i] = kEmpty;
    vals[i] = 0;
  }
  for (int i = tid; i < kPVHashWaves * static_cast<int>(kGather); i += kPVHashThreads) (&mflag[0][0])[i] = 0;
  cb[wave][lane] = 0;
  cu[wave][lane] = 0;
  const Marks<uint32_t> mk{mtab[wave], mflag[wave]};
  Sums sums;
  uint32_t graph = kNoGraph;
  for (;;) {
    if (tid == 0) {
      item_sh = static_cast<int32_t>(atomicAdd(a.queue, 1u));
      work_sh = 0;
    }
    __syncthreads();
    const int32_t i = item_sh;
    if (i >= a.n_items) break;
    const Item it = load_const(a.items, i);
    if (it.graph != graph) {
      if (graph != kNoGraph) flush_sums(sums, a.res + static_cast<size_t>(graph) * kResStride);
      sums = Sums{};
      graph = it.graph;
    }
    const DevSideConst sc = load_const(a.sides, 2 * it.graph + it.side);
    const uint32_t seg_end = it.seg_begin + it.seg_count;
    uint32_t w = 0;
    for (uint32_t k = it.seg_begin + tid; k < seg_end; k += kPVHashThreads) w += as_global(&sc.segs[k].len_g)[0] >> 1;
    atomicAdd(&work_sh, w);
    __syncthreads();
    const uint32_t passes = (work_sh + kPVHashSlots / 4 - 1) / (kPVHashSlots / 4);
    PairCredit<kEdge> pc;
    for (uint32_t pass = 0; pass < passes; ++pass) {
      auto mine = [&](uint32_t key, uint32_t& hk) {
        hk = mix32(key);
        return passes == 1 || (hk >> 16) % passes == pass;
      };
      for (uint32_t k0 = it.seg_begin + wave * kWave; k0 < seg_end; k0 += kPVHashThreads) {
        const uint32_t k1 = k0 + kWave < seg_end ? k0 + kWave : seg_end;
        RunEnds re;
        walk_regs<4>(load_seg_pv<false, kEdge>(sc.segs, sc.seg_mid, sc.seg_edge, k0, k1, re), sc.other_adj, mk, a.long_len,
                     hash_tally([&](uint32_t e, uint32_t tag) {
                       const uint32_t key = e >> 1;
                       uint32_t hk;
                       if (!mine(key, hk)) return;
                       const unsigned long long inc = ((e ^ tag) & 1u) ? (1ull << 32) : 1ull;
                       uint32_t h = hk & (kPVHashSlots - 1);
                       const uint32_t st = probe_step(key, kPVHashSlots - 1);
                       for (uint32_t probe = 0;; ++probe) {
                         if (probe >= static_cast<uint32_t>(kPVHashSlots)) {
                           atomicOr(a.err, kErrHashFull);
                           break;
                         }
                         // one compare-and-swap per probe (claims an empty slot)
                         const uint32_t c = atomicCAS(&keys[h], kEmpty, key);
                         if (c == kEmpty || c == key) {
                           atomicAdd(&vals[h], inc);
                           break;
                         }
                         h = (h + st) & (kPVHashSlots - 1);
                       }
                     }));
      }
      __syncthreads();
      for (uint32_t k0 = it.seg_begin + wave * kWave; k0 < seg_end; k0 += kPVHashThreads) {
        const uint32_t k1 = k0 + kWave < seg_end ? k0 + kWave : seg_end;
        RunEnds re;
        const SegReg sr = load_seg_pv<false, kEdge>(sc.segs, sc.seg_mid, sc.seg_edge, k0, k1, re);
        auto c = credit<kEdge>(
            [&](uint32_t e, uint32_t, uint32_t& p, uint32_t& n) {
              const uint32_t key = e >> 1;
              uint32_t hk;
              if (!mine(key, hk)) return false;
              uint32_t h = hk & (kPVHashSlots - 1);
              const uint32_t st = probe_step(key, kPVHashSlots - 1);
              for (int probe = 0; probe < kPVHashSlots; ++probe) {
                if (keys[h] == key) {
                  const unsigned long long v = vals[h];
                  p = static_cast<uint32_t>(v);
                  n = static_cast<uint32_t>(v >> 32);
                  return true;
                }
                h = (h + st) & (kPVHashSlots - 1);
              }
              atomicOr(a.err, kErrHashFull);
              return false;
            },
            cb[wave], cu[wave], sc, re);
        walk_regs<4, kEdge>(sr, sc.other_adj, mk, a.long_len, c);
        c.flush();
        flush_mid_credits<kEdge>(cb[wave], cu[wave], re, sc);
      }
      __syncthreads();
      for (int h = tid; h < kPVHashSlots; h += kPVHashThreads) {
        const uint32_t key = keys[h];
        if (key == kEmpty) continue;
        const unsigned long long v = vals[h];
        keys[h] = kEmpty;
        vals[h] = 0;
        pc.add(sc, key, static_cast<uint32_t>(v), static_cast<uint32_t>(v >> 32), sums);
      }
      __syncthreads();
    }
    pc.to_owner(sc, it.owner);
  }
  __shared__ WaveSums wsum[kPVHashWaves];
  flush_block_end(sums, graph, wsum, kPVHashWaves, a.res);
}

// ---------------------------------------------------------------------------
// Per-edge outputs in input-record order: each edge's credits from both
// CSRs (as a run's first edge on one side and as a walked entry on the
// other) added together.  One thread per U-CSR position, grid-stride.
__global__ __launch_bounds__(256) void k_edge_combine(EdgeCombineArgs a) {
  // edges that can hold two-word credits: U-CSR positions below kcut (rows
  // of U ranks below the first narrow one) or V ends ranked below vcut
  int64_t kcut = 0;
  uint32_t vcut = 0;
  if (a.wide) {
    if (a.wide_all) {
      kcut = a.m;
    } else {
      kcut = as_global(a.off_u)[first_narrow_rank(a.off_u, a.n_u, a.max_deg_v)];
      vcut = static_cast<uint32_t>(first_narrow_rank(a.off_v, a.n_v, a.max_deg_u));
    }
  }
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t k = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; k < a.m; k += stride) {
    const uint32_t r = as_global(a.rec)[k];
    const uint32_t q = as_global(a.pos_v)[k];
    const unsigned long long p0 = as_global(a.e_pack[0])[k], p1 = as_global(a.e_pack[1])[q];
    unsigned long long b = (p0 & 0xffffffffull) + (p1 & 0xffffffffull);
    unsigned long long u = (p0 >> 32) + (p1 >> 32);
    // the two-word words of other edges are zero: not read (the V side's
    // are at random positions, a cache line each)
    if (k < kcut || (as_global(a.adj_u)[k] >> 1) < vcut) {
      b += as_global(a.e_wb[0])[k] + as_global(a.e_wb[1])[q];
      u += as_global(a.e_wu[0])[k] + as_global(a.e_wu[1])[q];
    }
    as_global(a.out_bal)[r] = static_cast<long long>(b);
    as_global(a.out_unb)[r] = static_cast<long long>(u);
  }
}

}  // namespace dev

namespace {

template <bool kEdge>
hipError_t direct_(const DirectArgs& a, int grid, hipStream_t st) {
  if (a.n_items == 0) return hipSuccess;
  hipLaunchKernelGGL(dev::k_pv_direct<kEdge>, dim3(grid), dim3(dev::kPVDirectThreads), 0, st, a);
  return hipGetLastError();
}

template <bool kEdge>
hipError_t reverse_(const SmallArgs& a, int grid, hipStream_t st) {
  if (a.n_items == 0) return hipSuccess;
  const int64_t per = dev::kPVReverseBlockItems;
  const int64_t need = (static_cast<int64_t>(a.n_items) + per - 1) / per;
  if (grid < need) grid = static_cast<int>(need);
  hipLaunchKernelGGL(dev::k_pv_reverse<kEdge>, dim3(grid), dim3(dev::kPVReverseThreads), 0, st, a);
  return hipGetLastError();
}

template <bool kEdge>
hipError_t small_(const SmallArgs& a, int cus, hipStream_t st) {
  if (a.n_items == 0) return hipSuccess;
  if (small_team(a.n_items, cus) > 1)
    hipLaunchKernelGGL((dev::k_pv_small<kEdge, dev::kPVSmallWaves>), dim3(a.n_items), dim3(dev::kPVSmallThreads), 0, st,
                       a);
  else
    hipLaunchKernelGGL((dev::k_pv_small<kEdge, 1>), dim3(std::min(3 * cus, (a.n_items + 3) / 4)),
                       dim3(dev::kPVSmallThreads), 0, st, a);
  return hipGetLastError();
}

template <bool kEdge>
hipError_t hash_(const HashArgs& a, int grid, hipStream_t st) {
  if (a.n_items == 0) return hipSuccess;
  hipLaunchKernelGGL(dev::k_pv_hash<kEdge>, dim3(grid), dim3(dev::kPVHashThreads), 0, st, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_pv_heavy_tally(const DirectArgs& a, int grid, hipStream_t st) {
  if (a.n_items == 0) return hipSuccess;
  hipLaunchKernelGGL(dev::k_pv_heavy_tally, dim3(grid), dim3(dev::kPVDirectThreads), 0, st, a);
  return hipGetLastError();
}
hipError_t launch_pv_direct(const DirectArgs& a, int grid, hipStream_t st) { return direct_<false>(a, grid, st); }
hipError_t launch_pv_reverse(const SmallArgs& a, int grid, hipStream_t st) { return reverse_<false>(a, grid, st); }
hipError_t launch_pv_small(const SmallArgs& a, int cus, hipStream_t st) { return small_<false>(a, cus, st); }
hipError_t launch_pv_hash(const HashArgs& a, int grid, hipStream_t st) { return hash_<false>(a, grid, st); }
hipError_t launch_pe_direct(const DirectArgs& a, int grid, hipStream_t st) { return direct_<true>(a, grid, st); }
hipError_t launch_pe_reverse(const SmallArgs& a, int grid, hipStream_t st) { return reverse_<true>(a, grid, st); }
hipError_t launch_pe_small(const SmallArgs& a, int cus, hipStream_t st) { return small_<true>(a, cus, st); }
hipError_t launch_pe_hash(const HashArgs& a, int grid, hipStream_t st) { return hash_<true>(a, grid, st); }

hipError_t launch_pv_key_flush(const DevSideConst* sides, int32_t n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(dev::k_pv_key_flush, dim3((n + 255) / 256, 2), dim3(256), 0, st, sides, n);
  return hipGetLastError();
}

hipError_t launch_vertex_out(const VertexOutArgs& a, hipStream_t st) {
  const int32_t n = std::max({a.n[0], a.n[1], a.words});
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(dev::k_vertex_out, dim3(std::min((n + 255) / 256, 4096)), dim3(256), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_edge_combine(const EdgeCombineArgs& a, int grid, hipStream_t st) {
  if (a.m == 0) return hipSuccess;
  hipLaunchKernelGGL(dev::k_edge_combine, dim3(grid), dim3(256), 0, st, a);
  return hipGetLastError();
}

}  // namespace dbbc
