// Device ingestion of an edge list in text form: the one-GPU counterpart of
// the paper's Phase 1 (parallel loading, every range aligned to whole edge
// records) and Phase 2 (vertex identifiers made contiguous), ending in the
// device graph build.
//   1. line starts are counted per chunk of text; after a scan of the counts
//      each block takes a chunk into LDS and parses its lines, one thread a
//      line (the record alignment of Phase 1 at the finest grain): two
//      sequential reads of the text;
//   2. each line is parsed into (u, v, sign) or marked blank / comment /
//      malformed; records keep their line order (duplicates: the last one
//      wins in the build, as in the paper's datasets);
//   3. per side, the raw ids are radix-sorted with their record index; a
//      run of equal ids is one vertex, numbered by its place among the
//      distinct ids (increasing raw id), which is the compact identifier of
//      Phase 2; the distinct raw ids are kept as the compact -> raw map.
// Measured on 2.2M records (54 MB, ids of up to 11 digits), before the graph
// build: 8.3 ms with a flag and a selected position per byte (line counts
// added to one word by every wavefront 3.2 ms, the selection 1.3) -> 0.8 ms
// (the two reads of the text 0.12, the sorts 0.35).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <string>

#include "build_dev.h"
#include "kernels.h"
#include "radix.h"
#include "scan.h"

namespace dbbc {
namespace {

constexpr int kThreads = 256;

// The text in chunks of kChunk bytes, from the last 16-byte boundary at or
// before its first byte: byte p of the text is at place p + lead, so that
// whole 16-byte pieces are loaded (pieces that lie partly outside the text
// byte by byte).
constexpr int kPer = 32;  // bytes per thread
constexpr int kChunk = kThreads * kPer;
constexpr int kTail = 256;  // bytes past a chunk that its block holds too

struct Text {
  const char* base;  // 16-byte aligned
  uint32_t lead;     // places before the text
  uint32_t end;      // places of the text's end
  __device__ __forceinline__ uint4 piece(uint32_t q) const {
    if (q >= lead && static_cast<uint64_t>(q) + 16 <= end) return *reinterpret_cast<const uint4*>(base + q);
    uint4 r;
    uint32_t* w = reinterpret_cast<uint32_t*>(&r);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      w[k] = 0;
      for (int j = 0; j < 4; ++j) {
        const uint32_t p = q + 4 * k + j;
        if (p >= lead && p < end) w[k] |= static_cast<uint32_t>(static_cast<uint8_t>(base[p])) << (8 * j);
      }
    }
    return r;
  }
};

// Bit 7 of every byte of w that is a newline.
__device__ __forceinline__ uint32_t newlines(uint32_t w) {
  const uint32_t y = w ^ 0x0a0a0a0au;
  return ~(((y & 0x7f7f7f7fu) + 0x7f7f7f7fu) | y | 0x7f7f7f7fu);
}

// The line starts a thread's 32 bytes give: one after every newline that is
// not the text's last byte, and the text's first byte.  f(place) for each.
template <class F>
__device__ __forceinline__ void line_starts(const Text& t, uint32_t q, const uint4 (&v)[2], F&& f) {
  if (t.lead >= q && t.lead < q + kPer && t.lead < t.end) f(t.lead);
  const uint32_t w[8] = {v[0].x, v[0].y, v[0].z, v[0].w, v[1].x, v[1].y, v[1].z, v[1].w};
#pragma unroll
  for (int k = 0; k < 8; ++k)
    for (uint32_t b = newlines(w[k]); b; b &= b - 1) {
      const uint32_t p = q + 4 * k + (__builtin_ctz(b) >> 3) + 1;
      if (p < t.end) f(p);
    }
}

__global__ __launch_bounds__(kThreads) void k_count_lines(Text t, uint32_t* counts) {
  __shared__ uint32_t sh[kThreads / 64];
  const uint32_t q = blockIdx.x * kChunk + threadIdx.x * kPer;
  const uint4 v[2] = {t.piece(q), t.piece(q + 16)};
  uint32_t c = 0;
  line_starts(t, q, v, [&](uint32_t) { ++c; });
  uint32_t all;
  block_excl<kThreads>(c, sh, all);
  if (threadIdx.x == 0) counts[blockIdx.x] = all;
}

// Line kinds.
enum : uint8_t { kRecord = 0, kSkip = 1, kBad = 2 };

__device__ __forceinline__ bool is_space(char c) { return c == ' ' || c == '\t' || c == ',' || c == '\r'; }

// What parsing finds besides the records: the first malformed line, the
// records, and each side's largest raw id.
enum : int { kFirstBad = 0, kRecords = 1, kMaxU = 2, kMaxV = 3 };

struct Lines {
  uint64_t* u;
  uint64_t* v;
  int8_t* s;
  uint8_t* kind;
};

// One line, read through get(place) up to `limit`: its kind, and the fields of
// a record.  short_of is set when the line's bytes ran out at the limit.
struct Record {
  uint64_t u = 0, v = 0;
  bool neg = false;
};
template <class Get>
__device__ __forceinline__ uint8_t parse_line(Get get, uint32_t p, uint32_t limit, Record& r, bool& short_of) {
  // the character at p, '\n' at the end
  char c;
  auto read = [&]() {
    short_of = short_of || p >= limit;
    c = p < limit ? get(p) : '\n';
  };
  auto next = [&]() {
    ++p;
    read();
  };
  auto skip_space = [&]() {
    while (is_space(c)) next();
  };
  auto digit = [&]() { return c >= '0' && c <= '9'; };
  auto number = [&](uint64_t& x) {
    if (!digit()) return false;
    x = 0;
    do {
      if (x > (~0ull >> 1) / 10) return false;  // beyond 2^63
      x = x * 10 + static_cast<uint64_t>(c - '0');
      next();
    } while (digit());
    return (x >> 63) == 0 && (c == '\n' || is_space(c));
  };
  read();
  skip_space();
  if (c == '\n' || c == '#' || c == '%') return kSkip;
  if (!number(r.u)) return kBad;
  skip_space();
  if (!number(r.v)) return kBad;
  skip_space();
  const bool minus = c == '-';
  if (minus || c == '+') next();
  uint64_t sv = 0;
  if (!number(sv) || (minus ? sv != 1 : sv > 1)) return kBad;
  r.neg = minus || sv == 0;
  return kRecord;
}

// Every line "u v s" with u, v decimal ids below 2^63 and s one of 1, +1
// (positive), 0, -1 (negative); fields separated by spaces, tabs or commas;
// fields after the third are ignored.  Blank lines and lines whose first
// non-space character is '#' or '%' are skipped.  A block's chunk (and the
// kTail bytes after it) is parsed out of LDS; a line that needs more than
// that is read again from the text.  Each block leaves its records and
// largest ids in part (atomics of thousands of blocks to three words would
// take longer than the parsing).
struct Part {
  unsigned long long records, max_u, max_v;
};
__device__ __forceinline__ void join(Part& a, const Part& b) {
  a.records += b.records;
  a.max_u = max(a.max_u, b.max_u);
  a.max_v = max(a.max_v, b.max_v);
}
// The block's parts joined (in thread 0).
template <int kT>
__device__ __forceinline__ Part join_block(Part x) {
  __shared__ Part sh[kT / 64];
#pragma unroll
  for (int d = 32; d > 0; d >>= 1)
    join(x, Part{__shfl_xor(x.records, d, 64), __shfl_xor(x.max_u, d, 64), __shfl_xor(x.max_v, d, 64)});
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = x;
  __syncthreads();
  if (threadIdx.x == 0)
    for (int w = 1; w < kT / 64; ++w) join(x, sh[w]);
  return x;
}

__global__ __launch_bounds__(kThreads) void k_parse(Text t, const uint32_t* first, Lines out, Part* part,
                                                    unsigned long long* words) {
  __shared__ __attribute__((aligned(16))) char buf[kChunk + kTail];
  __shared__ uint16_t at[kChunk + 1];  // a chunk of newlines, and the text's first byte
  __shared__ uint32_t sh[kThreads / 64];
  const int tid = static_cast<int>(threadIdx.x);
  const uint32_t c0 = blockIdx.x * kChunk, q0 = c0 + tid * kPer;
  const uint4 v[2] = {t.piece(q0), t.piece(q0 + 16)};
  *reinterpret_cast<uint4*>(buf + tid * kPer) = v[0];
  *reinterpret_cast<uint4*>(buf + tid * kPer + 16) = v[1];
  if (tid < kTail / 16) *reinterpret_cast<uint4*>(buf + kChunk + 16 * tid) = t.piece(c0 + kChunk + 16 * tid);
  uint32_t c = 0;
  line_starts(t, q0, v, [&](uint32_t) { ++c; });
  uint32_t lines;
  uint32_t k = block_excl<kThreads>(c, sh, lines);
  line_starts(t, q0, v, [&](uint32_t p) { at[k++] = static_cast<uint16_t>(p - c0); });
  __syncthreads();
  const uint32_t end = t.end - c0, held = min(static_cast<uint32_t>(kChunk + kTail), end);
  const uint64_t l0 = first[blockIdx.x];
  Part mine{0, 0, 0};
  for (uint32_t i = tid; i < lines; i += kThreads) {
    Record r;
    bool short_of = false;
    uint8_t kind = parse_line([&](uint32_t p) { return buf[p]; }, at[i], held, r, short_of);
    if (short_of && held < end) {
      const char* rest = t.base + c0;
      kind = parse_line([&](uint32_t p) { return rest[p]; }, at[i], end, r, short_of);
    }
    const uint64_t l = l0 + i;
    if (kind == kRecord) {
      out.u[l] = r.u;
      out.v[l] = r.v;
      out.s[l] = r.neg ? int8_t(-1) : int8_t(1);
      join(mine, Part{1, r.u, r.v});
    }
    out.kind[l] = kind;
    if (kind == kBad) atomicMin(&words[kFirstBad], static_cast<unsigned long long>(l));
  }
  mine = join_block<kThreads>(mine);
  if (tid == 0) part[blockIdx.x] = mine;
}

__global__ __launch_bounds__(1024) void k_join_parts(const Part* part, uint32_t n, unsigned long long* words) {
  Part x{0, 0, 0};
  for (uint32_t i = threadIdx.x; i < n; i += 1024) join(x, part[i]);
  x = join_block<1024>(x);
  if (threadIdx.x == 0) {
    words[kRecords] = x.records;
    words[kMaxU] = x.max_u;
    words[kMaxV] = x.max_v;
  }
}

// The records alone, in line order (where some line is none).  A block takes
// kRecChunk lines; pass 0 counts, pass 1 moves.
constexpr uint32_t kRecChunk = 8 * kThreads;

template <int kPass>
__global__ __launch_bounds__(kThreads) void k_records(Lines in, uint32_t lines, uint32_t* counts, Lines out) {
  __shared__ uint32_t sh[kThreads / 64];
  uint32_t done = kPass ? counts[blockIdx.x] : 0u;
  for (uint32_t j = 0; j < kRecChunk; j += kThreads) {
    const uint64_t l = static_cast<uint64_t>(blockIdx.x) * kRecChunk + j + threadIdx.x;
    const bool rec = l < lines && in.kind[l] == kRecord;
    uint32_t all;
    const uint32_t k = done + block_excl<kThreads>(rec ? 1u : 0u, sh, all);
    if (kPass && rec) {
      out.u[k] = in.u[l];
      out.v[k] = in.v[l];
      out.s[k] = in.s[l];
    }
    done += all;
  }
  if (!kPass && threadIdx.x == 0) counts[blockIdx.x] = done;
}

// A side's raw ids as a sort's input: key, then record index.
struct RawIn {
  const uint64_t* raw;
  __device__ __forceinline__ radix::Elt<3> load(uint32_t i) const {
    const uint64_t k = raw[i];
    return {{static_cast<uint32_t>(k), static_cast<uint32_t>(k >> 32), i}};
  }
};

// Numbering of a side's sorted raw ids.  A block takes kIdChunk records;
// pass 0 counts the heads of runs of equal ids, pass 1 (after a scan) gives
// record idx its run's number and writes each run's raw id to the map.
constexpr uint32_t kIdChunk = 8 * kThreads;

template <int kPass>
__global__ __launch_bounds__(kThreads) void k_ids(radix::Soa<3> a, uint32_t m, uint32_t* counts, int32_t* id,
                                                  int64_t* raw_of) {
  __shared__ uint32_t sh[kThreads / 64];
  uint32_t done = kPass ? counts[blockIdx.x] : 0u;
  for (uint32_t j = 0; j < kIdChunk; j += kThreads) {
    const uint64_t i64 = static_cast<uint64_t>(blockIdx.x) * kIdChunk + j + threadIdx.x;
    const uint32_t i = static_cast<uint32_t>(i64);
    const bool in = i64 < m;
    const bool head = in && (i == 0 || a.p[0][i] != a.p[0][i - 1] || a.p[1][i] != a.p[1][i - 1]);
    uint32_t all;
    const uint32_t before = block_excl<kThreads>(head ? 1u : 0u, sh, all);
    if (kPass && in) {
      const uint32_t c = done + before + (head ? 1u : 0u) - 1u;
      id[a.p[2][i]] = static_cast<int32_t>(c);
      if (head) raw_of[c] = static_cast<int64_t>((static_cast<uint64_t>(a.p[1][i]) << 32) | a.p[0][i]);
    }
    done += all;
  }
  if (!kPass && threadIdx.x == 0) counts[blockIdx.x] = done;
}

// Device memory of one step, freed on scope exit (at least 16 bytes, so
// that even an empty array has an address).
struct Tmp : DevBuf {
  hipError_t alloc(size_t bytes) { return DevBuf::alloc(std::max<size_t>(bytes, 16)); }
};

struct Fail {
  int status;
  std::string msg;
};

#define DEV_TRY(expr)                                                                   \
  do {                                                                                  \
    hipError_t e_ = (expr);                                                             \
    if (e_ != hipSuccess)                                                               \
      throw Fail{e_ == hipErrorOutOfMemory ? DBBC_E_OOM : DBBC_E_DEVICE,                \
                 std::string(#expr) + ": " + hipGetErrorString(e_)};                    \
  } while (0)

#define LAUNCH(kernel, grid, ...)                                                  \
  do {                                                                             \
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(kThreads), 0, st, __VA_ARGS__);    \
    DEV_TRY(hipGetLastError());                                                    \
  } while (0)

void read_words(unsigned long long* h, const unsigned long long* d, int n, hipStream_t st) {
  DEV_TRY(hipMemcpyAsync(h, d, n * sizeof(*h), hipMemcpyDeviceToHost, st));
  DEV_TRY(hipStreamSynchronize(st));
}

int bits_for_max(uint64_t mx) {
  int b = 1;
  while (b < 64 && (mx >> b) != 0) ++b;
  return b;
}

Lines carve_lines(Carve& c, size_t n) {
  Lines l;
  l.u = reinterpret_cast<uint64_t*>(c.take(2 * n));
  l.v = reinterpret_cast<uint64_t*>(c.take(2 * n));
  l.s = reinterpret_cast<int8_t*>(c.take((n + 3) / 4));
  l.kind = reinterpret_cast<uint8_t*>(c.take((n + 3) / 4));
  return l;
}

void ingest(const char* text_in, int64_t len, uint32_t flags, hipStream_t st, HostGraph& g, DeviceCsr& csr,
            IngestOut& out) {
  Tmp dtext;
  const char* text = text_in;
  if (!(flags & DBBC_INPUT_DEVICE)) {
    DEV_TRY(dtext.alloc(static_cast<size_t>(len)));
    if (len) DEV_TRY(hipMemcpyAsync(dtext.p, text_in, static_cast<size_t>(len), hipMemcpyHostToDevice, st));
    text = dtext.as<char>();
  }
  const uint32_t lead = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(text) & 15u);
  const Text t{text - lead, lead, lead + static_cast<uint32_t>(len)};
  const uint32_t chunks = static_cast<uint32_t>((static_cast<uint64_t>(t.end) + kChunk - 1) / kChunk);
  Tmp words_b, counts_b, parts_b;  // the parse's words, then the number of lines and of each side's ids
  DEV_TRY(words_b.alloc(7 * 8));
  DEV_TRY(counts_b.alloc(static_cast<size_t>(chunks) * 4));
  DEV_TRY(parts_b.alloc(static_cast<size_t>(chunks) * sizeof(Part)));
  unsigned long long* words = words_b.as<unsigned long long>();
  uint32_t* counts = counts_b.as<uint32_t>();
  DEV_TRY(launch_fill_u64(words, 1, ~0ull, st));
  DEV_TRY(launch_fill_u64(words + 1, 6, 0ull, st));
  unsigned long long h[4] = {~0ull, 0, 0, 0}, n_lines = 0;
  if (len) {
    LAUNCH(k_count_lines, chunks, t, counts);
    DEV_TRY(scan_counts(counts, chunks, words + 4, st));
    read_words(&n_lines, words + 4, 1, st);
  }
  Tmp line_b, rec_b;
  Lines lines{}, recs{};
  {
    Carve c;
    carve_lines(c, n_lines);
    DEV_TRY(line_b.alloc(c.used * 4));
    c = Carve{line_b.as<uint32_t>(), 0};
    lines = carve_lines(c, n_lines);
  }
  if (n_lines) {
    LAUNCH(k_parse, chunks, t, counts, lines, parts_b.as<Part>(), words);
    hipLaunchKernelGGL(k_join_parts, dim3(1), dim3(1024), 0, st, parts_b.as<Part>(), chunks, words);
    DEV_TRY(hipGetLastError());
    read_words(h, words, 4, st);
  }
  if (h[kFirstBad] != ~0ull)
    throw Fail{DBBC_E_PARSE, "line " + std::to_string(h[kFirstBad] + 1) +
                                 ": expected \"u v s\" with ids below 2^63 and s in {1, 0, -1, +1}"};
  const int64_t m = static_cast<int64_t>(h[kRecords]);
  if (m >= (int64_t(1) << 31) - 1) throw Fail{DBBC_E_TOO_LARGE, "more than 2^31 - 2 edge records"};
  out.lines = static_cast<int64_t>(n_lines);
  out.records = m;
  if (m == 0) throw Fail{DBBC_E_INVALID_ARG, "the text holds no edge record"};
  const size_t M = static_cast<size_t>(m);
  const uint32_t m32 = static_cast<uint32_t>(m);
  recs = lines;
  if (n_lines != h[kRecords]) {  // some lines are no records
    const uint32_t blocks = static_cast<uint32_t>((n_lines + kRecChunk - 1) / kRecChunk);
    Carve c;
    carve_lines(c, M);
    c.take(blocks);
    DEV_TRY(rec_b.alloc(c.used * 4));
    c = Carve{rec_b.as<uint32_t>(), 0};
    recs = carve_lines(c, M);
    uint32_t* rc = c.take(blocks);
    LAUNCH(k_records<0>, blocks, lines, static_cast<uint32_t>(n_lines), rc, recs);
    DEV_TRY(scan_counts(rc, blocks, nullptr, st));
    LAUNCH(k_records<1>, blocks, lines, static_cast<uint32_t>(n_lines), rc, recs);
    (void)line_b.alloc(0);  // (given back in stream order, as below)
  }
  // compact ids: each side's raw ids sorted, the distinct ones counted, and
  // then numbered
  const uint64_t* raw[2] = {recs.u, recs.v};
  const radix::Digits dig[2] = {radix::digits_of(0, bits_for_max(h[kMaxU])),
                                radix::digits_of(0, bits_for_max(h[kMaxV]))};
  const uint32_t blocks = static_cast<uint32_t>((M + kIdChunk - 1) / kIdChunk);
  Tmp work, ids;
  uint32_t *arr[9], *idc[2];
  unsigned long long* ctl = nullptr;
  Carve c;
  for (int sizing = 1; sizing >= 0; --sizing) {
    if (!sizing) {
      DEV_TRY(work.alloc(c.used * 4));
      c = Carve{work.as<uint32_t>(), 0};
    }
    // six sort arrays, and three that keep side 0's sorted ids
    for (uint32_t*& a : arr) a = c.take(M);
    for (uint32_t*& a : idc) a = c.take(blocks);
    ctl = reinterpret_cast<unsigned long long*>(
        c.take(2 * std::max(radix::control_words(m, dig[0]), radix::control_words(m, dig[1]))));
  }
  DEV_TRY(ids.alloc(2 * Carve::round(M) * 4));
  int32_t* id[2] = {ids.as<int32_t>(), ids.as<int32_t>() + Carve::round(M)};
  const radix::Soa<3> buf[3] = {
      {{arr[0], arr[1], arr[2]}}, {{arr[3], arr[4], arr[5]}}, {{arr[6], arr[7], arr[8]}}};
  // a sort's result goes to the buffer its last pass does not read
  radix::Soa<3> sorted[2];
  const radix::Control cc{ctl};
  int rest = 2;  // the buffer that takes no part
  for (int s = 0; s < 2; ++s) {
    const radix::Soa<3> two[2] = {buf[(rest + 1) % 3], buf[(rest + 2) % 3]};
    const int at = (dig[s].passes - 1) & 1;
    sorted[s] = two[at];
    DEV_TRY(launch_fill_u64(ctl, radix::control_words(m, dig[s]), 0ull, st));
    DEV_TRY((radix::histogram<2>(RawIn{raw[s]}, m, dig[s], cc, st)));
    DEV_TRY((radix::passes<2, 3>(RawIn{raw[s]}, sorted[s], two, m, dig[s], cc, st)));
    LAUNCH(k_ids<0>, blocks, sorted[s], m32, idc[s], id[s], nullptr);
    DEV_TRY(scan_counts(idc[s], blocks, words + 5 + s, st));
    rest = (rest + 1 + at) % 3;  // keep this side's result
  }
  unsigned long long n[2];
  read_words(n, words + 5, 2, st);
  if (n[0] + n[1] >= (1ull << 30)) throw Fail{DBBC_E_TOO_LARGE, "n_u + n_v must be below 2^30"};
  for (int s = 0; s < 2; ++s) {
    DEV_TRY(out.raw[s].alloc(std::max<size_t>(static_cast<size_t>(n[s]) * 8, 16)));
    out.raw[s].bytes = static_cast<size_t>(n[s]) * 8;
    LAUNCH(k_ids<1>, blocks, sorted[s], m32, idc[s], id[s], out.raw[s].as<int64_t>());
  }
  (void)work.alloc(0);  // the sorts' memory goes before the build takes its own
  std::string err;
  const int rc = build_device_graph(static_cast<int32_t>(n[0]), static_cast<int32_t>(n[1]), m, id[0], id[1], recs.s,
                                    (flags & ~DBBC_INPUT_DEVICE) | DBBC_INPUT_DEVICE, st, g, csr, err);
  if (rc != DBBC_OK) throw Fail{rc, err};
}

}  // namespace

int ingest_text(const char* text, int64_t len, uint32_t flags, hipStream_t st, HostGraph& g, DeviceCsr& csr,
                IngestOut& out, std::string& err) {
  if (len < 0 || (len > 0 && !text)) {
    err = "text must not be NULL and len must be non-negative";
    return DBBC_E_INVALID_ARG;
  }
  if (len >= (int64_t(1) << 31) - 1) {
    err = "text longer than 2^31 - 2 bytes";
    return DBBC_E_TOO_LARGE;
  }
  auto drop_maps = [&]() {
    (void)hipStreamSynchronize(st);
    for (int s = 0; s < 2; ++s) out.raw[s].release();
  };
  try {
    ingest(text, len, flags, st, g, csr, out);
  } catch (const Fail& f) {
    err = f.msg;
    drop_maps();
    return f.status;
  } catch (const std::bad_alloc&) {
    err = "host allocation failed while reading the text";
    drop_maps();
    return DBBC_E_OOM;
  }
  return DBBC_OK;
}

}  // namespace dbbc
