// Test harness: a sort of (key, index) whose tiles publish 64-bit words, as sorts
// of 2^30 elements and more do, on any number of elements.
#include "../../paper_2609_21848_amd/csrc/radix.h"

using namespace dbbc;

namespace {
struct KeyIn {
  const uint32_t* key;
  __device__ __forceinline__ radix::Elt<2> load(uint32_t i) const { return {{key[i], i}}; }
};
__global__ void k_clear(unsigned long long* p, size_t n) {
  for (size_t i = blockIdx.x * static_cast<size_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<size_t>(gridDim.x) * blockDim.x)
    p[i] = 0;
}
template <class In, class Out>
hipError_t wide_pass(In in, Out out, int64_t n, const radix::Digits& d, int p, const radix::Control& c,
                     hipStream_t st) {
  if (n < radix::kSmallN)
    return radix::pass_as<1, 2, unsigned long long, radix::kThreadsS, radix::kItemsS>(in, out, n, d, p, c, st);
  return radix::pass_as<1, 2, unsigned long long, radix::kThreadsL, radix::kItemsL>(in, out, n, d, p, c, st);
}
}  // namespace

// Sorts the n keys (device memory, their low `bits` bits, stable) into out_key
// and out_index.  Returns a hipError_t.
extern "C" int radix_wide_sort(const uint32_t* key, int64_t n, int bits, uint32_t* out_key, uint32_t* out_index) {
  const radix::Digits d = radix::digits_of(0, bits);
  const size_t words = radix::kHistWords + radix::kMaxPasses / 2 +
                       static_cast<size_t>(d.passes) * static_cast<size_t>(radix::tiles_of(n)) * radix::kDigits;
  uint32_t* buf = nullptr;
  unsigned long long* ctl = nullptr;
  hipError_t e = hipMalloc(reinterpret_cast<void**>(&buf), static_cast<size_t>(4 * n + 4) * 4);
  if (e == hipSuccess) e = hipMalloc(reinterpret_cast<void**>(&ctl), words * 8);
  const radix::Control c{ctl};
  const radix::Soa<2> b[2] = {{{buf, buf + n}}, {{buf + 2 * n, buf + 3 * n}}}, out{{out_key, out_index}};
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_clear, dim3(256), dim3(256), 0, nullptr, ctl, words);
    e = radix::histogram<1>(KeyIn{key}, n, d, c, nullptr);
  }
  for (int p = 0; p < d.passes && e == hipSuccess; ++p) {
    const radix::Soa<2>& to = p + 1 == d.passes ? out : b[p & 1];
    e = p == 0 ? wide_pass(KeyIn{key}, to, n, d, p, c, nullptr) : wide_pass(b[(p - 1) & 1], to, n, d, p, c, nullptr);
  }
  const hipError_t s = hipDeviceSynchronize();
  (void)hipFree(buf);
  (void)hipFree(ctl);
  return e != hipSuccess ? e : s;
}
