// Test harness: counts the heap blocks that one shared library asks operator new
// for.  Loaded with RTLD_GLOBAL before that library, so that its calls come here.
#include <dlfcn.h>
#include <link.h>

#include <cstdint>
#include <cstdlib>
#include <new>

static long g_count;
static uintptr_t g_from, g_to;  // the library's addresses

static void* take(std::size_t n, const void* caller) {
  const uintptr_t at = reinterpret_cast<uintptr_t>(caller);
  if (at >= g_from && at < g_to) ++g_count;
  return std::malloc(n ? n : 1);
}

void* operator new(std::size_t n) { return take(n, __builtin_return_address(0)); }
void* operator new[](std::size_t n) { return take(n, __builtin_return_address(0)); }
void* operator new(std::size_t n, const std::nothrow_t&) noexcept { return take(n, __builtin_return_address(0)); }
void* operator new[](std::size_t n, const std::nothrow_t&) noexcept { return take(n, __builtin_return_address(0)); }
void operator delete(void* p) noexcept { std::free(p); }
void operator delete[](void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }
void operator delete[](void* p, std::size_t) noexcept { std::free(p); }

// Count the calls of the library that holds sym from here on.
extern "C" void new_watch(const void* sym) {
  Dl_info d;
  if (!dladdr(sym, &d)) return;
  g_count = 0;
  dl_iterate_phdr(
      [](dl_phdr_info* o, std::size_t, void* base) {
        if (o->dlpi_addr != reinterpret_cast<uintptr_t>(base)) return 0;
        uintptr_t end = 0;
        for (int k = 0; k < o->dlpi_phnum; ++k)
          if (o->dlpi_phdr[k].p_type == PT_LOAD && o->dlpi_phdr[k].p_vaddr + o->dlpi_phdr[k].p_memsz > end)
            end = o->dlpi_phdr[k].p_vaddr + o->dlpi_phdr[k].p_memsz;
        g_from = o->dlpi_addr;
        g_to = o->dlpi_addr + end;
        return 1;
      },
      d.dli_fbase);
}
extern "C" long new_count(void) { return g_count; }
