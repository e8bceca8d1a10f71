// WorkspaceCache (csrc/workspace_cache.hpp) runs under C entries: with no
// memory left for the host it neither allocates nor throws.  Prints "ok", or
// the failed check.
#include <cstdio>
#include <cstdlib>
#include <new>

static bool g_out_of_memory = false;

void* operator new(size_t n) {
  void* p = g_out_of_memory ? nullptr : std::malloc(n);
  if (!p) throw std::bad_alloc();
  return p;
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

#include "../paper_1506_01446_amd/csrc/workspace_cache.hpp"

struct Fake {
  size_t next = 1;
  bool fail_free = false;
  void* alloc(int, void*, size_t) { return reinterpret_cast<void*>(next++ << 12); }
  bool free(int, void*, void*) { return !fail_free; }
};
using Cache = bitonic::WorkspaceCache<Fake>;

int main() {
  const size_t MB = size_t(1) << 20;
  static Cache c;
  g_out_of_memory = true;
  try {
    for (size_t i = 1; i <= 100; ++i) {
      void* const stream = reinterpret_cast<void*>(i << 8);
      c.allocator().fail_free = i % 2 == 0;
      for (size_t mb : {1, 8, 300, 2})
        if (void* p = c.acquire(0, stream, mb * MB)) c.release(0, stream, p, mb * MB);
    }
  } catch (const std::bad_alloc&) {
    g_out_of_memory = false;
    std::printf("threw\n");
    return 1;
  }
  g_out_of_memory = false;
  if (c.kept_slots() > Cache::kKeepSlots || c.kept_bytes() > Cache::kKeepTotal) {
    std::printf("kept too much\n");
    return 1;
  }
  std::printf("ok\n");
  return 0;
}
