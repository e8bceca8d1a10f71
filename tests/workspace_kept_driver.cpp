// Checks which calls WorkspaceCache (csrc/workspace_cache.hpp) turns away
// rather than allocate for them alone; prints "ok", or the failed check.
#include <cstdio>
#include <cstdlib>
#include <map>

#include "../paper_1506_01446_amd/csrc/workspace_cache.hpp"

struct Fake {
  std::map<void*, size_t> live;
  size_t next = 1;
  int allocs = 0;
  void* alloc(int, void*, size_t bytes) {
    ++allocs;
    void* p = reinterpret_cast<void*>(next++ << 12);
    live[p] = bytes;
    return p;
  }
  bool free(int, void*, void* p) {
    if (live.erase(p) != 1) std::exit(2);
    return true;
  }
};
using Cache = bitonic::WorkspaceCache<Fake>;

#define CHECK(c)                                  \
  do {                                            \
    if (!(c)) {                                   \
      std::printf("line %d: %s\n", __LINE__, #c); \
      return 1;                                   \
    }                                             \
  } while (0)

static void* st(size_t i) { return reinterpret_cast<void*>(i << 8); }

int main() {
  const size_t MB = size_t(1) << 20;
  Cache c;
  // a stream's own buffer is had, allocated once
  void* a = c.acquire(0, st(1), MB, true, true);
  CHECK(a && c.allocator().allocs == 1);
  // lent to another thread meanwhile: none for this one
  CHECK(c.acquire(0, st(1), MB, true, true) == nullptr);
  CHECK(c.acquire(0, st(1), MB, true, false) != nullptr);
  c.release(0, st(1), a, MB);
  CHECK(c.acquire(0, st(1), MB, true, true) == a);
  c.release(0, st(1), a, MB);
  // a handle of many streams, a buffer above what is kept
  const int before = c.allocator().allocs;
  CHECK(c.acquire(0, st(2), MB, false, true) == nullptr);
  CHECK(c.acquire(0, st(3), Cache::kKeepBytes + 1, true, true) == nullptr);
  // more streams than buffers are kept for
  for (size_t i = 10; i < 10 + Cache::kKeepSlots; ++i) {
    void* p = c.acquire(0, st(i), MB, true, true);
    if (p) c.release(0, st(i), p, MB);
    CHECK((p != nullptr) == (i < 9 + Cache::kKeepSlots));
  }
  CHECK(c.allocator().allocs == before + (int)Cache::kKeepSlots - 1);
  std::printf("ok\n");
  return 0;
}
