// Checks the policy of WorkspaceCache (csrc/workspace_cache.hpp) with a
// counting allocator; prints "ok", or the failed check.
#include <cstdio>
#include <cstdlib>
#include <map>

#include "../paper_1506_01446_amd/csrc/workspace_cache.hpp"

struct Fake {
  std::map<void*, size_t> live;
  size_t next = 1;
  bool fail_alloc = false, fail_free = false;
  int allocs = 0;
  void* alloc(int, void*, size_t bytes) {
    if (fail_alloc) return nullptr;
    ++allocs;
    void* p = reinterpret_cast<void*>(next++ << 12);
    live[p] = bytes;
    return p;
  }
  bool free(int, void*, void* p) {
    if (fail_free) return false;
    if (live.erase(p) != 1) {
      std::printf("double free\n");
      std::exit(1);
    }
    return true;
  }
  size_t bytes() const {
    size_t b = 0;
    for (auto& l : live) b += l.second;
    return b;
  }
};
using Cache = bitonic::WorkspaceCache<Fake>;

#define CHECK(c)                                       \
  do {                                                 \
    if (!(c)) {                                        \
      std::printf("line %d: %s\n", __LINE__, #c);      \
      return 1;                                        \
    }                                                  \
  } while (0)

static void* st(size_t i) { return reinterpret_cast<void*>(i << 8); }

int main() {
  const size_t MB = size_t(1) << 20;
  {  // one buffer a stream, reused; another stream has its own
    Cache c;
    void* a = c.acquire(0, st(1), 3 * MB);
    CHECK(a && c.allocator().live[a] == 4 * MB);
    c.release(0, st(1), a, 3 * MB);
    CHECK(c.acquire(0, st(1), 4 * MB) == a);
    // lent: a second call on the stream gets another buffer, freed behind it
    void* b = c.acquire(0, st(1), MB);
    CHECK(b && b != a);
    c.release(0, st(1), b, MB);
    CHECK(c.allocator().live.count(b) == 0 && c.allocator().live.count(a) == 1);
    c.release(0, st(1), a, 4 * MB);
    void* d = c.acquire(0, st(2), MB);
    CHECK(d && d != a && c.kept_slots() == 2);
    c.release(0, st(2), d, MB);
    void* e = c.acquire(1, st(1), MB);  // the same handle on another device
    CHECK(e && e != a && c.kept_slots() == 3);
    c.release(1, st(1), e, MB);
    // a larger one replaces the stream's, which is freed
    void* f = c.acquire(0, st(1), 5 * MB);
    CHECK(f != a && c.allocator().live.count(a) == 0 && c.kept_bytes() == 10 * MB);
    c.release(0, st(1), f, 5 * MB);
    CHECK(c.allocator().bytes() == c.kept_bytes());
  }
  {  // not kept: too large, or a handle that names several streams
    Cache c;
    void* a = c.acquire(0, st(1), Cache::kKeepBytes + 1);
    CHECK(a && c.kept_bytes() == 0);
    c.release(0, st(1), a, Cache::kKeepBytes + 1);
    CHECK(c.allocator().live.empty());
    void* b = c.acquire(0, st(2), MB, false);
    CHECK(b && c.kept_slots() == 0);
    c.release(0, st(2), b, MB);
    CHECK(c.allocator().live.empty());
  }
  {  // the bounds on what is kept
    Cache c;
    for (size_t i = 1; i <= 100; ++i) {
      void* p = c.acquire(0, st(i), MB);
      CHECK(p);
      c.release(0, st(i), p, MB);
      CHECK(c.kept_slots() <= Cache::kKeepSlots && c.allocator().bytes() == c.kept_bytes());
    }
    CHECK(c.kept_slots() == Cache::kKeepSlots);
    Cache g;
    for (size_t i = 1; i <= 20; ++i) {
      void* p = g.acquire(0, st(i), Cache::kKeepBytes);
      CHECK(p);
      g.release(0, st(i), p, Cache::kKeepBytes);
      CHECK(g.kept_bytes() <= Cache::kKeepTotal && g.allocator().bytes() == g.kept_bytes());
    }
    CHECK(g.kept_bytes() == Cache::kKeepTotal);
    // a stream whose calls stay small gives its buffer back
    const size_t before = g.kept_bytes();
    for (int i = 0; i < Cache::kShrinkCalls; ++i) g.release(0, st(1), g.acquire(0, st(1), MB), MB);
    CHECK(g.kept_bytes() == before - Cache::kKeepBytes + MB);
    CHECK(g.allocator().bytes() == g.kept_bytes());
  }
  {  // failures: no memory; a free that is refused for now
    Cache c;
    c.allocator().fail_alloc = true;
    CHECK(c.acquire(0, st(1), MB) == nullptr);
    c.allocator().fail_alloc = false;
    void* a = c.acquire(0, st(1), 2 * MB);
    c.release(0, st(1), a, 2 * MB);
    c.allocator().fail_alloc = true;
    CHECK(c.acquire(0, st(1), 3 * MB) == nullptr);  // the old buffer stays
    CHECK(c.acquire(0, st(1), 2 * MB) == a);
    c.release(0, st(1), a, 2 * MB);
    c.allocator().fail_alloc = false;
    c.allocator().fail_free = true;
    void* b = c.acquire(0, st(1), 8 * MB);
    CHECK(b != a && c.parked() == 1);
    c.release(0, st(1), b, 8 * MB);
    CHECK(c.acquire(0, st(2), MB) != a);  // not another stream's
    CHECK(c.acquire(0, st(1), MB) == a);  // its own stream may use it
    CHECK(c.acquire(0, st(1), MB) == b);  // while it is lent, the kept one
    c.release(0, st(1), b, MB);
    c.release(0, st(1), a, MB);
    c.allocator().fail_free = false;
    CHECK(c.acquire(0, st(1), 4 * MB) == b && c.parked() == 0);
    CHECK(c.allocator().live.count(a) == 0);
  }
  std::printf("ok\n");
  return 0;
}
