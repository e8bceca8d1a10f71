// Checks that WorkspaceCache (csrc/workspace_cache.hpp) gives the buffers of
// streams that are used no more to new ones, and never one whose work may not
// be done; prints "ok", or the failed check.
#include <cstdio>
#include <cstdlib>
#include <map>

#include "../paper_1506_01446_amd/csrc/workspace_cache.hpp"

struct Fake {
  std::map<void*, size_t> live;
  size_t next = 1;
  int allocs = 0, stamps = 0;
  uint32_t sent[32] = {}, arrived[32] = {};
  bool hold = false;  // the streams' work is not done yet
  void* freed_on = nullptr;
  void* alloc(int, void*, size_t bytes) {
    ++allocs;
    void* p = reinterpret_cast<void*>(next++ << 12);
    live[p] = bytes;
    return p;
  }
  bool free(int, void* stream, void* p) {
    if (live.erase(p) != 1) std::exit(2);
    freed_on = stream;
    return true;
  }
  bool stamp(int, void*, int slot, uint32_t value) {
    ++stamps;
    sent[slot] = value;
    if (!hold) arrived[slot] = value;
    return true;
  }
  uint32_t stamped(int slot) { return arrived[slot]; }
  size_t bytes() const {
    size_t b = 0;
    for (auto& l : live) b += l.second;
    return b;
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
static bool use(Cache& c, int dev, size_t i, size_t bytes) {
  void* p = c.acquire(dev, st(i), bytes, true, true);
  if (p) c.release(dev, st(i), p, bytes);
  return p != nullptr;
}

int main() {
  const size_t MB = size_t(1) << 20;
  {  // few streams are never stamped
    Cache c;
    for (int r = 0; r < 3; ++r)
      for (size_t i = 1; i <= Cache::kQuietSlots; ++i) CHECK(use(c, 0, i, MB));
    CHECK(c.allocator().stamps == 0 && c.allocator().allocs == (int)Cache::kQuietSlots);
  }
  {  // streams that come and go: every one gets a kept buffer
    Cache c;
    for (size_t i = 1; i <= 1000; ++i) {
      const int before = c.allocator().allocs;
      CHECK(use(c, 0, i, MB));
      CHECK(use(c, 0, i, MB) && c.allocator().allocs == before + 1);
      CHECK(c.kept_slots() <= Cache::kKeepSlots && c.allocator().bytes() == c.kept_bytes());
    }
    CHECK(c.allocator().freed_on == st(1000));  // on a stream that is there
    // the longest unused went: the last ones are still kept
    const int before = c.allocator().allocs;
    for (size_t i = 1000; i > 1000 - 15; --i) CHECK(use(c, 0, i, MB));
    CHECK(c.allocator().allocs == before);
  }
  {  // one whose last work has not been seen done stays, and another device's
    Cache c;
    for (size_t i = 1; i <= Cache::kKeepSlots; ++i) {
      c.allocator().hold = i > 20;
      CHECK(use(c, i == 18 ? 1 : 0, i, MB));
    }
    // 1 .. 16 unstamped, 17, 19, 20 done, 18 on device 1, 21 .. pending
    CHECK(use(c, 0, 101, MB) && use(c, 0, 102, MB) && use(c, 0, 103, MB));
    CHECK(!use(c, 0, 104, MB));
    for (size_t i = 1; i <= 16; ++i) {
      const int before = c.allocator().allocs;
      CHECK(use(c, 0, i, MB) && c.allocator().allocs == before);
    }
    for (int s = 0; s < 32; ++s) c.allocator().arrived[s] = c.allocator().sent[s];
    CHECK(use(c, 0, 104, MB));
    // a lent one stays
    Cache l;
    void* held[Cache::kKeepSlots];
    for (size_t i = 0; i < Cache::kKeepSlots; ++i) CHECK((held[i] = l.acquire(0, st(i + 1), MB)));
    CHECK(!use(l, 0, 200, MB));
    for (size_t i = 0; i < Cache::kKeepSlots; ++i) l.release(0, st(i + 1), held[i], MB);
    CHECK(use(l, 0, 200, MB));
    CHECK(l.allocator().bytes() == l.kept_bytes());
  }
  {  // room in bytes: large buffers of idle streams go for new ones
    Cache c;
    for (size_t i = 1; i <= 40; ++i) {
      CHECK(use(c, 0, i, Cache::kKeepBytes));
      CHECK(c.kept_bytes() <= Cache::kKeepTotal && c.allocator().bytes() == c.kept_bytes());
    }
    // and for a kept one that grows
    CHECK(use(c, 0, 41, MB) && use(c, 0, 41, Cache::kKeepBytes));
    CHECK(c.kept_bytes() <= Cache::kKeepTotal && c.allocator().bytes() == c.kept_bytes());
  }
  {  // all given back but what is lent, or whose device cannot be waited for
    Cache c;
    for (size_t i = 1; i <= 5; ++i) CHECK(use(c, i == 3 ? 1 : 0, i, i * MB));
    void* p = c.acquire(0, st(9), MB);
    int waits = 0;
    auto after = [&](Fake&) { return true; };
    CHECK(!c.give_back_all([&](int dev) { return ++waits, dev == 0; }, after));
    CHECK(waits == 5 && c.kept_slots() == 2 && c.kept_bytes() == 5 * MB);
    CHECK(c.allocator().bytes() == c.kept_bytes() && c.allocator().freed_on == nullptr);
    CHECK(c.give_back_all([&](int) { return true; }, after) && c.kept_slots() == 1);
    c.release(0, st(9), p, MB);
    CHECK(c.give_back_all([&](int) { return true; }, after));
    CHECK(c.kept_bytes() == 0 && c.allocator().live.empty());
    CHECK(use(c, 0, 9, MB) && c.kept_bytes() == MB);
  }
  std::printf("ok\n");
  return 0;
}
