// Checks the routing of segmented sorts (csrc/segroute.hpp) on the host;
// prints "ok", or the failed check.
#include <cstdio>

#include "../paper_1506_01446_amd/csrc/segroute.hpp"

using namespace bitonic;

#define CHECK(c)                                            \
  do {                                                      \
    if (!(c)) {                                             \
      std::printf("line %d: %s (%d)\n", __LINE__, #c, wide); \
      return 1;                                             \
    }                                                       \
  } while (0)

static int check(bool wide) {
  const int least = seg_radix_min_class(wide), from = seg_radix_min_bound(wide);
  // the bound alone never brings the digit launches: they need elements for
  // at least one long segment, and a bound as far up as they are worth it
  for (int b = 0; b <= 31; ++b)
    for (int e = 0; e <= 40; ++e)
      for (int64_t d = -1; d <= 1; ++d) {
        const int64_t bound = (int64_t(1) << b) + (b < 31 ? d : 0), elems = (int64_t(1) << e) + d;
        if (!seg_digit_launches(bound, elems, wide)) continue;
        CHECK(bound > int64_t(1) << (from - 1) && elems > int64_t(1) << (from - 1));
        CHECK(elems <= kSegRadixMaxElems);
      }
  CHECK(from > least && least > kSegSmallMaxLog2 + 1);
  CHECK(seg_digit_launches(int64_t(1) << 22, 11000000, wide));
  CHECK(!seg_digit_launches(1 << 18, int64_t(1) << 25, wide));
  {  // no long segment: none by digits, whatever the bound was
    uint32_t cnt[32] = {};
    for (int c = 0; c < least; ++c) cnt[c] = 1000;
    CHECK(seg_digit_class(cnt, wide) == 32);
    // one long one among many of the middle classes: it alone
    for (int c = least; c <= 31; ++c) {
      cnt[c] = 1;
      CHECK(seg_digit_class(cnt, wide) == least);
      cnt[c] = 0;
    }
  }
  {  // few of the middle classes go with the long ones, as many do not
    for (int c = 14; c < least; ++c) {
      uint32_t cnt[32] = {};
      cnt[13] = 100000;
      cnt[20] = 2;
      cnt[c] = (uint32_t)(kSegRadixMaxMedium >> c);
      CHECK(seg_digit_class(cnt, wide) == 14);
      cnt[c] += 1;
      CHECK(seg_digit_class(cnt, wide) == least);
      cnt[20] = 0;
      CHECK(seg_digit_class(cnt, wide) == 32);
    }
    uint32_t cnt[32] = {};
    CHECK(seg_digit_class(cnt, wide) == 32);
    cnt[16] = 0xFFFFFFFFu;  // no wrap
    cnt[18] = 1;
    CHECK(seg_digit_class(cnt, wide) == least);
  }
  {  // elements: the runtime's records are asked for without a bound only
    bool asked = false;
    auto record = [&] {
      asked = true;
      return int64_t(5000);
    };
    CHECK(seg_elems(12, int64_t(1) << 22, 0, record) == int64_t(12) << 22 && !asked);
    CHECK(seg_elems(100, int64_t(1) << 22, 11000000, record) == 11000000 && !asked);
    CHECK(seg_elems(3, 100, 11000000, record) == 300 && !asked);
    CHECK(seg_elems(int64_t(1) << 30, int64_t(1) << 31, 0, record) > kSegRadixMaxElems);
    CHECK(seg_elems((int64_t(1) << 31) - 1, int64_t(1) << 31, 9, record) == 9 && !asked);
    CHECK(seg_elems(7, 0, 123, record) == 123 && !asked);
    CHECK(seg_elems(7, 0, 0, record) == 5000 && asked);
    // a hundred requests with one of 2^22 keys, in a large arena
    CHECK(!seg_digit_launches(1 << 22, seg_elems(100, 1 << 22, 0, record), wide));
    CHECK(seg_digit_launches(1 << 22, seg_elems(100, 1 << 22, 30000000, record), wide));
  }
  return 0;
}

int main() {
  if (check(false) || check(true)) return 1;
  std::printf("ok\n");
  return 0;
}
