// Which of a segmented sort's segments go by their digits (segradix.hpp) and
// which by the network (no HIP in here: host and device share it, and it is
// tested on the CPU).
//
// The host sees a bound on the segments, not their lengths, so it enqueues the
// network's launches for segments below seg_radix_min_class together with the
// digit sort's, and the prep kernel says who takes which segment; launches
// that find none of theirs take 2.0 to 2.5 us each.
#pragma once

#include <stdint.h>

namespace bitonic {

constexpr int kSegSmallMaxLog2 = 13;  // segments of up to 2^13 keys are "small"

// The least class (log2 of the padded length) of segments that go by digits.
// Sorts of segments of one class on MI355X in us, network against digits:
//                    class 16       17           18          20
//   int32  4 segments  62, 84     83, 85     108, 87     217, 112
//         32 segments  74, 114   120, 126    180, 149    704, 331
//        256 segments 187, 252   425, 378
//   int64  4 segments 112, 125   130, 137    180, 150    342, 233
//         32 segments 140, 192   207, 225    376, 318    -
//   pairs 32 segments 150, 200   216, 232    359, 318    -
constexpr int seg_radix_min_class(bool wide) { return wide ? 18 : 17; }

// The least class of the bound for which digit launches are enqueued.  They
// replace the network's launches from their least class up to the bound: from
// here on finding nothing in them takes no longer (4-byte keys 6 launches for
// 6 or more; 8-byte elements 10 for 8 or more, which take 23 and 24 us), so a
// bound far above the segments costs nothing.
constexpr int seg_radix_min_bound(bool wide) { return wide ? 20 : 19; }

// The most elements (by what is known of them, not by what the segments hold)
// that a segmented sort takes a digit workspace for: 1 GiB of 4-byte keys.
constexpr int64_t kSegRadixMaxElems = int64_t(1) << 28;

// Segments from class 14 up to that go by digits too if others do anyway and their
// padded lengths are not above this in all: a few more tiles in launches that
// run anyway, where the network's launches for them are a chain of their own.
// Per million elements the network takes 7 us in class 14 to 14 in class 17
// (4-byte keys; 8-byte elements 13 to 31), the digits 13 (31).
constexpr uint64_t kSegRadixMaxMedium = uint64_t(1) << 21;

// A bound on the elements of all segments, which the digit workspace is laid
// out for.  total: the caller's, 0 if not given; in_allocation: the elements
// to the end of the keys' allocation by the runtime's records, asked for only
// where the bound on the length is taken from them too (max_seg_len == 0): a
// record may cover a part of the keys' memory, and says nothing of a table in
// a larger buffer.
template <class F>
constexpr int64_t seg_elems(int64_t nseg, int64_t max_seg_len, int64_t total, F in_allocation) {
  if (max_seg_len == 0) return total ? total : (int64_t)in_allocation();
  const int64_t by_length = max_seg_len > INT64_MAX / nseg ? INT64_MAX : max_seg_len * nseg;
  return total && total < by_length ? total : by_length;
}

// Whether the digit launches are enqueued: by the caller's bound on the
// segment length and a bound on the elements of all segments.
constexpr bool seg_digit_launches(int64_t max_seg_len, int64_t elems, bool wide) {
  const int64_t longest = max_seg_len < elems ? max_seg_len : elems;
  return longest > int64_t(1) << (seg_radix_min_bound(wide) - 1) && elems <= kSegRadixMaxElems;
}

// The least class that goes by digits, given the number of segments of each
// class; 32 if none does.
constexpr int seg_digit_class(const uint32_t* segments_of, bool wide) {
  const int least = seg_radix_min_class(wide);
  uint32_t longer = 0;
  uint64_t medium = 0;
  for (int c = kSegSmallMaxLog2 + 1; c < 32; ++c) {
    if (c < least) medium += (uint64_t)segments_of[c] << c;
    else longer |= segments_of[c];
  }
  if (longer == 0) return 32;
  return medium <= kSegRadixMaxMedium ? kSegSmallMaxLog2 + 1 : least;
}

}  // namespace bitonic
