// Sort of a single array of up to 32 tiles in two launches (internal
// interface): the tiles are sorted into a workspace by the tile programs, and
// every element then goes to its rank, its place in its own tile plus the
// number of elements of each other tile that come before it
// (rank_kernels.hpp).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "radix.hpp"

namespace bitonic {

// log2 of the tile for n elements of elem_bytes (4 or 8): the least that makes
// at most 16 tiles, within the sizes that pay.  A larger tile takes the first
// launch longer (2^10, 2^11, 2^12 8-byte elements 8, 10, 16 us), more tiles
// the second one, whose searches are elements times tiles.  Whole sorts on
// MI355X in us, by tile, before load_checked took 1.5 to 2 us off each (2^13
// 4-byte keys at 16 a thread, else 8):
//   4-byte keys  2^14  2^10 10.9, 2^11 10.3    2^15  13.9, 12.0, 2^12 12.9
//                2^16  2^11 20.5, 2^12 17.8    2^17  2^12 37.0, 2^13 32.7
//   8-byte keys  2^12  2^9 12.8, 2^10 13.8     2^13  14.1, 13.7
//                2^15  2^10 19.5, 2^11 18.4    2^16  26.9, 2^12 27.6
//                2^17  2^12 (32 tiles) 48.3, 2^13 58.1
constexpr int rank_tile_log2(int64_t n, int elem_bytes) {
  const int least = elem_bytes == 4 ? 10 : 9, most = elem_bytes == 4 ? 13 : 12;
  int L = least;
  while (L < most && (n - 1) >> L >= 16) ++L;
  return L;
}

// Whether n elements are sorted this way: more than one launch of the network
// sorts (4-byte keys 2^12, 8-byte elements 2^11), and fewer than the digit
// sort is faster for.  Measured in us between two events (6 us of them the
// events'), network, rank and digits:
//   4-byte keys  4097   17.6, 14.6, 37.3   2^16    34.6, 23.5, 43.9
//                70000  56.4, 29.5, 43.7   2^17    45.1, 38.4, 44.6
//   8-byte keys  2049   22.6, 17.8, 56.7   2^16    58.6, 33.4, 70.8
//                70000  93.1, 42.4, 72.2   2^17    93.5, 51.5, 76.3
//   pairs        2049   23.0, 18.1, 62.3   2^16    57.8, 35.5, 74.3
//   (digits of pairs with values in order 52.7 and 59.3)
// At 2^17 pairs 32 tiles' searches took 57.5 against 45.5 and 66.6 by digits.
constexpr bool rank_pays(int64_t n, int elem_bytes, bool pairs) {
  return n > (elem_bytes == 4 ? 1 << 12 : 1 << 11) && n <= (pairs ? 1 << 16 : 1 << 17);
}
// Whether that is so even where the workspace has to be allocated and freed
// for the call, which takes the host 17 us (on the per-thread stream, in a
// second thread on one stream, on more streams than buffers are kept for).  A
// whole call on MI355X in us, network against rank with that:
//   4-byte keys  2^13  13.8, 24.8   2^14  19.2, 25.2   2^15  25.3, 26.3
//                40000 44.3, 25.7   2^16  31.8, 24.7   2^17  39.2, 31.7
//   8-byte keys  2^12  21.7, 24.2   6000  34.9, 24.7   2^14  50.2, 24.3
constexpr bool rank_pays_allocating(int64_t n, int elem_bytes) {
  return n > (elem_bytes == 4 ? 1 << 15 : 1 << 12);
}
constexpr uint32_t kRankMaxTiles = 32;
static_assert(((1u << 17) - 1) >> rank_tile_log2(1 << 17, 8) < kRankMaxTiles &&
              ((1u << 17) - 1) >> rank_tile_log2(1 << 17, 4) < 16 &&
              ((1u << 16) - 1) >> rank_tile_log2(1 << 16, 8) < 16,
              "searches per thread of the merging kernel");

// Workspace bytes: the array's size.
constexpr size_t rank_workspace_bytes(int64_t n, int elem_bytes) {
  return (size_t)n * (size_t)elem_bytes;
}

// Enqueue the sort of d's n elements on st; rank_pays(n).
void launch_rank_sort(const RadixData& d, uint32_t n, void* workspace, hipStream_t st);

// Per storage type (kernels_rank32.hip and so on).
void rank_run_keys32(const RadixData& d, uint32_t n, void* workspace, hipStream_t st);
void rank_run_keys64(const RadixData& d, uint32_t n, void* workspace, hipStream_t st);
void rank_run_pairs(const RadixData& d, uint32_t n, void* workspace, hipStream_t st);

}  // namespace bitonic
