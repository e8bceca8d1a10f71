// Big segments of a segmented sort by their digits (internal interface): the
// passes of the digit sort (radix.hpp) with every segment an array of its
// own.  See segradix_kernels.hpp.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "radix.hpp"
#include "segmented.hpp"

namespace bitonic {

// A tile of a big segment.
struct alignas(32) SegRadixTile {
  int64_t off;     // the segment's first element
  uint32_t len;    // the segment's elements
  uint32_t seg;    // its place among the big segments
  uint32_t first;  // its first tile
  uint32_t tile;   // this tile, in the segment
};

struct SegRadixSpace {
  RadixMeta* meta;      // trivial[0]: pairs, 1 if the values of some segment decrease
  uint32_t* base;       // big segments x passes x 256
  uint32_t* trivial;    // big segments x passes
  uint32_t* partial;    // blocks x 2 x passes x 256
  uint32_t* unordered;  // blocks x 2
  uint32_t* span;       // blocks: the segment that goes on past the block
  SegRadixTile* tiles;
  uint32_t* state[2];
  char* alt;            // element i of the keys at i - offsets[0]
  int64_t elems;        // what it was laid out for
  int64_t nseg;
  uint32_t max_tiles, max_segs;
};

// Bounds for segments of `elems` elements in all (host side): big segments
// have more than 2^kSegSmallMaxLog2 elements, and tiles of 2^tile_log
// (kSegTileLog32, kSegTileLog64) hold at least that many but the last.
constexpr int64_t segradix_max_segs(int64_t elems, int64_t nseg) {
  const int64_t most = elems >> kSegSmallMaxLog2;
  return most < nseg ? most : nseg;
}
constexpr int64_t segradix_max_tiles(int64_t elems, int64_t nseg, int tile_log) {
  return (elems >> tile_log) + segradix_max_segs(elems, nseg);
}

// Workspace bytes for segments of `elems` elements of elem_bytes (4 or 8) in
// all; with s, also the layout at p.
inline size_t segradix_space(char* p, int64_t elems, int64_t nseg, int elem_bytes,
                             SegRadixSpace* s) {
  const size_t passes = (size_t)elem_bytes;
  const size_t row = kRadixBins * sizeof(uint32_t);
  const size_t segs = (size_t)segradix_max_segs(elems, nseg);
  const size_t tiles =
      (size_t)segradix_max_tiles(elems, nseg, elem_bytes == 4 ? kSegTileLog32 : kSegTileLog64);
  const size_t states = radix_state_rows((uint32_t)tiles, (uint32_t)segs) * row;
  size_t at = 0;
  auto take = [&](size_t bytes) {
    char* const q = p + at;
    at += (bytes + 255) & ~size_t(255);
    return q;
  };
  SegRadixSpace r;
  r.meta = reinterpret_cast<RadixMeta*>(take(sizeof(RadixMeta)));
  r.base = reinterpret_cast<uint32_t*>(take(segs * passes * row));
  r.trivial = reinterpret_cast<uint32_t*>(take(segs * passes * sizeof(uint32_t)));
  r.partial = reinterpret_cast<uint32_t*>(take((size_t)kRadixHistBlocks * 2 * passes * row));
  r.unordered = reinterpret_cast<uint32_t*>(take(kRadixHistBlocks * 2 * sizeof(uint32_t)));
  r.span = reinterpret_cast<uint32_t*>(take(kRadixHistBlocks * sizeof(uint32_t)));
  r.tiles = reinterpret_cast<SegRadixTile*>(take(tiles * sizeof(SegRadixTile)));
  r.state[0] = reinterpret_cast<uint32_t*>(take(states));
  r.state[1] = reinterpret_cast<uint32_t*>(take(states));
  r.alt = take((size_t)elems * (size_t)elem_bytes);
  r.elems = elems;
  r.nseg = nseg;
  r.max_tiles = (uint32_t)tiles;
  r.max_segs = (uint32_t)segs;
  if (s) *s = r;
  return at;
}

// Enqueue the sort of every big segment of the prepared table (sc, after
// launch_seg_prep) behind it: a counting launch, one that scans, one per
// digit.
void launch_segradix(const SegData& d, const int64_t* offsets, const SegScratch& sc,
                     const SegRadixSpace& s, int cus, hipStream_t st);

// Per storage type (kernels_segradix32.hip and so on).
void segradix_run_keys32(const SegData& d, const int64_t* offsets, const SegScratch& sc,
                         const SegRadixSpace& s, int cus, hipStream_t st);
void segradix_run_keys64(const SegData& d, const int64_t* offsets, const SegScratch& sc,
                         const SegRadixSpace& s, int cus, hipStream_t st);
void segradix_run_pairs(const SegData& d, const int64_t* offsets, const SegScratch& sc,
                        const SegRadixSpace& s, int cus, hipStream_t st);

}  // namespace bitonic
