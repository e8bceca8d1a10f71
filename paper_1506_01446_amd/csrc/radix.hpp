// Sort of a long single array by its digits (internal interface): least
// significant digit first, eight bits a pass, out of place between the array
// and a workspace of its size (radix_kernels.hpp).  The plain sorts take it
// above the sizes that go by rank (rank_pays); explicit plans always run the
// network.  The method is published: radix sorts whose passes chain their
// prefix sums through device memory (Merrill and Garland 2016, "Single-pass
// Parallel Prefix Scan with Decoupled Look-back"; Adinets and Merrill 2022,
// "Onesweep"), with equal digits of a wave found by ballots.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "codec.hpp"

namespace bitonic {

constexpr int kRadixBits = 8;
constexpr int kRadixBins = 1 << kRadixBits;
constexpr int kRadixMaxPasses = 8;  // 8-byte elements
constexpr uint32_t kRadixHistBlocks = 512;  // most workgroups of the counting kernel
constexpr int kRadixThreads = 1024;
// A count of elements shares a 32-bit word with a flag bit.
constexpr int64_t kRadixMaxN = (int64_t(1) << 31) - 1;

// Device words of one sort, written by its counting and scan kernels.
struct RadixMeta {
  uint32_t ticket[kRadixMaxPasses];  // next tile of each pass
  // 1: the pass would leave the elements as they are (one digit value
  // throughout, or a value digit of pairs whose values come in order)
  uint32_t trivial[kRadixMaxPasses];
};

// The elements of one sort: 4-byte keys (keys, cd), pairs (keys and values,
// cd64) or 8-byte keys (keys64, cd64).
struct RadixData {
  int32_t* keys;
  int32_t* values;
  int64_t* keys64;
  Codec cd;
  Codec64 cd64;
};

// Elements per thread of a pass's tile (kRadixThreads threads).  The largest
// tile reads and writes the longest runs and looks back over the fewest
// tiles; an array that it would cut into fewer tiles than half the compute
// units takes a smaller one.
constexpr int radix_items(int64_t n, int elem_bytes) {
  // 4-byte: 2^14, 2^13, 2^12 keys a tile; 8-byte: 2^13, 2^12, 2^11
  const int most = elem_bytes == 4 ? 16 : 8;
  if (n >= (int64_t(128) * most * kRadixThreads) * (elem_bytes == 4 ? 2 : 1)) return most;
  if (n >= int64_t(128) * (most / 2) * kRadixThreads) return most / 2;
  return most / 4;
}

// Tiles per group and groups per supergroup of a pass's prefix sums, and the
// most rows of kRadixBins words that they take for `arrays` arrays of
// `tiles` tiles in all: the tiles' counts, the groups' sums, the
// supergroups' sums, and the counts ahead of each supergroup.
constexpr uint32_t kRadixGroupLog = 4;
constexpr uint32_t kRadixGroup = 1u << kRadixGroupLog;
__host__ __device__ constexpr uint32_t radix_state_rows(uint32_t tiles, uint32_t arrays) {
  return tiles + (tiles >> kRadixGroupLog) + arrays +
         2 * ((tiles >> (2 * kRadixGroupLog)) + arrays);
}

// Layout of the workspace.
struct RadixSpace {
  RadixMeta* meta;
  uint32_t* base;       // passes x 256: elements of smaller digits
  uint32_t* partial;    // blocks x passes x 256: the workgroups' counts
  uint32_t* unordered;  // blocks: pairs, 1 if values of the block decrease
  uint32_t* state[2];   // radix_state_rows x 256, one for each of two passes
  char* alt;            // n elements: where every other pass writes
};

constexpr uint32_t radix_tiles(uint32_t n, int elem_bytes) {
  const uint32_t tile = (uint32_t)(radix_items(n, elem_bytes) * kRadixThreads);
  return n / tile + (n % tile != 0);
}
// Counting workgroups, of 1024 threads: one per compute unit, as the scan
// reads a row of counts of each (whole sorts, with 512 of 512 threads before:
// 2^22 int32 97.7 -> 93.4 us, 2^24 int64 626 -> 614, 2^24 argsort 380 -> 370);
// two per compute unit from 2^25 elements on, where the count itself is long
// (2^26 argsort 1417 -> 1347 us, with one 1412).
constexpr uint32_t radix_hist_blocks(uint32_t n) {
  const uint32_t b = n / 4096 + (n % 4096 != 0);
  const uint32_t most = n >= (1u << 25) ? kRadixHistBlocks : kRadixHistBlocks / 2;
  return b < most ? b : most;
}

// Workspace bytes of a sort of n elements of `elem_bytes` (4; 8-byte keys
// and pairs 8); with s, also its layout at p (256-byte aligned).
inline size_t radix_space(char* p, uint32_t n, int elem_bytes, RadixSpace* s) {
  auto up = [](size_t b) { return (b + 255) & ~size_t(255); };
  const size_t row = kRadixBins * sizeof(uint32_t);
  const size_t passes = (size_t)elem_bytes;
  const size_t blocks = radix_hist_blocks(n);
  const size_t states = radix_state_rows(radix_tiles(n, elem_bytes), 1) * row;
  size_t at = 0;
  auto take = [&](size_t bytes) {
    char* const q = p + at;
    at += up(bytes);
    return q;
  };
  RadixSpace r;
  r.meta = reinterpret_cast<RadixMeta*>(take(sizeof(RadixMeta)));
  r.base = reinterpret_cast<uint32_t*>(take(passes * row));
  r.partial = reinterpret_cast<uint32_t*>(take(blocks * passes * row));
  r.unordered = reinterpret_cast<uint32_t*>(take(blocks * sizeof(uint32_t)));
  r.state[0] = reinterpret_cast<uint32_t*>(take(states));
  r.state[1] = reinterpret_cast<uint32_t*>(take(states));
  r.alt = take((size_t)n * (size_t)elem_bytes);
  if (s) *s = r;
  return at;
}

// Enqueue the sort of n elements, 1 <= n <= kRadixMaxN, on st: one launch
// that counts, one that scans the counts, one per digit.  workspace:
// radix_space(...) bytes of device memory, their contents arbitrary.
void launch_radix_sort(const RadixData& d, uint32_t n, void* workspace, hipStream_t st);

// Per storage type (kernels_radix32.hip, kernels_radix64.hip,
// kernels_radixpairs.hip).
void radix_run_keys32(const RadixData& d, uint32_t n, const RadixSpace& s, hipStream_t st);
void radix_run_keys64(const RadixData& d, uint32_t n, const RadixSpace& s, hipStream_t st);
void radix_run_pairs(const RadixData& d, uint32_t n, const RadixSpace& s, hipStream_t st);

// The scan kernel (kernels_radix32.hip), shared by the storages.
void launch_radix_scan(const RadixSpace& s, uint32_t n, int passes, bool pairs, hipStream_t st);

}  // namespace bitonic
