// Kernel templates of the rank sort (rank.hpp), over a storage type ST
// (column_pass.hpp): Keys32, Keys64 or Pairs.
//
// At these sizes the chip is nearly empty and a sort takes as long as its
// chain of dependent launches, steps and loads.  The network on 2^16 keys is
// a tile sort and four phases of merges; a search of every other tile for
// every element does the merges' work in one launch whose longest chain is
// seven reads of LDS and six of memory, at a cost in reads (elements x tiles)
// that the idle chip has.  Whole sorts on MI355X in us, network against rank:
//   4-byte keys  5000  12.5, 7.6    2^14  15.9, 8.9     20000  28.5, 9.2
//                2^15  22.5, 10.3   50000 35.0, 14.9    2^16   28.1, 16.1
//   8-byte keys  2^12  16.5, 11.0   2^13  24.0, 11.6    2^14   31.7, 13.9
//                2^15  40.3, 17.0   50000 53.0, 25.1    2^16   52.2, 26.4
//   pairs        2^13  23.5, 12.2   2^15  39.4, 17.8    2^16   51.1, 28.0
#pragma once

#include "column_pass.hpp"
#include "rank.hpp"

namespace bitonic {

// Sorts every 2^L-element tile of src into dst, mapped into the sorting
// domain, one tile per workgroup, in few-tile programs (kind 6: lanes on
// consecutive elements, so any alignment).  Bound by its steps' latency.
template <int L, int RL, class ST, class CD>
__global__ __launch_bounds__(1 << (L - RL)) void rank_tile_kernel(ST src, ST dst, uint32_t n,
                                                                  CD cd) {
  using PR = Prog<L, RL, 6>;
  using E = typename ST::E;
  constexpr int LAST = PR::value.ngroups - 1;
  __shared__ E lds[PR::LDSW];
  const uint32_t t0 = (uint32_t)blockIdx.x << L;
  const uint32_t valid = n - t0 < (uint32_t)PR::T ? n - t0 : (uint32_t)PR::T;
  const ST in = src.at(t0), out = dst.at(t0);
  uint32_t tid = threadIdx.x;
  E x[PR::R];
  {
    const uint32_t base = deposit<free_mask(PR::value.g[0], L)>(tid);
    load_checked(x, valid, [&](auto J) { return slot_index<PR, 0, J>(base); },
                 [&](uint32_t i) { return in.get(i); }, cd, ST::kPadE);
  }
  run_from<PR, 0>(x, lds, tid);
  asm volatile("" : "+v"(tid));  // the bases are computed anew: fewer registers
  {
    const uint32_t base = deposit<free_mask(PR::value.g[LAST], L)>(tid);
    static_for<0, PR::R>([&](auto J) {
      const uint32_t i = slot_index<PR, LAST, J>(base);
      if (i < valid) out.put(i, x[J]);
    });
  }
}

// A merging workgroup: kRankElems consecutive elements (of one tile) times
// kRankGroups groups of threads that share the other tiles.  The lanes of a
// wave search for neighbours in value, so their reads fall into the same few
// lines.  One group a workgroup of 256 elements took 40 us for 2^16 8-byte
// keys (one wave per SIMD waiting for its reads), four 28.7, eight 26.9,
// sixteen 28.7 (more workgroups load the samples).
constexpr uint32_t kRankThreads = 1024;
constexpr uint32_t kRankGroups = 8;
constexpr uint32_t kRankElems = kRankThreads / kRankGroups;

// Elements per sample.  Every workgroup keeps the first element of each 64 in
// LDS, which leaves a search log2(64) dependent loads of memory.  32 or 16
// save one or two of them and lose as much to loading the samples.
constexpr uint32_t kRankStep = 64;

// Every element of the sorted 2^L-element tiles of src to its rank in dst,
// mapped back.  Elements that tie rank by their tiles' order, so ranks are
// distinct.  At most kRankGroups * K tiles; K searches in flight per thread.
template <int L, int K, class ST, class CD>
__global__ __launch_bounds__(kRankThreads) void rank_merge_kernel(ST src, ST dst, uint32_t n,
                                                                  CD cd) {
  using E = typename ST::E;
  constexpr uint32_t T = 1u << L;
  constexpr uint32_t NS = T / kRankStep;  // samples per tile
  constexpr int LS = 6;
  static_assert(1u << LS == kRankStep && T % kRankElems == 0);
  extern __shared__ __attribute__((aligned(8))) char rank_lds[];
  __shared__ uint32_t sums[kRankGroups][kRankElems];
  E* const samples = reinterpret_cast<E*>(rank_lds);
  const uint32_t tiles = (n - 1) / T + 1;
  for (uint32_t i = threadIdx.x; i < tiles * NS; i += kRankThreads)
    if (i * kRankStep < n) samples[i] = src.get(i * kRankStep);
  const uint32_t lane = threadIdx.x % kRankElems, group = threadIdx.x / kRankElems;
  const uint32_t g = blockIdx.x * kRankElems + lane;
  const uint32_t own = blockIdx.x * kRankElems / T;  // uniform
  const E x = g < n ? src.get(g) : ST::kPadE;
  __syncthreads();
  uint32_t at[K], end[K];
  static_for<0, K>([&](auto k) {
    const uint32_t j = group + kRankGroups * k;
    const uint32_t len = j >= tiles || j == own ? 0u : (n - j * T < T ? n - j * T : T);
    const uint32_t ns = (len + kRankStep - 1) / kRankStep;
    // c: samples of tile j that come before x (of an earlier tile, also those
    // equal to it)
    uint32_t c = 0;
    static_for<0, L - LS + 1>([&](auto b) {
      constexpr uint32_t w = NS >> b;
      const uint32_t p = c + w - 1;
      if (p < ns) {
        const E s = samples[j * NS + p];
        if (s < x || (j < own && s == x)) c += w;
      }
    });
    // the last such sample comes before x; the next one does not
    at[k] = c == 0 ? 0u : (c - 1) * kRankStep + 1;
    end[k] = c == 0 ? 0u : (c * kRankStep < len ? c * kRankStep : len);
  });
  static_for<0, LS>([&](auto b) {
    constexpr uint32_t w = kRankStep / 2 >> b;
    E s[K];
    static_for<0, K>([&](auto k) {
      const uint32_t p = at[k] + w - 1;
      s[k] = src.get(p < end[k] ? (group + kRankGroups * k) * T + p : 0u);
    });
    static_for<0, K>([&](auto k) {
      const uint32_t p = at[k] + w - 1;
      if (p < end[k] && (s[k] < x || (group + kRankGroups * k < own && s[k] == x))) at[k] += w;
    });
  });
  uint32_t before = 0;
  static_for<0, K>([&](auto k) { before += at[k]; });
  sums[group][lane] = before;
  __syncthreads();
  if (group == 0 && g < n) {
    uint32_t rank = g % T;
    static_for<0, (int)kRankGroups>([&](auto k) { rank += sums[k][lane]; });
    dst.put(rank, cd.dec(x));
  }
}

template <int L, int RL, class ST, class CD>
static void rank_launch(ST a, ST b, CD cd, uint32_t n, hipStream_t st) {
  const uint32_t tiles = ((n - 1) >> L) + 1;
  const uint32_t blocks = (n - 1) / kRankElems + 1;
  const size_t lds = (size_t)tiles * ((1u << L) / kRankStep) * sizeof(typename ST::E);
  rank_tile_kernel<L, RL><<<tiles, 1 << (L - RL), 0, st>>>(a, b, n, cd);
  if constexpr (std::is_same_v<ST, Keys64> && L == 12)
    if (tiles > 2 * kRankGroups) {
      rank_merge_kernel<L, 4><<<blocks, kRankThreads, lds, st>>>(b, a, n, cd);
      return;
    }
  rank_merge_kernel<L, 2><<<blocks, kRankThreads, lds, st>>>(b, a, n, cd);
}

template <class ST, class CD>
static void rank_run(ST a, ST b, CD cd, uint32_t n, hipStream_t st) {
  constexpr bool wide = sizeof(typename ST::E) == 8;
  switch (rank_tile_log2(n, (int)sizeof(typename ST::E))) {
    case 9:
      if constexpr (wide) rank_launch<9, 3>(a, b, cd, n, st);
      break;
    case 10: rank_launch<10, 3>(a, b, cd, n, st); break;
    case 11: rank_launch<11, 3>(a, b, cd, n, st); break;
    case 12: rank_launch<12, 3>(a, b, cd, n, st); break;
    case 13:
      if constexpr (!wide) rank_launch<13, 4>(a, b, cd, n, st);
      break;
    default: break;
  }
}

}  // namespace bitonic
