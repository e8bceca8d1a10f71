// Kernel templates of the big segments' digit sort (segradix.hpp).
//
// The tiles of all big segments are one list (the prep kernel's prefix sums);
// each segment has its own digit counts, prefix sums, left-out passes and
// count of executed passes, so its elements move between the keys and the
// workspace as a single array's would.  The number of tiles is known on the
// device only: every launch has a fixed grid whose workgroups share the list.
#pragma once

#include "radix_kernels.hpp"
#include "seg_kernels.hpp"
#include "segradix.hpp"

namespace bitonic {

// log2 of the elements per tile of a pass: the prep kernel's tiles.
template <class ST>
constexpr int segradix_items() {
  return (1 << seg_tile_log<ST>()) / kRadixThreads;
}

// The workspace was laid out for a bound on the segments' elements (seg_elems):
// the caller's word, or without a bound on their length the runtime's record of
// the keys' allocation.  Should the table hold more than that, no kernel
// touches the workspace's arrays past their ends: the segments are then sorted
// where they are (segradix_in_place).
__device__ __forceinline__ bool segradix_fits(const int64_t* offsets, const SegMeta* seg_meta,
                                              const uint64_t* big_tiles, const SegRadixSpace& s) {
  const uint32_t nbig = seg_meta->nradix;
  return nbig <= s.max_segs && big_tiles[nbig] <= s.max_tiles &&
         offsets[s.nseg] - offsets[0] <= s.elems;
}

// The flip network on one segment, step by step in global memory, by one
// workgroup: slow, and for tables that do not fit the workspace only.
template <class ST, class MAP>
__device__ void segradix_in_place(const ST& a, uint32_t len, const MAP& map) {
  for (int p = 1; p == 1 || (1ull << (p - 1)) < len; ++p)
    for (int q = p - 1; q >= 0; --q) {
      for (uint64_t c = threadIdx.x; c < (uint64_t)len; c += blockDim.x) {
        // c as the lower end of its comparator (a mirror image in the
        // phase's first step)
        const uint64_t hi = q == p - 1 ? c ^ ((2ull << q) - 1) : c ^ (1ull << q);
        if (hi > c && hi < len) {
          const auto x = map.enc(a.get((uint32_t)c)), y = map.enc(a.get((uint32_t)hi));
          if (y < x) {
            a.put((uint32_t)c, map.dec(y));
            a.put((uint32_t)hi, map.dec(x));
          }
        }
      }
      __syncthreads();
    }
}

// Threads of a counting workgroup: smaller ones than a single array's, as a
// workgroup counts one segment of its range after another, with a barrier
// around each (a batch of 12 requests of 2^8 .. 2^22 keys: 219 us, with 1024
// threads 221).
constexpr int kSegRadixHistThreads = 512;

// One row of a segment's counts as the passes take it: where each digit
// begins in the segment, and whether the pass is to be left out.  All
// kSegRadixHistThreads threads call it, `count` for the first 256.
__device__ __forceinline__ void segradix_finish(uint32_t count, uint32_t len, bool ordered_values,
                                                uint32_t* base, uint32_t* trivial,
                                                uint32_t* wave_sum, uint32_t* one_digit) {
  const uint32_t tid = threadIdx.x;
  const bool in = tid < kRadixBins;
  if (tid == 0) *one_digit = 0;
  __syncthreads();
  if (in && count == len) *one_digit = 1;
  const uint32_t before = radix_scan_bins(in ? count : 0u, in, tid >> 6, wave_sum);
  if (in) base[tid] = before;
  if (tid == 0) *trivial = *one_digit || ordered_values ? 1u : 0u;
  __syncthreads();
}

// Each workgroup counts the digits of a contiguous range of the tiles,
// segment by segment.  A segment inside one range is finished at once; of a
// segment that goes over into other ranges each leaves its counts: in row 0
// those of the segment its range begins within, in row 1 those of the one
// that begins in it and goes on (span).
template <bool FL, class ST, class CD>
__global__ __launch_bounds__(kSegRadixHistThreads) void segradix_hist_kernel(
    ST a, CD cd, const int64_t* __restrict__ offsets, const SegMeta* __restrict__ seg_meta,
    const uint32_t* __restrict__ big_ids, const uint64_t* __restrict__ big_tiles,
    SegRadixSpace s) {
  constexpr int P = radix_passes<ST>();
  constexpr uint32_t NT = kSegRadixHistThreads;
  constexpr uint32_t T = 1u << seg_tile_log<ST>();
  __shared__ RadixBinsLds<ST> lds;
  __shared__ uint32_t wave_sum[kRadixBins / 64];
  __shared__ uint32_t one_digit;
  const uint32_t tid = threadIdx.x;
  const uint32_t nbig = seg_meta->nradix;
  if (tid == 0) s.span[blockIdx.x] = ~0u;
  if (nbig == 0 || !segradix_fits(offsets, seg_meta, big_tiles, s)) return;
  if (blockIdx.x == 0 && tid < kRadixMaxPasses) s.meta->ticket[tid] = 0;
  const uint32_t tiles = (uint32_t)big_tiles[nbig];
  const uint64_t words = (uint64_t)radix_state_rows(tiles, nbig) * kRadixBins;
  for (uint64_t i = blockIdx.x * NT + tid; i < words; i += gridDim.x * NT) s.state[0][i] = 0;
  uint64_t u, uend;
  unit_range(tiles, &u, &uend);
  if (u >= uend) return;
  const uint64_t u0 = u;
  const RadixMap<ST, FL, CD> map{cd};
  for (uint32_t i = upper_index(big_tiles, nbig, u); u < uend; ++i) {
    const uint64_t first = big_tiles[i], end = big_tiles[i + 1];
    const uint32_t id = big_ids[i];
    const int64_t off = offsets[id];
    const uint32_t len = (uint32_t)(offsets[id + 1] - off);
    const uint64_t stop = end < uend ? end : uend;
    const uint64_t lo = (u - first) * T;
    const uint64_t hi = (stop - first) * T < len ? (stop - first) * T : len;
    for (uint64_t t = u + tid; t < stop; t += NT)
      s.tiles[t] = SegRadixTile{off, len, i, (uint32_t)first, (uint32_t)(t - first)};
    radix_count<NT>(lds, map, a.at(off), lo, hi, len);
    if (first >= u0 && end <= uend) {
      const bool ordered = std::is_same_v<ST, Pairs> && lds.decrease == 0;
      if (tid == 0 && lds.decrease) s.meta->trivial[0] = 1;
      for (int p = 0; p < P; ++p) {
        const uint32_t c = tid < kRadixBins ? radix_bin_count(lds, p * kRadixBins + tid) : 0u;
        segradix_finish(c, len, ordered && p < P / 2, s.base + ((size_t)i * P + p) * kRadixBins,
                        s.trivial + (size_t)i * P + p, wave_sum, &one_digit);
      }
    } else {
      const uint32_t row = blockIdx.x * 2 + (first >= u0 ? 1u : 0u);
      for (uint32_t b = tid; b < P * kRadixBins; b += NT)
        s.partial[(size_t)row * (P * kRadixBins) + b] = radix_bin_count(lds, b);
      if (tid == 0) {
        s.unordered[row] = lds.decrease;
        if (lds.decrease) s.meta->trivial[0] = 1;
        if (first >= u0) s.span[blockIdx.x] = i;
      }
      __syncthreads();
    }
    u = stop;
  }
}

// Pass blockIdx.y of the segment that begins in counting range blockIdx.x and
// goes on past it: the sum of its ranges' counts.
template <class ST>
__global__ __launch_bounds__(kSegRadixHistThreads) void segradix_scan_kernel(
    const int64_t* __restrict__ offsets, const SegMeta* __restrict__ seg_meta,
    const uint32_t* __restrict__ big_ids, const uint64_t* __restrict__ big_tiles,
    SegRadixSpace s) {
  constexpr int P = radix_passes<ST>();
  constexpr uint32_t G = kSegRadixHistThreads / kRadixBins;
  constexpr uint32_t K = 32;  // loads in flight
  __shared__ uint32_t sums[G][kRadixBins];
  __shared__ uint32_t wave_sum[kRadixBins / 64];
  __shared__ uint32_t one_digit, down;
  const uint32_t i = s.span[blockIdx.x];
  if (i == ~0u) return;
  const int pass = (int)blockIdx.y;
  const uint32_t tid = threadIdx.x;
  const uint32_t d = tid % kRadixBins, g = tid / kRadixBins;
  const uint32_t id = big_ids[i];
  const uint32_t len = (uint32_t)(offsets[id + 1] - offsets[id]);
  const uint64_t tiles = big_tiles[seg_meta->nradix];
  const uint32_t last = unit_owner(tiles, big_tiles[i + 1] - 1);
  // row 1 of the first range, row 0 of the others
  auto row = [&](uint32_t r) { return (blockIdx.x + r) * 2 + (r == 0 ? 1u : 0u); };
  const uint32_t rows = last - blockIdx.x + 1;
  if (tid == 0) down = 0;
  __syncthreads();
  uint32_t c = 0;
  for (uint32_t r0 = g; r0 < rows; r0 += G * K) {
    uint32_t w[K];
    static_for<0, (int)K>([&](auto k) {
      const uint32_t r = r0 + G * k;
      w[k] = r < rows ? s.partial[((size_t)row(r) * P + pass) * kRadixBins + d] : 0u;
    });
    static_for<0, (int)K>([&](auto k) { c += w[k]; });
  }
  sums[g][d] = c;
  const bool value_pass = std::is_same_v<ST, Pairs> && pass < P / 2;
  if (value_pass && tid < rows && s.unordered[row(tid)]) down = 1;
  __syncthreads();
  static_assert(kRadixHistBlocks <= kSegRadixHistThreads, "one thread per counting range");
  c = 0;
  if (g == 0) static_for<0, (int)G>([&](auto k) { c += sums[k][d]; });
  segradix_finish(c, len, value_pass && down == 0, s.base + ((size_t)i * P + pass) * kRadixBins,
                  s.trivial + (size_t)i * P + pass, wave_sum, &one_digit);
}

// The pass on digit `pass` of every big segment: each between its part of the
// keys and of the workspace, by the number of passes it has executed.
template <bool FL, class ST, class CD>
__global__ __launch_bounds__(kRadixThreads, 8) void segradix_pass_kernel(
    ST a, ST b, CD cd, int pass, const int64_t* __restrict__ offsets,
    const SegMeta* __restrict__ seg_meta, const uint32_t* __restrict__ big_ids,
    const uint64_t* __restrict__ big_tiles, SegRadixSpace s) {
  using MAP = RadixMap<ST, FL, CD>;
  constexpr int P = radix_passes<ST>();
  constexpr int IPT = segradix_items<ST>();
  constexpr uint32_t T = kRadixThreads * IPT;
  __shared__ RadixLds<typename MAP::U, IPT> lds;
  const uint32_t nbig = seg_meta->nradix;
  if (nbig == 0) return;
  // pairs whose values come in order in every segment: the passes on the
  // values' digits are the first to be left out, in all of them
  if (std::is_same_v<ST, Pairs> && pass < P / 2 && s.meta->trivial[0] == 0 &&
      segradix_fits(offsets, seg_meta, big_tiles, s))
    return;
  if (!segradix_fits(offsets, seg_meta, big_tiles, s)) {
    for (uint32_t i = blockIdx.x; pass == 0 && i < nbig; i += gridDim.x) {
      const int64_t off = offsets[big_ids[i]];
      segradix_in_place(a.at((size_t)off), (uint32_t)(offsets[big_ids[i] + 1] - off), MAP{cd});
    }
    return;
  }
  const uint32_t tiles = (uint32_t)big_tiles[nbig];
  const int64_t off0 = offsets[0];
  for (;;) {
    __syncthreads();  // the last tile's LDS
    if (threadIdx.x == 0) lds.tile = atomicAdd(&s.meta->ticket[pass], 1u);
    __syncthreads();
    const uint32_t u = __builtin_amdgcn_readfirstlane(lds.tile);
    if (u >= tiles) break;
    const SegRadixTile t = s.tiles[u];
    bool odd;
    if (!radix_executes<P>(s.trivial + (size_t)t.seg * P, pass, &odd)) continue;
    const ST key = a.at((size_t)t.off), alt = b.at((size_t)(t.off - off0));
    const uint32_t t0 = t.tile * T;
    const ST src = odd ? alt : key;
    radix_tile<IPT>(lds, MAP{cd}, src.at(t0), odd ? key : alt, t.len - t0 < T ? t.len - t0 : T,
                    t.tile, pass * kRadixBits, s.base + ((size_t)t.seg * P + pass) * kRadixBins,
                    radix_rows(s.state[odd ? 1 : 0], tiles, nbig, t.first, t.seg),
                    radix_rows(s.state[odd ? 0 : 1], tiles, nbig, t.first, t.seg));
  }
}

template <bool FL, class ST, class CD>
static void segradix_launch(ST a, ST b, CD cd, const int64_t* offsets, const SegScratch& sc,
                            const SegRadixSpace& s, int cus, hipStream_t st) {
  constexpr int P = radix_passes<ST>();
  segradix_hist_kernel<FL><<<kRadixHistBlocks, kSegRadixHistThreads, 0, st>>>(
      a, cd, offsets, sc.meta, sc.big_ids, sc.big_tiles, s);
  segradix_scan_kernel<ST><<<dim3(kRadixHistBlocks, P), kSegRadixHistThreads, 0, st>>>(
      offsets, sc.meta, sc.big_ids, sc.big_tiles, s);
  // two workgroups per CU (68 KiB of LDS, 1,024 threads)
  const uint32_t grid = s.max_tiles < 2u * (uint32_t)cus ? s.max_tiles : 2u * (uint32_t)cus;
  for (int p = 0; p < P; ++p)
    segradix_pass_kernel<FL><<<grid, kRadixThreads, 0, st>>>(a, b, cd, p, offsets, sc.meta,
                                                             sc.big_ids, sc.big_tiles, s);
}

template <class ST, class CD>
static void segradix_run(ST a, ST b, CD cd, const int64_t* offsets, const SegScratch& sc,
                         const SegRadixSpace& s, int cus, hipStream_t st) {
  if (cd.fmask != 0)
    segradix_launch<true>(a, b, cd, offsets, sc, s, cus, st);
  else
    segradix_launch<false>(a, b, cd, offsets, sc, s, cus, st);
}

}  // namespace bitonic
