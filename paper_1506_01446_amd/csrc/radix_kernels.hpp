// Kernel templates of the digit sort (radix.hpp), over a storage type ST
// (column_pass.hpp): Keys32, Keys64 or Pairs.
//
// Launch sequence (one stream, no host synchronisation):
//   radix_hist_kernel  reads the elements once and counts every digit of
//                      every pass, a row of counts per workgroup
//   radix_scan_kernel  one workgroup per pass sums the rows and scans them:
//                      where each digit's elements begin in the pass's output
//   radix_pass_kernel  one launch per digit: every tile of elements is put in
//                      order of its digit in LDS, and written behind the
//                      elements of the same digit of the tiles before it
// Every pass keeps the order of elements with equal digits, so after the
// last one the array is in order; elements that are equal in all digits are
// identical, so the result is the unique one of the network's sorts.
#pragma once

#include <type_traits>

#include "column_pass.hpp"
#include "radix.hpp"

namespace bitonic {

// Elements as unsigned numbers in sorting order (the codecs map to signed
// order).  FL: the type's map depends on the sign (float keys); the others
// are one xor.
template <class ST, bool FL, class CD>
struct RadixMap {
  using E = typename ST::E;
  using U = std::make_unsigned_t<E>;
  static constexpr U kSign = (U)1 << (8 * sizeof(U) - 1);
  CD cd;
  __device__ __forceinline__ U enc(E v) const {
    if constexpr (FL) return (U)cd.enc(v) ^ kSign;
    else return (U)v ^ ((U)cd.flip ^ kSign);
  }
  __device__ __forceinline__ E dec(U u) const {
    if constexpr (FL) return cd.dec((E)(u ^ kSign));
    else return (E)(u ^ ((U)cd.flip ^ kSign));
  }
};

template <class ST>
constexpr int radix_passes() {
  return (int)sizeof(typename ST::E) * 8 / kRadixBits;
}

// ---------------------------------------------------------------------------
// counting

// One workgroup's waves fill a CU's LDS-atomic pipe, so a share of the array
// can be large and its rows of counts few (radix_hist_blocks).
constexpr int kRadixHistThreads = 1024;

// LDS of a counting workgroup.  A bin is kept in 64 / passes copies (64 KiB
// in all, two workgroups per CU), lane l adding to copy l mod copies: an
// array whose digits are all alike then adds at most `passes` times in turn
// to one word per wave, and not 64 times.
template <class ST>
struct RadixBinsLds {
  static constexpr int P = radix_passes<ST>();
  static constexpr int C = 64 / P;
  uint32_t bins[P * kRadixBins * C];
  uint32_t decrease;
};

// Counts every digit of elements lo .. hi of a (n in all) with the whole
// workgroup of NT threads; then bin b's count (pass b / 256, digit b mod 256) is
// radix_bin_count(lds, b), and lds.decrease is 1 if a pair's value (Pairs) is
// above the next one's.
template <uint32_t NT, class MAP, class ST>
__device__ __forceinline__ void radix_count(RadixBinsLds<ST>& lds, const MAP& map, const ST& a,
                                            uint64_t lo, uint64_t hi, uint64_t n) {
  using E = typename ST::E;
  using L = RadixBinsLds<ST>;
  const uint32_t tid = threadIdx.x;
  for (uint32_t i = tid; i < L::P * kRadixBins * L::C; i += NT) lds.bins[i] = 0;
  if (tid == 0) lds.decrease = 0;
  __syncthreads();
  const uint32_t copy = tid % L::C;
  auto count = [&](E x) {
    const auto u = map.enc(x);
    static_for<0, L::P>([&](auto p) {
      const uint32_t d = (uint32_t)(u >> (kRadixBits * (int)p)) & (kRadixBins - 1);
      atomicAdd(&lds.bins[((int)p * kRadixBins + d) * L::C + copy], 1u);
    });
  };
  constexpr int U = 8;
  uint64_t i = lo + tid;
  for (; i + (U - 1) * NT < hi; i += U * NT) {
    E x[U];
    static_for<0, U>([&](auto J) { x[J] = a.get((uint32_t)(i + J * NT)); });
    static_for<0, U>([&](auto J) { count(x[J]); });
  }
  if (i < hi) {
    E x[U];
    static_for<0, U>([&](auto J) { x[J] = a.get((uint32_t)(i + J * NT < hi ? i + J * NT : i)); });
    static_for<0, U>([&](auto J) {
      if (i + J * NT < hi) count(x[J]);
    });
  }
  if constexpr (std::is_same_v<ST, Pairs>) {
    // U comparisons' loads in flight, those past the end at the first one's
    // place (one at a time the loop took longer than the counting)
    bool down = false;
    const uint64_t last = hi < n ? hi : n - 1;  // j + 1 < n
    for (uint64_t j = lo + tid; j < last; j += U * NT) {
      int32_t v[U], w[U];
      static_for<0, U>([&](auto J) {
        const uint64_t at = j + J * NT < last ? j + J * NT : j;
        v[J] = a.v[at];
        w[J] = a.v[at + 1];
      });
      static_for<0, U>([&](auto J) { down |= v[J] > w[J]; });
    }
    if (down) lds.decrease = 1;
  }
  __syncthreads();
}

template <class ST>
__device__ __forceinline__ uint32_t radix_bin_count(const RadixBinsLds<ST>& lds, uint32_t b) {
  uint32_t s = 0;
  static_for<0, RadixBinsLds<ST>::C>([&](auto k) {
    s += lds.bins[b * RadixBinsLds<ST>::C + (k + threadIdx.x) % RadixBinsLds<ST>::C];
  });
  return s;
}

// Each workgroup counts a contiguous share of the array.
template <bool FL, class ST, class CD>
__global__ __launch_bounds__(kRadixHistThreads) void radix_hist_kernel(
    ST a, uint32_t n, CD cd, RadixMeta* __restrict__ meta, uint32_t* __restrict__ partial,
    uint32_t* __restrict__ unordered, uint32_t* __restrict__ state, uint32_t state_words) {
  constexpr int P = radix_passes<ST>();
  constexpr uint32_t NT = kRadixHistThreads;
  __shared__ RadixBinsLds<ST> lds;
  const uint32_t tid = threadIdx.x;
  // the first executed pass's prefix sums, and every pass's ticket
  for (uint32_t i = blockIdx.x * NT + tid; i < state_words; i += gridDim.x * NT) state[i] = 0;
  if (blockIdx.x == 0 && tid < kRadixMaxPasses) meta->ticket[tid] = 0;
  const uint32_t per = ((n - 1) / gridDim.x / NT + 1) * NT;
  const uint64_t lo = (uint64_t)blockIdx.x * per;
  const uint64_t hi = lo + per < n ? lo + per : n;
  radix_count<NT>(lds, RadixMap<ST, FL, CD>{cd}, a, lo, hi, n);
  for (uint32_t b = tid; b < P * kRadixBins; b += NT)
    partial[(size_t)blockIdx.x * (P * kRadixBins) + b] = radix_bin_count(lds, b);
  if (tid == 0) unordered[blockIdx.x] = lds.decrease;
}

// With 256 consecutive threads (four waves, wave_sum of four words): the sum
// of the smaller digits' counts.  Every thread of the workgroup calls it;
// `in` says whether the thread is one of the 256, `four` its wave among them.
__device__ __forceinline__ uint32_t radix_scan_bins(uint32_t count, bool in, uint32_t four,
                                                    uint32_t* wave_sum) {
  const uint32_t lane = threadIdx.x & 63u;
  uint32_t incl = count;
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(incl, o);
    if (lane >= (uint32_t)o) incl += y;
  }
  if (in && lane == 63) wave_sum[four] = incl;
  __syncthreads();
  uint32_t before = incl - count;
  if (in)
    for (uint32_t w = 0; w < four; ++w) before += wave_sum[w];
  __syncthreads();
  return before;
}

// ---------------------------------------------------------------------------
// one pass

// Words of the prefix sums.  A tile's counts and the counts ahead of a
// supergroup are written once, with a flag; the sums of groups and
// supergroups grow by their tiles' additions, with the number of additions
// above the sum (a sum is at most 256 tiles of 2^14 elements).
constexpr uint32_t kRadixReady = 1u << 31;
constexpr uint32_t kRadixGroupOne = 1u << 27;
constexpr uint32_t kRadixSuperOne = 1u << 23;

__device__ __forceinline__ uint32_t radix_state_get(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void radix_state_put(uint32_t* p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void radix_state_add(uint32_t* p, uint32_t v) {
  (void)__hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Sum over `count` (uniform, < kRadixGroup) rows of the word at p, each
// waited for until it holds FULL times ONE.  Flag and count are one word, so
// a word that is read complete holds its count; no other memory is read on
// its strength.
template <uint32_t ONE, uint32_t FULL>
__device__ __forceinline__ uint32_t radix_state_sum(const uint32_t* p, uint32_t count) {
  constexpr int K = 8;  // loads in flight
  uint32_t sum = 0;
  for (uint32_t r = 0; r < count;) {
    uint32_t w[K];
    bool all = true;
    uint32_t part = 0;
    static_for<0, K>([&](auto k) {
      w[k] = ONE * FULL;
      if (r + (uint32_t)k < count) w[k] = radix_state_get(p + (size_t)(r + k) * kRadixBins);
    });
    static_for<0, K>([&](auto k) {
      all = all && w[k] >= ONE * FULL;
      part += w[k] & (ONE - 1);
    });
    if (__builtin_amdgcn_ballot_w64(!all) == 0) {
      sum += part;
      r += K;
    } else {
      __builtin_amdgcn_s_sleep(1);
    }
  }
  return sum;
}

// Trivial passes are left out, an even number of them, so that the last
// executed pass writes the caller's array.  False if pass is one of them;
// else *odd says whether an odd number of passes ran before it.
template <int P>
__device__ __forceinline__ bool radix_executes(const uint32_t* trivial, int pass, bool* odd) {
  int leave = 0;
  static_for<0, P>([&](auto p) { leave += (int)trivial[p]; });
  leave &= ~1;
  int executed = 0;
  bool skip = false;
  for (int p = 0; p <= pass; ++p) {
    executed += p > 0 && !skip;
    skip = leave > 0 && trivial[p] != 0;
    leave -= skip;
  }
  *odd = (executed & 1) != 0;
  return !skip;
}

// Where the prefix sums of an array's pass are: rows of 256 words for its
// tiles, their groups, their supergroups, and what is ahead of those.
struct RadixRows {
  uint32_t* tiles;
  uint32_t* groups;
  uint32_t* supers;
  uint32_t* ahead;
};

// The rows of an array whose first tile is `first` of the sort's `tiles`
// tiles, behind `arrays` arrays before it: every array begins its groups and
// supergroups with rows of its own (sum of ceil(t / 16) over them is at most
// first / 16 + arrays).
__device__ __forceinline__ RadixRows radix_rows(uint32_t* state, uint32_t tiles, uint32_t narrays,
                                                uint32_t first, uint32_t arrays) {
  const size_t g = (size_t)tiles + (first >> kRadixGroupLog) + arrays;
  const size_t g_rows = (size_t)(tiles >> kRadixGroupLog) + narrays;
  const size_t s_rows = (size_t)(tiles >> (2 * kRadixGroupLog)) + narrays;
  const size_t s = (size_t)tiles + g_rows + (first >> (2 * kRadixGroupLog)) + arrays;
  return RadixRows{state + (size_t)first * kRadixBins, state + g * kRadixBins,
                   state + s * kRadixBins, state + (s + s_rows) * kRadixBins};
}

// LDS of a pass's workgroup.
template <class U, int IPT>
struct RadixLds {
  static constexpr uint32_t NT = kRadixThreads;
  static constexpr int NW = NT / 64;
  static constexpr size_t TILE = (size_t)NT * IPT * sizeof(U);
  static constexpr size_t HIST = (size_t)NW * kRadixBins * 4;
  // the waves' digit counts, and then the tile in order of its digit
  alignas(16) char shared[TILE > HIST ? TILE : HIST];
  uint32_t part[2][kRadixBins];
  uint32_t shift_of[kRadixBins];  // output index minus tile position, per digit
  uint32_t wave_sum[kRadixBins / 64];
  uint32_t tile;
};

// One tile of a pass on the digit at bit `shift`: tile `tile` of an array,
// its elements src.get(0 .. valid), written to their places in dst (the
// output array's start).  base: where each digit begins in the output.
//
// The caller takes tiles from a ticket, so every tile before this one is
// already being worked on; what is waited for below are the counts of those
// tiles, which each publishes without waiting for anything, and (in the
// first tile of a supergroup) the sums ahead of the supergroup before, which
// wait for earlier tiles only.  So the wait ends whatever else runs on the
// GPU, in whatever order the hardware starts workgroups.
//
// The tile's digits are counted before they are ranked: the counts are on
// their way to the tiles behind while this one does the ranking, its longest
// part.  The ranking's ballots bound the pass (61 % VALU busy at 2^24 4-byte
// keys, 46 us against 19 us for a copy of the keys): about 70 VALU
// instructions per element, 32 of them the ballots' masks.
template <int IPT, class ST, class MAP>
__device__ __forceinline__ void radix_tile(RadixLds<typename MAP::U, IPT>& lds, const MAP& map,
                                           const ST& src, const ST& dst, uint32_t valid,
                                           uint32_t tile, int shift, const uint32_t* base,
                                           const RadixRows& rows, const RadixRows& clear) {
  using U = typename MAP::U;
  constexpr uint32_t NT = kRadixThreads;
  constexpr int NW = NT / 64;
  constexpr uint32_t T = NT * IPT;
  constexpr uint32_t BINS = kRadixBins;
  U* const exch = reinterpret_cast<U*>(lds.shared);
  uint32_t (*const whist)[BINS] = reinterpret_cast<uint32_t (*)[BINS]>(lds.shared);
  auto digit = [&](U u) { return (uint32_t)(u >> shift) & (BINS - 1); };
  const uint32_t tid = threadIdx.x;
  const uint32_t lane = tid & 63u;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t super = tile >> (2 * kRadixGroupLog), group = tile >> kRadixGroupLog;
  const uint32_t in_group = tile & (kRadixGroup - 1), in_super = group & (kRadixGroup - 1);

  for (uint32_t i = tid; i < NW * BINS; i += NT) (&whist[0][0])[i] = 0;
  // Items of a wave are 64 consecutive elements each.  Past the end of the
  // array the largest element stands in: it ranks behind the real ones of
  // its digit, the last.
  U x[IPT];
  const uint32_t first = wave * (64u * IPT) + lane;
  if (valid == T) {
    static_for<0, IPT>([&](auto I) { x[I] = (U)src.getb((first + 64u * I) * ST::kUnit); });
    static_for<0, IPT>([&](auto I) { x[I] = map.enc((typename ST::E)x[I]); });
  } else {
    // every load before the first use (load_checked); valid > 0
    static_for<0, IPT>([&](auto I) {
      x[I] = (U)src.get(first + 64u * I < valid ? first + 64u * I : 0u);
    });
    static_for<0, IPT>([&](auto I) {
      x[I] = first + 64u * I < valid ? map.enc((typename ST::E)x[I]) : ~(U)0;
    });
  }
  // this tile's rows of the next executed pass
  if (tid < BINS) {
    clear.tiles[(size_t)tile * BINS + tid] = 0;
    if (in_group == 0) clear.groups[(size_t)group * BINS + tid] = 0;
    if (in_group == 0 && in_super == 0) {
      clear.supers[(size_t)super * BINS + tid] = 0;
      clear.ahead[(size_t)super * BINS + tid] = 0;
    }
  }
  __syncthreads();

  uint32_t* const wh = whist[wave];
  U differ = 0;
  static_for<1, IPT>([&](auto I) { differ |= x[I] ^ x[0]; });
  const uint32_t d0 = __builtin_amdgcn_readfirstlane(digit(x[0]));
  if (__builtin_amdgcn_ballot_w64(digit(differ) != 0 || digit(x[0]) != d0) == 0) {
    // one digit in the whole wave: its lanes would add to one word in turn
    if (lane == 0) wh[d0] = 64u * IPT;
  } else {
    static_for<0, IPT>([&](auto I) {
      __hip_atomic_fetch_add(&wh[digit(x[I])], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    });
  }
  __syncthreads();
  uint32_t total = 0, incl = 0, excl = 0;
  if (tid < BINS) {
    static_for<0, NW>([&](auto w) { total += whist[w][tid]; });
    const uint32_t real = tid == BINS - 1 ? total - (T - valid) : total;
    radix_state_put(rows.tiles + (size_t)tile * BINS + tid, kRadixReady | real);
    radix_state_add(rows.groups + (size_t)group * BINS + tid, kRadixGroupOne | real);
    radix_state_add(rows.supers + (size_t)super * BINS + tid, kRadixSuperOne | real);
    incl = total;
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(incl, o);
      if (lane >= (uint32_t)o) incl += y;
    }
    if (lane == 63) lds.wave_sum[wave] = incl;
  }
  __syncthreads();
  if (tid < BINS) {
    // where each digit begins in the tile, then where each wave's share does
    uint32_t before = 0;
    for (uint32_t w = 0; w < wave; ++w) before += lds.wave_sum[w];
    excl = before + incl - total;
    uint32_t run = excl;
    static_for<0, NW>([&](auto w) {
      const uint32_t c = whist[w][tid];
      whist[w][tid] = run;
      run += c;
    });
  }
  __syncthreads();
  // Positions in the tile: the lanes of an item that share a digit are found
  // with one ballot per bit of it; each takes the digit's next position plus
  // the number of its fellows in lower lanes.
  uint32_t pos[(IPT + 1) / 2];  // two 16-bit positions a word
  static_for<0, IPT>([&](auto I) {
    const uint32_t d = digit(x[I]);
    uint32_t lo = ~0u, hi = ~0u;
    static_for<0, kRadixBits>([&](auto B) {
      int32_t m = (int32_t)(d << (31 - (int)B)) >> 31;
      asm volatile("" : "+v"(m));  // keep it a mask (one bfe, used three times)
      const uint64_t v = __builtin_amdgcn_ballot_w64(m != 0);
      lo = __builtin_amdgcn_bitop3_b32(lo, (uint32_t)m, (uint32_t)v, 0x90);  // lo & ~(m ^ v)
      hi = __builtin_amdgcn_bitop3_b32(hi, (uint32_t)m, (uint32_t)(v >> 32), 0x90);
    });
    const uint32_t lower = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0));
    // LDS operations of a wave keep their order: every lane reads, then the
    // digit's lowest lane moves the position on
    const uint32_t at =
        lower + __hip_atomic_load(&wh[d], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    if (lower == 0)
      __hip_atomic_fetch_add(&wh[d], (uint32_t)(__popc(lo) + __popc(hi)), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_WAVEFRONT);
    if constexpr (I % 2 == 0) pos[I / 2] = at;
    else pos[I / 2] |= at << 16;
  });
  __syncthreads();
  static_for<0, IPT>([&](auto I) { exch[(pos[I / 2] >> (I % 2 * 16)) & 0xFFFFu] = x[I]; });

  // the elements of each digit ahead of this tile's
  const uint32_t d = tid & (BINS - 1);
  if (wave < BINS / 64) {
    lds.part[0][d] =
        radix_state_sum<kRadixReady, 1>(rows.tiles + (size_t)(tile - in_group) * BINS + d,
                                        in_group) -
        excl;
  } else if (wave < 2 * BINS / 64) {
    uint32_t start;
    if (super == 0) {
      start = base[d];
    } else {
      start = radix_state_sum<kRadixReady, 1>(rows.ahead + (size_t)(super - 1) * BINS + d, 1);
      start += radix_state_sum<kRadixSuperOne, kRadixGroup * kRadixGroup>(
          rows.supers + (size_t)(super - 1) * BINS + d, 1);
    }
    if (in_group == 0 && in_super == 0)
      radix_state_put(rows.ahead + (size_t)super * BINS + d, kRadixReady | start);
    lds.part[1][d] = start + radix_state_sum<kRadixGroupOne, kRadixGroup>(
                                 rows.groups + (size_t)(group - in_super) * BINS + d, in_super);
  }
  __syncthreads();
  if (tid < BINS) lds.shift_of[tid] = lds.part[0][tid] + lds.part[1][tid];
  __syncthreads();
  auto put = [&](uint32_t i) {
    const U u = exch[i];
    dst.put(lds.shift_of[digit(u)] + i, map.dec(u));
  };
  if (valid == T) {
    static_for<0, IPT>([&](auto I) { put((uint32_t)I * NT + tid); });
  } else {
    static_for<0, IPT>([&](auto I) {
      if ((uint32_t)I * NT + tid < valid) put((uint32_t)I * NT + tid);
    });
  }
}

// The pass on digit `pass` of the elements: from a to b after an even number
// of executed passes, else from b to a.  One workgroup per tile.
template <bool FL, int IPT, class ST, class CD>
__global__ __launch_bounds__(kRadixThreads, 8) void radix_pass_kernel(
    ST a, ST b, uint32_t n, CD cd, int pass, RadixMeta* __restrict__ meta,
    const uint32_t* __restrict__ base, uint32_t* __restrict__ state_a,
    uint32_t* __restrict__ state_b) {
  using MAP = RadixMap<ST, FL, CD>;
  constexpr uint32_t T = kRadixThreads * IPT;
  __shared__ RadixLds<typename MAP::U, IPT> lds;
  bool odd;
  if (!radix_executes<radix_passes<ST>()>(meta->trivial, pass, &odd)) return;
  if (threadIdx.x == 0) lds.tile = atomicAdd(&meta->ticket[pass], 1u);
  __syncthreads();
  const uint32_t tile = __builtin_amdgcn_readfirstlane(lds.tile);
  const uint32_t t0 = tile * T;
  const ST src = odd ? b : a;
  const ST dst = odd ? a : b;
  radix_tile<IPT>(lds, MAP{cd}, src.at(t0), dst, n - t0 < T ? n - t0 : T, tile,
                  pass * kRadixBits, base + pass * kRadixBins,
                  radix_rows(odd ? state_b : state_a, gridDim.x, 1, 0, 0),
                  radix_rows(odd ? state_a : state_b, gridDim.x, 1, 0, 0));
}

// ---------------------------------------------------------------------------
// launches of one sort

template <bool FL, int IPT, class ST, class CD>
static void radix_run_items(ST a, ST b, CD cd, uint32_t n, const RadixSpace& s, hipStream_t st) {
  constexpr int P = radix_passes<ST>();
  constexpr uint32_t T = kRadixThreads * IPT;
  const uint32_t tiles = n / T + (n % T != 0);
  radix_hist_kernel<FL><<<radix_hist_blocks(n), kRadixHistThreads, 0, st>>>(
      a, n, cd, s.meta, s.partial, s.unordered, s.state[0], radix_state_rows(tiles, 1) * kRadixBins);
  launch_radix_scan(s, n, P, std::is_same_v<ST, Pairs>, st);
  for (int p = 0; p < P; ++p)
    radix_pass_kernel<FL, IPT><<<tiles, kRadixThreads, 0, st>>>(a, b, n, cd, p, s.meta, s.base,
                                                                s.state[0], s.state[1]);
}

template <class ST, class CD>
static void radix_run(ST a, ST b, CD cd, uint32_t n, const RadixSpace& s, hipStream_t st) {
  constexpr int EB = (int)sizeof(typename ST::E);
  constexpr int M = EB == 4 ? 16 : 8;  // radix_items
  const int items = radix_items(n, EB);
  if (cd.fmask != 0) {
    if (items == M) radix_run_items<true, M>(a, b, cd, n, s, st);
    else if (items == M / 2) radix_run_items<true, M / 2>(a, b, cd, n, s, st);
    else radix_run_items<true, M / 4>(a, b, cd, n, s, st);
  } else {
    if (items == M) radix_run_items<false, M>(a, b, cd, n, s, st);
    else if (items == M / 2) radix_run_items<false, M / 2>(a, b, cd, n, s, st);
    else radix_run_items<false, M / 4>(a, b, cd, n, s, st);
  }
}

}  // namespace bitonic
