// Kernels of the sort on 8-byte elements: int64 / uint64 / float64 keys, and
// (key, value) pairs of 4-byte words, which travel through the network as one
// 8-byte element (key word high, value word low; see Codec64).
//
// The network, the plan and the tile programs are those of the 4-byte sort
// (sections 3.1-4.2 of the paper): a tile sort of phases 1..L per 2^L-element
// tile in registers and LDS, then for every phase p > L its long strides in
// fused passes over global memory and its last L strides in a tile merge.
// The element width changes, and with it the register count (16 elements per
// thread), the regroups (high words, then low words, through 4-byte LDS
// words: a 2^13-element tile is an eight-wave workgroup of 34 KiB and four
// share a CU) and the global access pattern:
// threads move one element per register slot with lanes on consecutive
// elements (8-byte accesses for int64 keys, a 4-byte access into each array
// for pairs), which needs no alignment beyond the element's own.
//
//  wide_tile_kernel<L, RL, KIND, CX, ST>  tile sort (KIND 6), merge (KIND 3)
//                                     or phase L (KIND 7: phase t+1 on tiles
//                                     twice the sort's tile), 2^RL elements
//                                     per thread
//  column_pass_kernel<F, MIRROR, B, ST>  F long-stride steps, one column of
//                                        2^F elements per thread (column_pass.hpp)
//  wide_lanes_pass_kernel<FR, G, MIRROR, ST>  F = FR + G = 7, 8 steps, each
//                                        column split over 2^G lanes (as
//                                        column_lanes_pass_kernel)
//
// ST is the storage: Keys64 (one array of 8-byte keys) or Pairs (an array of
// 4-byte keys and an array of int32 values).  Indices >= n are absent
// INT64_MAX sentinels of the sorting domain.
#include "column_pass.hpp"
#include "launch.hpp"
#include "split_regroup.hpp"

namespace bitonic {

// One tile of 2^L elements per workgroup, `valid` of them real.  16 elements
// per thread (RL = 4) regroup through 4-byte LDS words; with fewer, the
// programs of launches with few tiles, whose workgroups need not share a CU,
// through 8-byte words.
template <int L, int RL, int KIND, int CX, class ST>
__global__ __launch_bounds__(1 << (L - RL)) void wide_tile_kernel(ST st, uint32_t n,
                                                                  Codec64 codec) {
  using PR = Prog<L, RL, KIND>;
  constexpr int LAST = PR::value.ngroups - 1;
  constexpr bool SPLIT = RL == kWideRegLog;
  __shared__ __attribute__((aligned(8))) uint32_t lds[PR::LDSW * (SPLIT ? 1 : 2)];
  const KeyIO<CX, Codec64> cd{codec};
  const uint32_t t0 = (uint32_t)blockIdx.x << L;
  const uint32_t left = n - t0;
  const uint32_t valid = left < (uint32_t)PR::T ? left : (uint32_t)PR::T;
  const bool full = valid == (uint32_t)PR::T;  // uniform
  const ST tile = st.at(t0);
  int64_t x[PR::R];
  {
    constexpr Group gr = PR::value.g[0];
    const uint32_t base = deposit<free_mask(gr, L)>(threadIdx.x);
    if (full) {
      static_for<0, PR::R>([&](auto J) { x[J] = cd.enc(tile.get(slot_index<PR, 0, J>(base))); });
    } else {
      load_checked(x, valid, [&](auto J) { return slot_index<PR, 0, J>(base); },
                   [&](uint32_t i) { return tile.get(i); }, cd, kPad64);
    }
  }
  if constexpr (SPLIT)
    run_from_split<PR, 0>(x, lds, threadIdx.x);
  else
    run_from<PR, 0>(x, reinterpret_cast<int64_t*>(lds), threadIdx.x);
  {
    uint32_t tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    constexpr Group gr = PR::value.g[LAST];
    const uint32_t base = deposit<free_mask(gr, L)>(tid);
    if (full) {
      static_for<0, PR::R>([&](auto J) { tile.put(slot_index<PR, LAST, J>(base), cd.dec(x[J])); });
    } else {
      static_for<0, PR::R>([&](auto J) {
        const uint32_t i = slot_index<PR, LAST, J>(base);
        if (i < valid) tile.put(i, cd.dec(x[J]));
      });
    }
  }
}

// F = FR + G long-stride steps of an 8-byte sort with every column of a
// 2^(q+F) block split over 2^G neighbouring lanes of 2^FR elements (the
// layout of column_lanes_pass_kernel: lane s holds rows s 2^FR .. of column
// c, or with MIRROR in the upper half of the lanes the mirrored rows of the
// mirrored column, ascending).  Whole blocks only, lane byte offsets below
// 2^(q+F) kUnit <= 2^32 (wide_lanes_fit).
template <int FR, int G, bool MIRROR, class ST>
__global__ __launch_bounds__(256) void wide_lanes_pass_kernel(ST st, int q) {
  constexpr int F = FR + G;
  constexpr int M = 1 << FR;
  constexpr uint32_t SUBS = 1u << G;
  constexpr uint32_t HALF = SUBS >> 1;
  static_assert(G >= 1 && G <= 2, "one or two lane bits per column");
  int64_t x[M];
  const uint32_t gw = blockIdx.x * 256u;                        // uniform
  const uint32_t bs = (gw >> (q + G)) << (q + F);               // uniform block start
  const uint32_t t = (gw + threadIdx.x) & ((1u << (q + G)) - 1u);
  const uint32_t s = t & (SUBS - 1u);
  const uint32_t col = t >> G;
  const bool upper = MIRROR && s >= HALF;
  const uint32_t colx = upper ? ((1u << q) - 1u) - col : col;
  const uint32_t row0 = upper ? (1u << F) - (s - HALF + 1u) * (uint32_t)M : s * (uint32_t)M;
  const uint32_t off = ((row0 << q) + colx) * ST::kUnit;       // lane byte offset
  static_for<0, M>([&](auto J) {
    const uint32_t r0 = bs + ((uint32_t)J << q);                // uniform row start
    x[J] = st.at(r0).getb(off);
  });
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (MIRROR) {
    static_for<0, M / 2>([&](auto J) {
      constexpr int j = J;
      constexpr int jj = M - 1 - j;
      const int64_t pa = lane_xor64<HALF>(x[jj]);
      const int64_t pb = lane_xor64<HALF>(x[j]);
      x[j] = keep_of_pair64(x[j], pa, upper);
      x[jj] = keep_of_pair64(x[jj], pb, upper);
    });
  }
  constexpr int NL = MIRROR ? G - 1 : G;
  static_for<0, NL>([&](auto I) {
    constexpr int b = NL - 1 - I;
    const bool bit = ((s >> b) & 1u) != 0;
    const bool keep_max = upper ? !bit : bit;
    static_for<0, M>([&](auto J) {
      x[J] = keep_of_pair64(x[J], lane_xor64<(1u << b)>(x[J]), keep_max);
    });
  });
  pass_steps<FR, false, 1>(x);
  __builtin_amdgcn_sched_barrier(0);
  static_for<0, M>([&](auto J) {
    const uint32_t r0 = bs + ((uint32_t)J << q);
    st.at(r0).putb(off, x[J]);
    __builtin_amdgcn_sched_barrier(0);
  });
}

// ---------------------------------------------------------------------------
// launchers

template <int L, int RL, int KIND, int CX, class ST>
static void launch_wide(ST st, uint32_t n, Codec64 cd, hipStream_t s) {
  wide_tile_kernel<L, RL, KIND, CX, ST><<<((n - 1) >> L) + 1, 1 << (L - RL), 0, s>>>(st, n, cd);
}

// A tile sort (kind 6: with lane steps) or a merge or phase.
template <int L, int RL, class ST>
static void launch_wide_sort(ST st, uint32_t n, Codec64 cd, int cx, hipStream_t s) {
  if (cx == CX_NONE) launch_wide<L, RL, 6, CX_NONE>(st, n, cd, s);
  else if (cx == CX_ENC) launch_wide<L, RL, 6, CX_ENC>(st, n, cd, s);
  else launch_wide<L, RL, 6, CX_BOTH>(st, n, cd, s);
}
template <int L, int RL, int KIND, class ST>
static void launch_wide_merge(ST st, uint32_t n, Codec64 cd, int cx, hipStream_t s) {
  if (cx == CX_NONE) launch_wide<L, RL, KIND, CX_NONE>(st, n, cd, s);
  else launch_wide<L, RL, KIND, CX_DEC>(st, n, cd, s);
}

// Launches of few tiles (few_tiles) take 8 elements per thread (4 for 2^10):
// one tile sort on MI355X, 16 against 8 per thread, 2^11 elements 15.1 and
// 10.0 us, 2^12 20.8 and 16.4, and 2^10 with 4 per thread 5.7; on a full chip
// (2^23 elements) 2^12-element tiles take 72 us with either.
template <class ST>
static void launch_wide_tile_st(int L, int kind, ST st, uint32_t n, Codec64 cd, int cx,
                                hipStream_t s) {
  if (codec_is_identity(cd)) cx = CX_NONE;
  const bool few = few_tiles(n, L);
  if (kind == 0) {
    switch (L) {
      case 10: launch_wide_sort<10, 2>(st, n, cd, cx, s); break;
      case 11:
        if (few) launch_wide_sort<11, 3>(st, n, cd, cx, s);
        else launch_wide_sort<11, kWideRegLog>(st, n, cd, cx, s);
        break;
      case 12:
        if (few) launch_wide_sort<12, 3>(st, n, cd, cx, s);
        else launch_wide_sort<12, kWideRegLog>(st, n, cd, cx, s);
        break;
      case 13: launch_wide_sort<13, kWideRegLog>(st, n, cd, cx, s); break;
      default: break;
    }
  } else {
    switch (L) {
      case 11:
        if (few) launch_wide_merge<11, 3, 3>(st, n, cd, cx, s);
        else launch_wide_merge<11, kWideRegLog, 3>(st, n, cd, cx, s);
        break;
      case 12: launch_wide_merge<12, kWideRegLog, 3>(st, n, cd, cx, s); break;
      case 13: launch_wide_merge<13, kWideRegLog, 3>(st, n, cd, cx, s); break;
      default: break;
    }
  }
}

template <class ST>
static void launch_wide_phase_st(int L, ST st, uint32_t n, Codec64 cd, int cx, hipStream_t s) {
  if (codec_is_identity(cd)) cx = CX_NONE;
  switch (L) {
    case 12:
      if (few_tiles(n, L)) launch_wide_merge<12, 3, 7>(st, n, cd, cx, s);
      else launch_wide_merge<12, kWideRegLog, 7>(st, n, cd, cx, s);
      break;
    case 13: launch_wide_merge<13, kWideRegLog, 7>(st, n, cd, cx, s); break;
    case 14: launch_wide_merge<14, kWideRegLog, 7>(st, n, cd, cx, s); break;
    default: break;
  }
}

template <int G, class ST>
static void launch_wide_lanes_G(bool mirror, ST st, uint32_t n, int q, hipStream_t s) {
  constexpr int FR = kWideLaneRegLog;
  const uint32_t blocks = n >> (FR + 8);  // n / 2^FR threads, 256 per workgroup
  if (mirror)
    wide_lanes_pass_kernel<FR, G, true, ST><<<blocks, 256, 0, s>>>(st, q);
  else
    wide_lanes_pass_kernel<FR, G, false, ST><<<blocks, 256, 0, s>>>(st, q);
}

template <class ST>
static void launch_wide_pass_st(int f, bool mirror, ST st, uint32_t n, int q, hipStream_t s) {
  if (f > kWideFuseMaxColumn) {  // the planner checked wide_lanes_fit
    if (f == kWideLaneRegLog + 1) launch_wide_lanes_G<1>(mirror, st, n, q, s);
    if (f == kWideLaneRegLog + 2) launch_wide_lanes_G<2>(mirror, st, n, q, s);
    return;
  }
  switch (f) {
    case 1: launch_column_pass_F<1>(mirror, st, n, q, s); break;
    case 2: launch_column_pass_F<2>(mirror, st, n, q, s); break;
    case 3: launch_column_pass_F<3>(mirror, st, n, q, s); break;
    case 4: launch_column_pass_F<4>(mirror, st, n, q, s); break;
    case 5: launch_column_pass_F<5>(mirror, st, n, q, s); break;
    case 6: launch_column_pass_F<6>(mirror, st, n, q, s); break;
    default: break;
  }
}

void launch_wide_tile(int L, int kind, int64_t* keys64, int32_t* keys32, int32_t* values,
                      uint32_t n, Codec64 cd, int cx, hipStream_t s) {
  if (values)
    launch_wide_tile_st(L, kind, Pairs{keys32, values}, n, cd, cx, s);
  else
    launch_wide_tile_st(L, kind, Keys64{keys64}, n, cd, cx, s);
}

void launch_wide_phase(int L, int64_t* keys64, int32_t* keys32, int32_t* values, uint32_t n,
                       Codec64 cd, int cx, hipStream_t s) {
  if (values)
    launch_wide_phase_st(L, Pairs{keys32, values}, n, cd, cx, s);
  else
    launch_wide_phase_st(L, Keys64{keys64}, n, cd, cx, s);
}

void launch_wide_pass(int f, bool mirror, int64_t* keys64, int32_t* keys32, int32_t* values,
                      uint32_t n, int q, hipStream_t s) {
  if (values)
    launch_wide_pass_st(f, mirror, Pairs{keys32, values}, n, q, s);
  else
    launch_wide_pass_st(f, mirror, Keys64{keys64}, n, q, s);
}

}  // namespace bitonic
