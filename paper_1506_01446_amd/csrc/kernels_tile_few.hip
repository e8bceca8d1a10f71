// Tile kernels of launches with few tiles: eight keys per thread (see
// launch_tile_few; tile_kernels.hpp).
#include "tile_kernels.hpp"

namespace bitonic {

constexpr int kFewRegLog = 3;

template <int L, int KIND, int CX>
static void launch_few(int32_t* keys, uint32_t n, Codec cd, hipStream_t st) {
  tile_kernel<L, kFewRegLog, KIND, CX>
      <<<((n - 1) >> L) + 1, 1 << (L - kFewRegLog), 0, st>>>(keys, n, cd);
}

template <int L>
static void launch_few_sort(int32_t* keys, uint32_t n, Codec cd, int cx, hipStream_t st) {
  if (cx == CX_NONE) launch_few<L, 4, CX_NONE>(keys, n, cd, st);
  else if (cx == CX_ENC) launch_few<L, 4, CX_ENC>(keys, n, cd, st);
  else launch_few<L, 4, CX_BOTH>(keys, n, cd, st);
}

template <int L, int KIND>
static void launch_few_merge(int32_t* keys, uint32_t n, Codec cd, int cx, hipStream_t st) {
  if (cx == CX_NONE) launch_few<L, KIND, CX_NONE>(keys, n, cd, st);
  else launch_few<L, KIND, CX_DEC>(keys, n, cd, st);
}

bool launch_tile_few(int L, int kind, int32_t* keys, uint32_t n, Codec cd, int cx,
                     hipStream_t st) {
  if (codec_is_identity(cd)) cx = CX_NONE;
  if (kind == 4) {
    switch (L) {
      case 9: launch_few_sort<9>(keys, n, cd, cx, st); return true;
      case 10: launch_few_sort<10>(keys, n, cd, cx, st); return true;
      case 11: launch_few_sort<11>(keys, n, cd, cx, st); return true;
      case 12: launch_few_sort<12>(keys, n, cd, cx, st); return true;
      default: return false;
    }
  }
  if (kind == 1 && L == 11) launch_few_merge<11, 1>(keys, n, cd, cx, st);
  else if (kind == 1 && L == 12) launch_few_merge<12, 1>(keys, n, cd, cx, st);
  else if (kind == 5 && L == 12) launch_few_merge<12, 5>(keys, n, cd, cx, st);
  else if (kind == 5 && L == 13) launch_few_merge<13, 5>(keys, n, cd, cx, st);
  else return false;
  return true;
}

}  // namespace bitonic
