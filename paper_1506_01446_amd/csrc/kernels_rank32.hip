// Rank sort of 4-byte keys, and the dispatch.
#include "rank_kernels.hpp"

namespace bitonic {

void rank_run_keys32(const RadixData& d, uint32_t n, void* workspace, hipStream_t st) {
  rank_run(Keys32{d.keys}, Keys32{static_cast<int32_t*>(workspace)}, d.cd, n, st);
}

void launch_rank_sort(const RadixData& d, uint32_t n, void* workspace, hipStream_t st) {
  if (d.keys64)
    rank_run_keys64(d, n, workspace, st);
  else if (d.values)
    rank_run_pairs(d, n, workspace, st);
  else
    rank_run_keys32(d, n, workspace, st);
}

}  // namespace bitonic
