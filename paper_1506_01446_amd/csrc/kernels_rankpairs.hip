// Rank sort of (key, value) pairs.
#include "rank_kernels.hpp"

namespace bitonic {

void rank_run_pairs(const RadixData& d, uint32_t n, void* workspace, hipStream_t st) {
  int32_t* const alt = static_cast<int32_t*>(workspace);
  rank_run(Pairs{d.keys, d.values}, Pairs{alt, alt + n}, d.cd64, n, st);
}

}  // namespace bitonic
