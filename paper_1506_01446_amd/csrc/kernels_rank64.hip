// Rank sort of 8-byte keys.
#include "rank_kernels.hpp"

namespace bitonic {

void rank_run_keys64(const RadixData& d, uint32_t n, void* workspace, hipStream_t st) {
  rank_run(Keys64{d.keys64}, Keys64{static_cast<int64_t*>(workspace)}, d.cd64, n, st);
}

}  // namespace bitonic
