// Digit sort of 8-byte keys.
#include "radix_kernels.hpp"

namespace bitonic {

void radix_run_keys64(const RadixData& d, uint32_t n, const RadixSpace& s, hipStream_t st) {
  radix_run(Keys64{d.keys64}, Keys64{reinterpret_cast<int64_t*>(s.alt)}, d.cd64, n, s, st);
}

}  // namespace bitonic
