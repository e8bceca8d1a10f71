// Digit sort of (key, value) pairs: 8-byte elements, the value's digits
// first.
#include "radix_kernels.hpp"

namespace bitonic {

void radix_run_pairs(const RadixData& d, uint32_t n, const RadixSpace& s, hipStream_t st) {
  int32_t* const alt = reinterpret_cast<int32_t*>(s.alt);
  radix_run(Pairs{d.keys, d.values}, Pairs{alt, alt + n}, d.cd64, n, s, st);
}

}  // namespace bitonic
