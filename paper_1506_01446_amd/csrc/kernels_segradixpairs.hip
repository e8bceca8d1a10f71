// Digit sort of the big segments of (key, value) pairs.
#include "segradix_kernels.hpp"

namespace bitonic {

void segradix_run_pairs(const SegData& d, const int64_t* offsets, const SegScratch& sc,
                        const SegRadixSpace& s, int cus, hipStream_t st) {
  int32_t* const alt = reinterpret_cast<int32_t*>(s.alt);
  segradix_run(Pairs{d.keys, d.values}, Pairs{alt, alt + s.elems}, d.cd64, offsets, sc, s, cus, st);
}

}  // namespace bitonic
