// Digit sort of the big segments of 8-byte keys.
#include "segradix_kernels.hpp"

namespace bitonic {

void segradix_run_keys64(const SegData& d, const int64_t* offsets, const SegScratch& sc,
                         const SegRadixSpace& s, int cus, hipStream_t st) {
  segradix_run(Keys64{d.keys64}, Keys64{reinterpret_cast<int64_t*>(s.alt)}, d.cd64, offsets, sc,
               s, cus, st);
}

}  // namespace bitonic
