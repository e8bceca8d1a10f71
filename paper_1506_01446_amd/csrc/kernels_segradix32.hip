// Digit sort of the big segments of 4-byte keys, and its dispatch.
#include "segradix_kernels.hpp"

namespace bitonic {

void segradix_run_keys32(const SegData& d, const int64_t* offsets, const SegScratch& sc,
                         const SegRadixSpace& s, int cus, hipStream_t st) {
  segradix_run(Keys32{d.keys}, Keys32{reinterpret_cast<int32_t*>(s.alt)}, d.cd, offsets, sc, s,
               cus, st);
}

void launch_segradix(const SegData& d, const int64_t* offsets, const SegScratch& sc,
                     const SegRadixSpace& s, int cus, hipStream_t st) {
  if (d.keys64)
    segradix_run_keys64(d, offsets, sc, s, cus, st);
  else if (d.values)
    segradix_run_pairs(d, offsets, sc, s, cus, st);
  else
    segradix_run_keys32(d, offsets, sc, s, cus, st);
}

}  // namespace bitonic
