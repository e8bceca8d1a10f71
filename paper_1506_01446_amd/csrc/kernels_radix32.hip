// Digit sort of 4-byte keys, and what its storages share.
#include "radix_kernels.hpp"

namespace bitonic {

// One workgroup per pass: sums the counting workgroups' rows (four threads
// per digit, 32 loads of each in flight: the sum is latency-bound) and scans
// the 256 sums.
__global__ __launch_bounds__(1024) void radix_scan_kernel(const uint32_t* __restrict__ partial,
                                                          const uint32_t* __restrict__ unordered,
                                                          uint32_t blocks, uint32_t n, int pairs,
                                                          uint32_t* __restrict__ base,
                                                          RadixMeta* __restrict__ meta) {
  constexpr uint32_t K = 32;
  __shared__ uint32_t sums[4][kRadixBins];
  __shared__ uint32_t wave_sum[kRadixBins / 64];
  __shared__ uint32_t one_digit, down;
  const uint32_t tid = threadIdx.x;
  const uint32_t pass = blockIdx.x;
  const uint32_t row = gridDim.x * kRadixBins;
  const uint32_t d = tid % kRadixBins, g = tid / kRadixBins;
  if (tid == 0) {
    one_digit = 0;
    down = 0;
  }
  __syncthreads();
  uint32_t s = 0;
  for (uint32_t b0 = g; b0 < blocks; b0 += 4 * K) {
    uint32_t w[K];
    static_for<0, (int)K>([&](auto k) {
      const uint32_t b = b0 + 4 * k;
      w[k] = b < blocks ? partial[(size_t)b * row + pass * kRadixBins + d] : 0u;
    });
    static_for<0, (int)K>([&](auto k) { s += w[k]; });
  }
  sums[g][d] = s;
  // pairs whose values never decrease: the passes on the value's digits
  // would keep every pair of equal keys in place, and the passes on the
  // keys' digits do that anyway
  const bool value_pass = pairs && pass < sizeof(int32_t) * 8 / kRadixBits;
  if (value_pass && tid < blocks && unordered[tid]) down = 1;
  __syncthreads();
  const uint32_t t = g == 0 ? sums[0][d] + sums[1][d] + sums[2][d] + sums[3][d] : 0u;
  if (g == 0 && t == n) one_digit = 1;
  const uint32_t before = radix_scan_bins(t, g == 0, tid >> 6, wave_sum);
  if (g == 0) base[pass * kRadixBins + d] = before;
  if (tid == 0) meta->trivial[pass] = one_digit || (value_pass && !down) ? 1u : 0u;
}

void launch_radix_scan(const RadixSpace& s, uint32_t n, int passes, bool pairs, hipStream_t st) {
  static_assert(kRadixHistBlocks <= 1024, "one thread per counting workgroup");
  radix_scan_kernel<<<passes, 1024, 0, st>>>(s.partial, s.unordered, radix_hist_blocks(n), n,
                                             pairs ? 1 : 0, s.base, s.meta);
}

void radix_run_keys32(const RadixData& d, uint32_t n, const RadixSpace& s, hipStream_t st) {
  radix_run(Keys32{d.keys}, Keys32{reinterpret_cast<int32_t*>(s.alt)}, d.cd, n, s, st);
}

void launch_radix_sort(const RadixData& d, uint32_t n, void* workspace, hipStream_t st) {
  RadixSpace s;
  radix_space(static_cast<char*>(workspace), n, d.keys64 || d.values ? 8 : 4, &s);
  if (d.keys64)
    radix_run_keys64(d, n, s, st);
  else if (d.values)
    radix_run_pairs(d, n, s, st);
  else
    radix_run_keys32(d, n, s, st);
}

}  // namespace bitonic
