// Internal: order-preserving counting inside a workgroup, shared by the device pruner and the
// device packer.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace twg {

constexpr int SCAN_T = 1024;                    // threads of the workgroups that count
constexpr int SCAN_WAVES = SCAN_T / 64;

// Number of lanes with `v` set in front of this thread, over the workgroup's SCAN_T threads in
// order; *total: over all of them.  `part` is SCAN_WAVES ints of LDS; the caller puts a barrier
// between two uses of the same array.
__device__ __forceinline__ int count_before(bool v, int* part, int* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const unsigned long long b = __ballot(v);
  if (lane == 0) part[wave] = __popcll(b);
  __syncthreads();
  int before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < SCAN_WAVES; ++w) {
    const int n = part[w];
    before += w < wave ? n : 0;
    all += n;
  }
  *total = all;
  return before + __popcll(b & ((1ull << lane) - 1ull));
}

}  // namespace twg
