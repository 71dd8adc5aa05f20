// Internal: grids of more workgroups than one dimension takes (plain arithmetic, also built without HIP).
#pragma once
#include <stdint.h>

namespace twg {

// A launch may have at most 2^32 - 1 threads in x.  n workgroups as x * y, y = 1 while they fit; a workgroup's number is
// blockIdx.y * gridDim.x + blockIdx.x, and those past the last one have nothing to do.
struct Grid2 {
  uint32_t x, y;
};
constexpr Grid2 grid_of(uint64_t n, uint32_t threads) {
  const uint64_t most = 0xffffffffull / threads;
  return n <= most ? Grid2{(uint32_t)n, 1u} : Grid2{(uint32_t)most, (uint32_t)((n + most - 1) / most)};
}

}  // namespace twg
