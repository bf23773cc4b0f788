// morton.h -- Morton key of a position: 21-bit cells per axis of the cubic box,
// x > y > z interleaved.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace sfmm {

__device__ __forceinline__ uint64_t spread3(uint64_t v) {
  v &= 0x1fffffull;
  v = (v | (v << 32)) & 0x1f00000000ffffull;
  v = (v | (v << 16)) & 0x1f0000ff0000ffull;
  v = (v | (v << 8)) & 0x100f00f00f00f00full;
  v = (v | (v << 4)) & 0x10c30c30c30c30c3ull;
  v = (v | (v << 2)) & 0x1249249249249249ull;
  return v;
}

// box: min corner, cube extent, 2^21 / extent (0 if flat)
__device__ __forceinline__ uint64_t morton(const double* p, const double* box) {
  uint64_t c[3] = {0, 0, 0};
  if (box[3] > 0.0) {
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const double f = floor((p[d] - box[d]) * box[4]);
      c[d] = f > 2097151.0 ? 2097151ull : (uint64_t)f;
    }
  }
  return (spread3(c[0]) << 2) | (spread3(c[1]) << 1) | spread3(c[2]);
}

}  // namespace sfmm
