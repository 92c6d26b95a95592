// Leaf keys of the forest: tree id in the high bits, then the Morton code of
// the anchor scaled to level kKeyLevel with x in the lowest bit, so that key
// order is "tree by tree, Morton order inside a tree" (block n = leaf n).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace f4 {

// The low 16 bits of x spread to every third (every second) bit: at each step
// the upper half of every group of bits moves up by the width that is missing.
__host__ __device__ inline uint64_t spread3(uint64_t x) {
  x = (x | x << 16) & 0x0000FF0000FFull;
  x = (x | x << 8) & 0x00F00F00F00Full;
  x = (x | x << 4) & 0x0C30C30C30C3ull;
  return (x | x << 2) & 0x249249249249ull;
}
__host__ __device__ inline uint64_t spread2(uint64_t x) {
  x = (x | x << 8) & 0x00FF00FFull;
  x = (x | x << 4) & 0x0F0F0F0Full;
  x = (x | x << 2) & 0x33333333ull;
  return (x | x << 1) & 0x55555555ull;
}

__host__ __device__ inline uint64_t leaf_key(int ndim, const int32_t nt[3], int32_t level,
                                             const int32_t g[3]) {
  constexpr int KL = 16;
  int32_t t[3] = {0, 0, 0};
  uint32_t a[3] = {0, 0, 0};
  for (int d = 0; d < ndim; d++) {
    t[d] = g[d] >> level;
    a[d] = (uint32_t)(g[d] - (t[d] << level)) << (KL - level);
  }
  const uint64_t tid = (uint64_t)t[0] + (uint64_t)nt[0] * ((uint64_t)t[1] + (uint64_t)nt[1] * (uint64_t)t[2]);
  const uint64_t m = ndim == 3 ? spread3(a[0]) | spread3(a[1]) << 1 | spread3(a[2]) << 2
                               : spread2(a[0]) | spread2(a[1]) << 1;
  return (tid << (ndim * KL)) | m;
}

}  // namespace f4
