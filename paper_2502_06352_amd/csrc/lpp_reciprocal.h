// Division by numbers that the host knows, as the upper half of a product.  On the host as well:
// tests/test_reciprocal.py tries its range there.
#ifndef LPP_RECIPROCAL_H_
#define LPP_RECIPROCAL_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

// ceil(2^32 / d) as the two below take it (0: d = 1, 1: divide); n_max: the largest n (div_rc: kept below 2^32 / d by its callers)
inline uint32_t reciprocal(uint32_t d, uint64_t n_max = 0) {
  return d <= 1 ? 0u : (n_max * d >= 0x100000000ull ? 1u : (uint32_t)((0x100000000ull + d - 1) / d));
}

// n / d for wave-uniform operands through the host's reciprocal: scalar multiplies, no division
__host__ __device__ inline uint32_t div_rc(uint32_t n, uint32_t d, uint32_t rc) {
  const uint32_t q = (uint32_t)(((uint64_t)n * rc) >> 32);   // (rc = 0 for d = 1)
  return rc == 0 ? n : q;
}
// The same, rc = 1 where n d can reach 2^32: divided.
__host__ __device__ inline uint32_t div_or_rc(uint32_t n, uint32_t d, uint32_t rc) {
  return rc == 1 ? n / d : div_rc(n, d, rc);
}

// Layers of `most`, of so many units each, that one launch takes: unit / units by div_rc needs units * units * layers below 2^32.
inline int32_t layers_per_launch(int64_t units, int32_t most) {
  while (most > 1 && (uint64_t)units * (uint64_t)units >= 0x100000000ull / (uint32_t)most) --most;
  return most;
}

#endif  // LPP_RECIPROCAL_H_
