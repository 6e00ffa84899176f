// The value of a list word of the neighbour build, and how far apart two of them have to be before their
// order is that of the similarities.  On the host as well: tests/test_knn_list_value.py tries the bound there.
#ifndef LPP_KNN_LIST_H_
#define LPP_KNN_LIST_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

// d: a similarity less the row's threshold, not negative; a = qmax / range of d.  Rounded once by the product, and
// once more by the caller where d was an integer of more than 24 bits.
__host__ __device__ inline uint32_t list_value(float d, float a, uint32_t qmax) {
  const uint32_t v = (uint32_t)(d * a);
  return v < qmax ? v : qmax;
}

// What those two roundings, 2^-24 of the value each, come to between two values, in units of the value.
__host__ __device__ inline double list_rounding(uint32_t qmax) { return 4.0 / 16777216.0 * ((double)qmax + 1.0); }

// Values that differ by more than this belong to similarities that differ by more than 2 e: the difference of
// the exact products is at most 2 e a plus the roundings, and taking the floor adds less than one.  (e, range in
// the same units; 2.002 for the rounding of a itself.)  Limited to 2^30: beyond it everything is near.
__host__ __device__ inline int32_t list_margin(double e, double range, uint32_t qmax) {
  const double m = 2.002 * e * (double)qmax / range + list_rounding(qmax);
  return m < 1073741823.0 ? (int32_t)m + 1 : 1 << 30;                 // (also where m is NaN)
}

// Float64 sums of the D products of two pairs (a row with two codes), in any order, that differ by more than this: added
// in index order they have the same order.  Each of the four sums is off by at most D 2^-53 of the magnitudes added,
// which `reach`, the row's 1-norm times the largest magnitude of the codebook, bounds: 4 D 2^-53, and as much again in
// hand, of which 5 % are for the rounding of `reach` itself (its D float32 additions and a product).
__host__ __device__ inline double key_margin(float reach, int32_t D) { return 8.4 * 1.1102230246251565e-16 * D * (double)reach; }

#endif  // LPP_KNN_LIST_H_
