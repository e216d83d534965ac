// The first digit of the selection's keys, as the pooling kernel counts it (select.hip): plain integer arithmetic.
#pragma once

#include <stdint.h>

namespace speckv {

// Scores are sums of probabilities (or their means, or maxima): none negative, most within a few powers of two of each other, but
// the ones that a peaked softmax leaves far below its peak may be as small as numbers get, and normalisers from the caller may make
// them any size.  2048 digits cover all of it, in the order of the keys (ordered_key: positive numbers are the keys from 2^31 on):
//   0                 keys below zero's
//   1 .. 392          0 up to 2^-29 by the 11 leading bits of the key (sign, exponent, 2 bits of mantissa)
//   393 .. 1544       2^-29 up to 2^7 by 14 leading bits (5 bits of mantissa)
//   1545 .. 2032      2^7 and above, infinity, NaN by 11 leading bits
// With 2 bits of mantissa everywhere a quarter of a row of scores within a factor of four shares the threshold's digit; with 5 bits
// everywhere there are digits for 64 powers of two only, and rows whose threshold lies outside them had to be counted again: one
// query row of logits with a standard deviation of 40, calls with 2 bits everywhere / 5 bits from 2^-51 to 2^13 / these digits: 8 rows
// of 128K keys 111.2 / 141.5 / 75.9 us, 2 rows of 200K 81.6 / 154.0 / 53.8, 256 rows of 128K 2231 / 2276 / 2223; selection kernel of 16
// rows of 60K whose scores overflow 92.0 / 118.3 / 87.  Pooling and selection
// of 256 rows of 128K ordinary scores: one query row 105 + 54 / 118 + 46 / 119 + 47 us; 512 rows 174 + 64 / 131 + 58 / 131 + 59, but
// with heavy hitters among the keys 122 + 50 / 147 + 47 / 150 + 46 (a tile's counters then have more entries to add to the row's).
constexpr uint32_t kFineKey = 0x80000000u | ((127u - 29u) << 23), kFineEnd = 0x80000000u | ((127u + 7u) << 23);
constexpr int kCoarseBase = (int)(0x80000000u >> 21) - 1;
constexpr int kFineDigit = (int)(kFineKey >> 21) - kCoarseBase;                       // first of the finer digits
constexpr int kFineDigits = (int)((kFineEnd - kFineKey) >> 18);
constexpr int kExtra = kFineDigits - (int)((kFineEnd - kFineKey) >> 21);              // digits they are more than coarse ones would be
constexpr int kLastDigit = (int)(0xffffffffu >> 21) - kCoarseBase + kExtra;
static_assert(kFineDigit == 393 && kFineDigits == 1152 && kLastDigit == 2032, "the digits above");

__host__ __device__ inline int first_digit_of(uint32_t key) {
  const uint32_t below = key < kFineEnd ? key : kFineEnd, inside = (below > kFineKey ? below : kFineKey) - kFineKey;
  const int coarse = (int)(key >> 21) - kCoarseBase;
  return (coarse > 0 ? coarse : 0) + (int)((inside >> 18) - (inside >> 21));
}

// What digit D says of the keys it stands for: all but their last `open` bits, which are zero in the result.  open = 32: nothing.
__host__ __device__ inline uint32_t key_prefix_of(uint32_t D, int *open) {
  if (D - 1u >= (uint32_t)kLastDigit) { *open = 32; return 0u; }
  if (D - (uint32_t)kFineDigit < (uint32_t)kFineDigits) { *open = 18; return kFineKey + ((D - (uint32_t)kFineDigit) << 18); }
  *open = 21;
  return (D - (D < (uint32_t)kFineDigit ? 0u : (uint32_t)kExtra) + (uint32_t)kCoarseBase) << 21;
}

}  // namespace speckv
