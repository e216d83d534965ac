// The first digit of the selection's keys, as the pooling kernel counts it (select.hip): plain integer arithmetic.
#pragma once

#include <stdint.h>

namespace speckv {

// Scores are sums of probabilities (or their means, or maxima): none negative, none above the 4096 rows of a group, most within a
// few powers of two of each other, but the ones that a peaked softmax leaves far below its peak may be as small as numbers get.
// 2048 digits cover all of it, in the order of the keys (ordered_key: positive numbers are the keys from 2^31 on):
//   0                  keys below zero's
//   1 .. 348           0 up to 2^-40 by the 11 leading bits of the key (sign, exponent, 2 bits of mantissa)
//   349 .. 2044        2^-40 up to 2^13 by 14 leading bits (5 bits of mantissa)
//   2045               2^13 and above, infinity, NaN
// With 2 bits of mantissa everywhere a quarter of a row of scores within a factor of four shares the threshold's digit; with 5 bits
// everywhere there are digits for 64 powers of two only, and rows whose threshold lies outside them had to be counted again: one
// query row of logits with a standard deviation of 40, calls with 2 bits everywhere / 5 bits down to 2^-51 / these digits: 8 rows of
// 128K keys 111.2 / 141.5 / 75.9 us, 2 rows of 200K 81.6 / 154.0 / 53.8, 256 rows of 128K 2231 / 2276 / 2223.  Pooling and selection
// of 256 rows of 128K ordinary scores: one query row 105 + 54 / 118 + 46 / 119 + 47 us; 512 rows 174 + 64 / 131 + 58 / 131 + 59, but
// with heavy hitters among the keys 122 + 50 / 147 + 47 / 150 + 46 (a tile's counters then have more entries to add to the row's).
constexpr uint32_t kFineKey = 0x80000000u | ((127u - 40u) << 23), kTopKey = 0x80000000u | ((127u + 13u) << 23);
constexpr int kCoarseBase = (int)(0x80000000u >> 21) - 1;
constexpr int kFineDigit = (int)(kFineKey >> 21) - kCoarseBase;
constexpr int kFineBase = (int)(kFineKey >> 18) - kFineDigit;
constexpr int kTopDigit = (int)(kTopKey >> 18) - kFineBase;
static_assert(kFineDigit == 349 && kTopDigit == 2045, "the digits above");

__host__ __device__ inline int first_digit_of(uint32_t key) {
  // below kFineKey the coarse digit is the larger of the two, from there on the fine one
  const int coarse = (int)(key >> 21) - kCoarseBase, fine = (int)(key >> 18) - kFineBase;
  const int top = fine < kTopDigit ? fine : kTopDigit, low = coarse > 0 ? coarse : 0;
  return low > top ? low : top;
}

// What digit D says of the keys it stands for: all but their last `open` bits, which are zero in the result.  open = 32: nothing.
__host__ __device__ inline uint32_t key_prefix_of(uint32_t D, int *open) {
  if (D - 1u >= (uint32_t)kTopDigit - 1u) { *open = 32; return 0u; }
  if (D < (uint32_t)kFineDigit) { *open = 21; return (D + (uint32_t)kCoarseBase) << 21; }
  *open = 18;
  return (D + (uint32_t)kFineBase) << 18;
}

}  // namespace speckv
