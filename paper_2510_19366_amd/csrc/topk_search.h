// The search of the top-k kernel for the border between a token's picks and the rest.  Integer keys
// only, the same in every lane; plain C++, so that it can be run on the host as well.
#pragma once
#include <stdint.h>

#include "host_device.h"

namespace mp {

MP_HD int float_bits(float f) { return __builtin_bit_cast(int, f); }
MP_HD float bits_float(int b) { return __builtin_bit_cast(float, b); }

// Keys: key(f) = bits ^ ((bits >> 31) & 0x7fffffff) orders like f for
// every non-NaN binary32 once -0.0 has been replaced by +0.0 (the two compare equal, and equal
// logits go to the lower id).  INT_MIN and INT_MAX are the keys of no logit (two NaNs could be): the one
// marks absent elements, the other is behind every key.
MP_HD int ordered_bits(int b) { return b ^ ((b >> 31) & 0x7fffffff); }
MP_HD int topk_key(float f) {
  int b = float_bits(f);
  b = b == INT32_MIN ? 0 : b;  // -0.0 -> +0.0
  b = ordered_bits(b);
  b = b < INT32_MIN + 1 ? INT32_MIN + 1 : b;
  return b > INT32_MAX - 1 ? INT32_MAX - 1 : b;
}
MP_HD float topk_unkey(int k) { return bits_float(ordered_bits(k)); }

// picks: all keys > thr and the first `rem` keys == thr in id order
struct TopkCut {
  int thr, rem;
};
constexpr int TOPK_VALUE_STEPS = 16;

// at_least(key): number of keys >= key.  at_least(lo) >= k > at_least(hi).  A threshold with exactly k
// keys above it ends the search; with equal keys at the border there is none and lo ends as the border key.
// uniform(m): m, into a scalar register.  Any m with lo < m < hi will do, also one that is no logit's key.
// Thresholds are taken midway between the logits: few steps, because the gaps between neighbouring order
// statistics are wide compared to the range.  First, though, an end more than 2^8 times the other (a
// mask of the lowest finite value, an infinity, an absent element), which midpoints would only halve, 128
// steps from the lowest value to 1, is cut off: between ends of different sign at minus half the
// smaller one, between ends of one sign at the mean of their bit patterns, about the geometric mean.
// And from TOPK_VALUE_STEPS steps on thresholds are taken midway between the keys, 32 steps at most: many
// logits equal to zero at the border would otherwise take a step per power of two.
// 16 384 x 128, half of the logits masked, 8 picks: 15.5 us, midpoints alone 138.
template <class Uniform, class Count>
MP_HD TopkCut topk_cut(int lo, int hi, int k, Uniform&& uniform, Count&& at_least) {
  int above = 0;  // keys >= hi
  auto found = [&](int m) {
    const int c = at_least(m);
    if (c > k) {
      lo = m;
    } else {
      hi = m;
      above = c;
    }
    return c == k;  // the picks are the keys >= hi
  };
  for (;;) {
    const int a = float_bits(topk_unkey(lo)), b = float_bits(topk_unkey(hi));
    const uint32_t ma = (uint32_t)a & 0x7fffffffu, mb = (uint32_t)b & 0x7fffffffu;
    if ((ma > mb ? ma - mb : mb - ma) <= (8u << 23)) break;
    const int m = uniform(ordered_bits((lo ^ hi) < 0 ? float_bits(-0.5f * bits_float(ma > mb ? b : a))
                                                     : (a & INT32_MIN) | (int)((ma + mb) >> 1)));
    if (m <= lo || m >= hi) break;
    if (found(m)) return TopkCut{hi - 1, 0};
  }
  for (int step = 0; (uint32_t)hi - (uint32_t)lo > 1u; ++step) {
    int m = uniform(ordered_bits(float_bits(0.5f * topk_unkey(lo) + 0.5f * topk_unkey(hi))));
    if (m <= lo || m >= hi || step >= TOPK_VALUE_STEPS) m = (int)((uint32_t)lo + (((uint32_t)hi - (uint32_t)lo) >> 1));
    if (found(m)) return TopkCut{hi - 1, 0};
  }
  return TopkCut{lo, k - above};
}

}  // namespace mp
