// quotient(w, divisor_magic(d)) and quotient(w, divisor_of(d, end)) against w / d: every small pair, and around multiples of d up to
// the limit of the range.
#include <cstdio>
#include <initializer_list>

#include "divide.h"

using kvp::divisor_magic;
using kvp::divisor_of;
using kvp::quotient;

static bool right(unsigned w, unsigned d) {
  if (quotient(w, divisor_magic(d)) == w / d) return true;
  std::printf("%u / %u: %u\n", w, d, quotient(w, divisor_magic(d)));
  return false;
}

// with the divisor for dividends up to w, and up to the largest
static bool right_anywhere(unsigned w, unsigned d) {
  for (unsigned end : {w + 1, 1u << 31})
    if (quotient(w, divisor_of(d, end)) != w / d) {
      std::printf("%u / %u below %u: %u\n", w, d, end, quotient(w, divisor_of(d, end)));
      return false;
    }
  return true;
}

int main() {
  for (unsigned d = 1; d <= 512; ++d)
    for (unsigned w = 0; w <= 4096; ++w)
      if (!right(w, d) || !right_anywhere(w, d)) return 1;
  for (unsigned d = 1; d <= 46340; d = d < 300 ? d + 1 : d + 1 + d / 7) {
    const unsigned last = ((1u << 31) - 1) / d;                  // the largest w of the range
    for (unsigned k = 1; k <= 2000; ++k) {
      const unsigned w = (unsigned)((unsigned long long)last * k / 2000), at = w / d * d;
      if (!right(w, d) || !right(at, d) || (at > 0 && !right(at - 1, d))) return 1;
    }
  }
  for (unsigned d = 1; d < (1u << 31); d = d < 70000 ? d + 1 + d / 300 : d + 1 + d / 7) {
    const unsigned last = (1u << 31) - 1;
    for (unsigned k = 1; k <= 200; ++k) {
      const unsigned w = (unsigned)((unsigned long long)last * k / 200), at = w / d * d;
      if (!right_anywhere(w, d) || !right_anywhere(at, d) || (at > 0 && !right_anywhere(at - 1, d))) return 1;
    }
  }
  // KV head of the last query head of a launch
  for (unsigned heads_per_kv : {46341u, 46410u, 100000u, 1u << 20})
    for (unsigned kv_heads : {1u, 2u, 1000u})
      if (!right_anywhere(heads_per_kv * kv_heads - 1, heads_per_kv)) return 1;
  if (!right_anywhere(2 * 32950 - 1, 32950)) return 1;
  if (!right_anywhere((1u << 31) - 1, (1u << 31) - 1) || !right_anywhere((1u << 31) - 2, (1u << 31) - 1)) return 1;
  return 0;
}
