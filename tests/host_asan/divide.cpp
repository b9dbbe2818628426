// quotient(w, divisor_magic(d)) against w / d: every small pair, and around every multiple of d up to the limit of the range.
#include <cstdio>

#include "divide.h"

using kvp::divisor_magic;
using kvp::quotient;

static bool right(unsigned w, unsigned d) {
  if (quotient(w, divisor_magic(d)) == w / d) return true;
  std::printf("%u / %u: %u\n", w, d, quotient(w, divisor_magic(d)));
  return false;
}

int main() {
  for (unsigned d = 1; d <= 512; ++d)
    for (unsigned w = 0; w <= 4096; ++w)
      if (!right(w, d)) return 1;
  for (unsigned d = 1; d <= 46340; d = d < 300 ? d + 1 : d + 1 + d / 7) {
    const unsigned last = ((1u << 31) - 1) / d;                  // the largest w of the range
    for (unsigned k = 1; k <= 2000; ++k) {
      const unsigned w = (unsigned)((unsigned long long)last * k / 2000), at = w / d * d;
      if (!right(w, d) || !right(at, d) || (at > 0 && !right(at - 1, d))) return 1;
    }
  }
  return 0;
}
