// Division by a number that the host knows, as a multiplication.  An integer division is some forty instructions on this
// GPU, and the kernels would make two or three of them on the way to their first load.  No device code: the host
// tests run it, too.
#pragma once

#include "key_range.h"

namespace kvp {

// w / d = quotient(w, divisor_magic(d)) for d >= 1, w * d < 2^31: the magic number is at most one above 2^31 / d, which
// moves the quotient by less than w / 2^31 < 1 / d.
KVP_HOST_DEVICE unsigned divisor_magic(unsigned d) { return (unsigned)(((1ull << 31) + d - 1) / d); }
KVP_HOST_DEVICE unsigned quotient(unsigned w, unsigned magic) { return (unsigned)(((unsigned long long)(2u * w) * magic) >> 32); }

// The same for all w < end <= 2^31, 1 <= d <= 2^31: without a shift where the above will do, else with 2^shift >= d.  The magic
// number is then less than one above 2^(31 + shift) / d, which moves the quotient by less than w / 2^(31 + shift) < 1 / d; and
// with 2^shift < 2 d it has 32 bits.  (attention.hip, whose launches may have any number of heads: 46410 query heads of one KV
// head are out of the other's range.  The shift holds up the addresses of a workgroup's first loads; launches of 8 us,
// which are of few workgroups, became 0.3 to 0.6 % longer by it and do without.)
struct Divisor {
  unsigned magic, shift;
};
KVP_HOST_DEVICE Divisor divisor_of(unsigned d, unsigned end) {
  unsigned shift = 0;
  if ((unsigned long long)end * d > 1ull << 31)
    while ((1ull << shift) < d) ++shift;
  return Divisor{(unsigned)(((1ull << (31 + shift)) + d - 1) / d), shift};
}
KVP_HOST_DEVICE unsigned quotient(unsigned w, Divisor d) { return (unsigned)(((unsigned long long)(2u * w) * d.magic) >> 32) >> d.shift; }

}  // namespace kvp
