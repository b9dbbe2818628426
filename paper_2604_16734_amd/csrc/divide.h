// Division by a number that the host knows, as one multiplication.  An integer division is some forty instructions on this
// GPU, and the kernels would make two or three of them on the way to their first load.  No device code: the host
// tests run it, too.
#pragma once

#include "key_range.h"

namespace kvp {

// w / d = quotient(w, divisor_magic(d)) for d >= 1, w * d < 2^31: the magic number is at most one above 2^31 / d, which
// moves the quotient by less than w / 2^31 < 1 / d.
KVP_HOST_DEVICE unsigned divisor_magic(unsigned d) { return (unsigned)(((1ull << 31) + d - 1) / d); }
KVP_HOST_DEVICE unsigned quotient(unsigned w, unsigned magic) { return (unsigned)(((unsigned long long)(2u * w) * magic) >> 32); }

}  // namespace kvp
