// The search for the budget-th largest selection key: the range of keys that still holds it, cut into
// at most 2^kBits bins of equal width.  The selection counts its keys by bin, enters the bin with the
// wanted key and, if that holds too many, divides it in turn.  No device code: the host tests run it, too.
#pragma once

#if defined(__HIPCC__)
#include <hip/hip_runtime.h>
#define KVP_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define KVP_HOST_DEVICE inline
#endif

namespace kvp {

constexpr int kSelectBinBits = 11;
constexpr int kSelectBins = 1 << kSelectBinBits;   // histogram bins of the selection
constexpr int kSelectFewBinBits = 9;               // ... of one with 512 threads (kvp_internal.h: SelectPlan::threads)

template <int kBits>
struct KeyRangeOf {
  unsigned long long lo;     // the first key of the range
  int shift;                 // a bin spans 1 << shift keys
  unsigned bins;             // the range ends with this many bins: keys beyond are larger ones, counted before

  // every key whose high word lies in [hi_min, hi_max]
  static KVP_HOST_DEVICE KeyRangeOf over(unsigned hi_min, unsigned hi_max) {
    const unsigned long long lo = (unsigned long long)hi_min << 32;
    const unsigned long long span = (((unsigned long long)hi_max << 32) | 0xFFFFFFFFull) - lo;
    return KeyRangeOf{lo, 64 - (int)__builtin_clzll(span) - kBits, 1u << kBits};   // 32 bits of span or more
  }
  KVP_HOST_DEVICE bool holds(unsigned long long key, unsigned& bin) const {
    const unsigned long long b = (key - lo) >> shift;
    bin = (unsigned)b;
    return key >= lo && b < (unsigned long long)bins;
  }
  // the range is one of its bins
  KVP_HOST_DEVICE void enter(unsigned bin) {
    lo += (unsigned long long)bin << shift;
    bins = 1u;
  }
  // A range of one bin, cut anew.  A bin of fewer keys than the histogram has bins has one bin for each of them and
  // no more: as many bins as the histogram has would reach into the range above.
  KVP_HOST_DEVICE void divide() {
    bins = 1u << (shift < kBits ? shift : kBits);
    shift = shift < kBits ? 0 : shift - kBits;
  }
};

}  // namespace kvp
