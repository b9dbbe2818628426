// Vector types and small device helpers shared by the MFMA kernels of attention.
#pragma once
#include "kvp_internal.h"
#include "lane_tools.h"

namespace kvp {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef short i16x4 __attribute__((ext_vector_type(4)));

namespace {

// value of the same row held by the other half of the wave (lane ^ 32)
__device__ __forceinline__ float max_with_other_half(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_with_other_half(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ __forceinline__ bf16x8 lds_read_b128(const u16* p) {
  return *reinterpret_cast<const bf16x8*>(p);
}
// two transposing reads: keys k .. k+3 and k+8 .. k+11 of this lane's channel
__device__ __forceinline__ bf16x8 lds_read_vt(const u16* p, int eight_rows) {
  const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((i16x4 __attribute__((address_space(3)))*)(p));
  const i16x4 hi =
      __builtin_amdgcn_ds_read_tr16_b64_v4i16((i16x4 __attribute__((address_space(3)))*)(p + eight_rows));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// A row-major V tile in LDS holds the 16-byte chunk ch of row r at position ch ^ v_swizzle(r).  Rows are
// read four at a time by each half of a wave (transposing 8-byte reads, 64 bytes of each row): the
// swizzle sends those four 64-byte pieces to four different quarters of the 64 banks (D = 128: a
// row spans all banks; D = 64: rows r and r + 2 share their banks).
template <int D>
__device__ __forceinline__ int v_swizzle(int row) {
  return 4 * ((row % 4) >> (D == 64 ? 1 : 0));
}

}  // namespace
}  // namespace kvp
