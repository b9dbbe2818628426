// bf16 values two to a register.  Sums and maxima across the lanes of a wave when kPieces = D / 8 neighbouring lanes hold a row of D channels in 16-byte
// pieces: on the DPP network and by lane swaps, never through LDS.
#pragma once
#include "kvp_internal.h"

namespace kvp {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

namespace {

__device__ __forceinline__ unsigned pack_bf16(float lo, float hi) {
  f32x2 v = {lo, hi};
  bf16x2 b = __builtin_convertvector(v, bf16x2);   // v_cvt_pk_bf16_f32, round to nearest even
  return __builtin_bit_cast(unsigned, b);
}
__device__ __forceinline__ float bf16_lo(unsigned x) { return __uint_as_float(x << 16); }
__device__ __forceinline__ float bf16_hi(unsigned x) { return __uint_as_float(x & 0xFFFF0000u); }
// c + lo(x) lo(y) + hi(x) hi(y) of bf16 pairs, in fp32
__device__ __forceinline__ float dot2(unsigned x, unsigned y, float c) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, x), __builtin_bit_cast(bf16x2, y), c, false);
}
__device__ __forceinline__ void unpack8(const uint4 w, float (&x)[8]) {
  x[0] = bf16_lo(w.x); x[1] = bf16_hi(w.x); x[2] = bf16_lo(w.y); x[3] = bf16_hi(w.y);
  x[4] = bf16_lo(w.z); x[5] = bf16_hi(w.z); x[6] = bf16_lo(w.w); x[7] = bf16_hi(w.w);
}

template <int kCtrl>
__device__ __forceinline__ float dpp_lane(float x) {
  return __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), kCtrl, 0xF, 0xF, false));
}
// sum over the kPieces (8 or 16) neighbouring lanes that hold a row, in all of them
template <int kPieces>
__device__ __forceinline__ float row_sum(float x) {
  x += dpp_lane<0xB1>(x);                             // lane ^ 1
  x += dpp_lane<0x4E>(x);                             // lane ^ 2
  x += dpp_lane<0x141>(x);                            // the other four of eight lanes
  if constexpr (kPieces == 16) x += dpp_lane<0x140>(x);   // the other eight of sixteen
  return x;
}
// The lane swaps exchange the upper half (16: the odd rows of sixteen lanes) of the first operand with the lower half
// (the even rows) of the second.
template <int kLanes>
__device__ __forceinline__ void swap_lanes(float& x, float& y) {
  const unsigned a = __float_as_uint(x), b = __float_as_uint(y);
  if constexpr (kLanes == 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    x = __uint_as_float(r[0]); y = __uint_as_float(r[1]);
  } else {
    const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    x = __uint_as_float(r[0]); y = __uint_as_float(r[1]);
  }
}
template <class Op>
__device__ __forceinline__ float over_rows(float x, Op op, bool eight_lanes) {    // over the rows of a wave, in all lanes
  if (eight_lanes) x = op(x, dpp_lane<0x128>(x));     // rows of eight lanes: the other one of the sixteen
  float y = x;
  swap_lanes<16>(x, y);
  x = op(x, y);
  y = x;
  swap_lanes<32>(x, y);
  return op(x, y);
}
struct FloatMax { __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); } };
struct FloatSum { __device__ __forceinline__ float operator()(float a, float b) const { return a + b; } };

// Sums of v[0 .. N - 1] over the rows of a wave; lanes 16 r .. 16 r + 15 (r = 0 .. 3) end up with those of
// v[r N / 4 .. (r + 1) N / 4 - 1], in v[0 .. N / 4 - 1].
template <int kPieces, int N>
__device__ __forceinline__ void sum_rows(float (&v)[N]) {
#pragma unroll
  for (int i = 0; i < N / 2; ++i) { swap_lanes<32>(v[i], v[i + N / 2]); v[i] += v[i + N / 2]; }
#pragma unroll
  for (int i = 0; i < N / 4; ++i) { swap_lanes<16>(v[i], v[i + N / 4]); v[i] += v[i + N / 4]; }
  if constexpr (kPieces == 8) {
#pragma unroll
    for (int i = 0; i < N / 4; ++i) v[i] += dpp_lane<0x128>(v[i]);
  }
}

}  // namespace
}  // namespace kvp
