// Scores by the keys alone (Sec. 3.2, "Query-Agnostic Eviction") of a KV head whose keys a workgroup of 512 threads can hold in
// its registers: it reads them once, adds them up to the anchor and takes every key's cosine with it.
//
// Bound by the vector work of one CU (some 50 instructions for 16 bytes of a key), 6 to 7 us at 768 keys of d 128; so
// the split-key attention launch has workgroups that do it beside the attention (attention_split.hip), and the
// compaction launch does it itself only behind the attention kernel whose workgroups fill the chip.
#pragma once
#include <type_traits>

#include "kvp_internal.h"
#include "lane_tools.h"

namespace kvp {
namespace {

constexpr int kKeyScoreThreads = 512;

// k_old [c][D], k_add [n_cand - c][n_kv_heads][D]: the head's keys; lds: D floats for each of the eight waves and for the anchor;
// scores[p] of candidate p, in LDS or in memory
template <int D>
__device__ __forceinline__ void score_head_by_keys(const u16* k_old, const u16* k_add, int n_kv_heads, int c, int n_cand, float* lds,
                                                   float* scores) {
  constexpr int kPieces = D / 8, kRows = kKeyScoreThreads / kPieces, kWaves = kKeyScoreThreads / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int piece = tid % kPieces, row0 = tid / kPieces;
  k_old += 8 * piece;
  k_add += 8 * piece;
  float* const s_part = lds;                           // [kWaves][D], then the anchor
  float* const s_mu = s_part + kWaves * D;
  auto score_keys = [&](auto rows) __attribute__((always_inline)) {
    constexpr int kN = decltype(rows)::value;
    typedef unsigned Piece __attribute__((ext_vector_type(4)));
    Piece w[kN];
#pragma unroll
    for (int i = 0; i < kN; ++i) {
      const int p = min(row0 + i * kRows, n_cand - 1);
      w[i] = *reinterpret_cast<const Piece*>(row_of_two<unsigned long long>(k_old, 2 * D, k_add, 2 * D * (unsigned)n_kv_heads, p, c));
      if (i % 4 == 3) __builtin_amdgcn_sched_barrier(0);       // (or the addresses of all rows are worked out first, in registers)
    }
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < kN; ++i) {
      if (row0 + i * kRows >= n_cand) w[i] = Piece{0u, 0u, 0u, 0u};
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        acc[2 * k] += bf16_lo(w[i][k]);
        acc[2 * k + 1] += bf16_hi(w[i][k]);
      }
      asm volatile("" : "+v"(w[i]));                   // or the unpacked channels stay in registers until the second pass
    }
    sum_rows<kPieces, 8>(acc);                         // lanes 16 r ..: channels 2 r, 2 r + 1 of the piece
    if (lane % 16 < kPieces)
      *reinterpret_cast<float2*>(&s_part[wave * D + 8 * piece + 2 * (lane / 16)]) = make_float2(acc[0], acc[1]);
    __syncthreads();
    if (tid < D) {
      float t = 0.f;
#pragma unroll
      for (int w2 = 0; w2 < kWaves; ++w2) t += s_part[w2 * D + tid];
      s_mu[tid] = t / (float)n_cand;
    }
    __syncthreads();
    float mu[8], mu2 = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) { mu[e] = s_mu[8 * piece + e]; mu2 = __builtin_fmaf(mu[e], mu[e], mu2); }
    mu2 = row_sum<kPieces>(mu2);
    // every lane of a row has its sums; lane i % kPieces keeps those of the i-th row and takes its cosine
    constexpr int kMine = (kN + kPieces - 1) / kPieces;
    float my_dot[kMine], my_k2[kMine];
#pragma unroll
    for (int i = 0; i < kN; ++i) {
      float dot = 0.f, k2 = 0.f;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float x = bf16_lo(w[i][k]), y = bf16_hi(w[i][k]);
        dot = __builtin_fmaf(x, mu[2 * k], dot); dot = __builtin_fmaf(y, mu[2 * k + 1], dot);
        k2 = __builtin_fmaf(x, x, k2); k2 = __builtin_fmaf(y, y, k2);
      }
      dot = row_sum<kPieces>(dot);
      k2 = row_sum<kPieces>(k2);
      my_dot[i / kPieces] = i % kPieces == 0 || piece == i % kPieces ? dot : my_dot[i / kPieces];
      my_k2[i / kPieces] = i % kPieces == 0 || piece == i % kPieces ? k2 : my_k2[i / kPieces];
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int u = 0; u < kMine; ++u) {
      const int i = u * kPieces + piece, p = row0 + i * kRows;
      if (i < kN && p < n_cand) scores[p] = -my_dot[u] / (sqrtf(my_k2[u]) * sqrtf(mu2));
    }
  };
  const int passes = (n_cand + kRows - 1) / kRows;
  constexpr int kMost = kKeydiffRowsPerThread;
  if (passes <= kMost / 4) score_keys(std::integral_constant<int, kMost / 4>{});
  else if (passes <= kMost / 2) score_keys(std::integral_constant<int, kMost / 2>{});
  else if (passes <= 3 * kMost / 4) score_keys(std::integral_constant<int, 3 * kMost / 4>{});
  else score_keys(std::integral_constant<int, kMost>{});
}

}  // namespace
}  // namespace kvp
