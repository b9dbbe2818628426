// The plain append of a block to a cache that is not full (Alg. 1 line 7 without lines 8-11): token i goes
// to slot c + i.  A row pair (the K row and the V row of one slot) is carried by 2 D / 8 lanes,
// 16 bytes each: 32 lanes at head dimension 128 (two pairs per wave), 16 at 64 (four pairs per wave).
// A launch covers a group of layers: grid (row blocks, KV heads, layers).  Also the fill of a new cache.
#include "kvp_internal.h"

namespace kvp {
namespace {

constexpr int kThreads = kCompactThreads;

template <int D>
__global__ void __launch_bounds__(kThreads)
append_kernel(const CompactArgs a) {
  constexpr int kPerRow = D / 8;                       // 16-byte pieces of a row
  constexpr int kPerPair = 2 * kPerRow;                // K row then V row
  constexpr int kPairsPerBlock = kThreads / kPerPair;
  const int hk = blockIdx.y, li = blockIdx.z;
  const int sub = threadIdx.x % kPerPair;
  const bool is_v = sub >= kPerRow;
  const int piece = sub % kPerRow;
  const u16* const k_new = a.layer[li].k_new;
  const u16* const v_new = a.layer[li].v_new;
  const u16* const src = (is_v ? v_new : k_new) + (size_t)hk * D + 8 * piece;
  u16* const dst = (is_v ? a.v_cache : a.k_cache) + (long long)li * a.g.kv_stride + ((size_t)hk * a.budget + a.c) * D + 8 * piece;
  const size_t m = (size_t)((long long)li * a.g.meta_stride) + (size_t)hk * a.budget + a.c;
  // The grid is capped (a launch for sixteen layers would otherwise be mostly workgroups of a few rows,
  // and starting those costs more than the rows take): a workgroup walks the rows with its stride.
  for (int i = blockIdx.x * kPairsPerBlock + threadIdx.x / kPerPair; i < a.n; i += gridDim.x * kPairsPerBlock) {
    *reinterpret_cast<uint4*>(dst + (size_t)i * D) = *reinterpret_cast<const uint4*>(src + (size_t)i * a.n_kv_heads * D);
    if (sub == 0) {
      a.token_idx[m + i] = a.t0 + i;
      a.weight[m + i] = 1.f;
    }
  }
}

struct InitArgs {
  Seg segs[KVP_MAX_SEGMENTS];
  Seg* dst;
  unsigned long long* totals;
  int n_segs;
};

__global__ void fill_kernel(int32_t* token_idx, float* weight, size_t n, InitArgs ia) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) {
    token_idx[i] = -1;
    weight[i] = 0.f;
  }
  if (i < (size_t)ia.n_segs) ia.dst[i] = ia.segs[i];
  if (i < (size_t)KVP_T_COUNT) ia.totals[i] = 0ull;
}

}  // namespace

hipError_t launch_move(const CompactArgs& a, hipStream_t s) {
  // row blocks per (KV head, layer): what the rows could need, but not more than keeps the whole
  // launch at about kCompactTargetWorkgroups workgroups
  const int pairs = a.n_kv_heads * a.g.n_layers;
  const int rows = rows_per_compact_block(a.head_dim), need = (a.n + rows - 1) / rows;
  const int cap = (kCompactTargetWorkgroups + pairs - 1) / pairs;
  const dim3 grid(need < cap ? need : cap, a.n_kv_heads, a.g.n_layers);
  if (a.head_dim == 128) hipLaunchKernelGGL(append_kernel<128>, grid, dim3(kThreads), 0, s, a);
  else hipLaunchKernelGGL(append_kernel<64>, grid, dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_init(int32_t* token_idx, float* weight, size_t n_slots, const Seg* host_segs,
                       int n_segs, Seg* dev_segs, unsigned long long* totals, hipStream_t s) {
  InitArgs ia;
  for (int i = 0; i < KVP_MAX_SEGMENTS; ++i) ia.segs[i] = i < n_segs ? host_segs[i] : Seg{0, 0, 0, 0, 0, 0, 0};
  ia.dst = dev_segs;
  ia.totals = totals;
  ia.n_segs = n_segs;
  size_t n = n_slots > (size_t)KVP_MAX_SEGMENTS ? n_slots : (size_t)KVP_MAX_SEGMENTS;
  const unsigned blocks = (unsigned)((n + 255) / 256);
  hipLaunchKernelGGL(fill_kernel, dim3(blocks), dim3(256), 0, s, token_idx, weight, n_slots, ia);
  return hipGetLastError();
}

}  // namespace kvp
