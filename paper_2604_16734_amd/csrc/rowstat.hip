// Row statistics (log2-domain log-sum-exp of every softmax row of Eq. 4) for a
// short list of proxy queries (Sec. 3.2) over all candidates of a KV head.
//
// The attention kernel gives these statistics as a by-product, but it spreads
// its work over query rows: a few dozen proxy queries would leave most of the
// chip idle while a handful of workgroups walk all the keys.  Here the keys are
// spread instead.  A workgroup takes 256 keys of one KV head, which its four
// waves keep in registers (64 each), and a share of the (query head, 32-row
// tile) items of the KV group; per item a wave computes S^T = K Q^T (a lane then
// holds one query row, its logits in registers), reduces them to (max, sum of
// exp2) per row, and the four pairs are folded through LDS into one partial per
// (head, row, key block).  A second, tiny kernel folds the
// partials of all key blocks, in a fixed order, into the statistic the scoring
// kernel reads.  Every candidate is visible to every proxy query (the prompt
// follows the visual tokens), so there is no mask beyond the end of the keys.
//
// Bound by the vector unit (maximum, difference, scale, exponential, sum: 22 cycles per logit and SIMD
// against 8 of the matrix pipe).  What it must avoid is fetching operands in operand layout, where
// neighbouring lanes read different rows: that runs at 16 bytes a clock, a quarter of a CU's path, and with
// every wave fetching every query tile by itself it was two thirds of the time.  Keys and queries
// therefore come through LDS in whole rows, the queries once per workgroup: 72 -> 48 us for 16 layers of 32/8
// heads, d 128, 64 queries over 3072 keys (without the fetch of the keys 36, without the matrix products 37, without the
// exponentials 44), 44 -> 28 us for 8 layers of 28/4 heads, 128 queries over 1536.  Products of the next item among the
// exponentials of this one, two waves per SIMD instead of four: the same times.
#include <type_traits>

#include "kvp_internal.h"
#include "mfma_tools.h"

namespace kvp {

namespace {

constexpr int kWaves = 4;
constexpr int kThreads = 64 * kWaves;
constexpr int kSub = 2;                        // 32-key subtiles per wave
constexpr int kWaveKeys = 32 * kSub;
constexpr int kBlockKeys = kWaves * kWaveKeys;
constexpr int kRing = 4;                       // query tiles in LDS: the pair in use and the pair in flight
constexpr int kStats = 4;                      // items whose statistics wait in LDS: the pair in work and the pair being folded
static_assert(kBlockKeys == kRowstatBlockKeys, "the host plans with this block size");

// grid (key blocks, KV heads x item splits, layers of the group).  An item is one 32-row tile of
// one query head of the KV group; a workgroup takes `items_per_wg` of them, in pairs.
template <int D>
__global__ void __launch_bounds__(kThreads, 4)
rowstat_kernel(const RowstatArgs a) {
  constexpr int kChunks = D / 8;                   // 16-byte chunks per row
  constexpr int kTile = 32 * D;
  constexpr int kRowsPerLoad = 64 / kChunks;       // rows one wave instruction brings in
  constexpr int kLoads = 32 / kRowsPerLoad;        // instructions for 32 rows
  __shared__ __align__(1024) u16 q_lds[kRing][kTile];        // (and, before the first of them, each wave's keys)
  auto& k_lds = q_lds;
  static_assert(kRing >= kWaves);
  __shared__ float s_m[kStats][kWaves][32], s_l[kStats][kWaves][32];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, g = lane >> 5;
  const int group = a.group;
  const int kb = blockIdx.x, li = blockIdx.z;
  have_arguments(a.layer[li].q, a.layer[li].k_new, a.k_cache, a.part_m, a.part_l, a.g.first_set, a.g.n_sets, a.g.set_stride, a.g.kv_stride,
                 a.n, a.c, a.n_keys, a.budget, a.item_splits, a.items_per_wg, a.splits_magic, a.tiles_magic, a.group);
  const int hk = (int)quotient(blockIdx.y, a.splits_magic), isplit = (int)blockIdx.y - hk * a.item_splits;
  const int n_rt = (a.n + 31) / 32;
  const int n_items = group * n_rt;
  const int item0 = isplit * a.items_per_wg, item1 = min(n_items, item0 + a.items_per_wg);
  if (item0 >= item1) return;
  const u16* const q_rows = a.layer[li].q;
  const u16* const k_new = a.layer[li].k_new;
  const u16* const k_cache = a.k_cache + (long long)li * a.g.kv_stride;
  float* const part_m = in_set_of(a.part_m, a.g, li);
  float* const part_l = in_set_of(a.part_l, a.g, li);
  const int c = a.c, n_cand = a.c + a.n_keys;
  const int key0 = kb * kBlockKeys + wave * kWaveKeys;
  const float sl2 = a.scale_log2;

  // global memory -> LDS, 16 bytes per lane, as inline assembly (the compiler would make every later LDS
  // read wait for a load it knows about); row r keeps its chunk ch at ch ^ (r % kChunks), so
  // that the fragment reads are free of bank conflicts
  auto load16 = [&](const u16* src, const u16* to) __attribute__((always_inline)) {
    const unsigned dst = __builtin_amdgcn_readfirstlane((unsigned)(size_t)(__attribute__((address_space(3))) const void*)to);
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(dst) : "m0", "memory");
  };
  const int ld_sub = lane / kChunks, ld_pos = lane % kChunks;
  // the query tile of item `i` (past the last one: that again), shared out among the waves
  auto issue_item = [&](int i) __attribute__((always_inline)) {
    const int item = min(i, item1 - 1);
    const int head = (int)quotient((unsigned)item, a.tiles_magic), h = hk * group + head, rt = item - head * n_rt;
#pragma unroll
    for (int j = 0; j < kLoads / kWaves; ++j) {
      const int first = kRowsPerLoad * (wave + kWaves * j);
      const int row = first + ld_sub;
      load16(q_rows + ((size_t)min(32 * rt + row, a.n - 1) * a.n_q_heads + h) * D + 8 * (ld_pos ^ (row % kChunks)),
             &q_lds[(i - item0) % kRing][first * D]);
    }
  };
  static_assert(kLoads % kWaves == 0, "every wave brings in as much of a query tile");
  int off[D / 16];             // fragment st of row l32: chunk 2 st + g
#pragma unroll
  for (int st = 0; st < D / 16; ++st) off[st] = l32 * D + 8 * ((2 * st + g) ^ (l32 % kChunks));

  // A operand: subtile t of this wave is keys key0 + 32 t + (0..31); lane holds K[key][16 s + 8 g .. + 7]
  bf16x8 kf[kSub][D / 16];
#pragma unroll
  for (int t = 0; t < kSub; ++t) {
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
      const int row = kRowsPerLoad * j + ld_sub;
      const int kv = min(key0 + 32 * t + row, n_cand - 1);
      const u16* src = kv < c ? k_cache + ((size_t)hk * a.budget + kv) * D : k_new + ((size_t)(kv - c) * a.n_kv_heads + hk) * D;
      load16(src + 8 * (ld_pos ^ (row % kChunks)), &k_lds[wave][kRowsPerLoad * j * D]);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
    for (int st = 0; st < D / 16; ++st) kf[t][st] = lds_read_b128(&k_lds[wave][off[st]]);
    // the strip is read before the next keys are on their way into it
#pragma unroll
    for (int st = 0; st < D / 16; ++st) asm volatile("" : "+v"(kf[t][st]));
  }
  __syncthreads();             // everybody has its keys
  issue_item(item0);
  issue_item(item0 + 1);

  // S^T of the query tile in ring buffer BUF, subtile t: rows = keys, columns = the 32 query rows
  auto logits = [&](int buf, f32x16 (&s)[kSub]) __attribute__((always_inline)) {
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int st = 0; st < D / 16; ++st) {
      const bf16x8 qf = lds_read_b128(&q_lds[buf][off[st]]);
#pragma unroll
      for (int t = 0; t < kSub; ++t) s[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[t][st], qf, st == 0 ? zero : s[t], 0, 0, 0);
    }
  };
  // (maximum, sum of exp2) of every row over this wave's keys, for item `i`.  `cut`: some of the keys lie past the end.
  auto statistics = [&](const f32x16 (&s_in)[kSub], int i, auto cut) __attribute__((always_inline)) {
    f32x16 s[kSub] = {s_in[0], s_in[1]};
    float mx[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll
    for (int t = 0; t < kSub; ++t) {
      // accumulator register r of lane group g is key 8 (r / 4) + 4 g + r % 4 of the subtile
      const int left = n_cand - (key0 + 32 * t) - 4 * g;      // keys of this lane's list that exist
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (decltype(cut)::value && 8 * (r >> 2) + (r & 3) >= left) s[t][r] = -INFINITY;
#pragma unroll
      for (int r = 0; r < 16; r += 2) mx[r / 2 % 4] = fmaxf(fmaxf(mx[r / 2 % 4], s[t][r]), s[t][r + 1]);
    }
    // lanes l and l + 32 hold the two halves of a row's keys
    const float m = max_with_other_half(fmaxf(fmaxf(mx[0], mx[1]), fmaxf(mx[2], mx[3])));
    const float m_use = decltype(cut)::value && m == -INFINITY ? 0.f : m;
    float l = 0.f;
#pragma unroll
    for (int t = 0; t < kSub; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) l += __builtin_amdgcn_exp2f((s[t][r] - m_use) * sl2);
    const float sum = sum_with_other_half(l);
    const int at = i - item0;
    s_m[at % kStats][wave][l32] = m;           // (both halves write the same)
    s_l[at % kStats][wave][l32] = sum;
  };
  // the four waves' pairs of the items `first`, `first + 1`
  auto fold = [&](int first) __attribute__((always_inline)) {
    const int row_of = tid & 31, item = first + (tid >> 5);
    if (first < item0 || tid >= 64 || item >= item1) return;
    const int at = (item - item0) % kStats;
    float mm = s_m[at][0][row_of];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) mm = fmaxf(mm, s_m[at][w][row_of]);       // finite: a block holds at least one key
    float ll = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) ll += s_l[at][w][row_of] * __builtin_amdgcn_exp2f((s_m[at][w][row_of] - mm) * sl2);
    const int head = (int)quotient((unsigned)item, a.tiles_magic), h = hk * group + head, row = 32 * (item - head * n_rt) + row_of;
    if (row < a.n) {
      const size_t to = ((size_t)kb * a.n_q_heads + h) * a.n + row;
      part_m[to] = mm;
      part_l[to] = ll;
    }
  };
  // One barrier per pair of items: this wave's share of the pair from item i on has landed and everybody is
  // through with the pair before: its buffers take the next pair, and its statistics are folded.
  auto publish = [&](int i) __attribute__((always_inline)) {
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    issue_item(i + 2);
    issue_item(i + 3);
    fold(i - 2);
  };
  auto all_items = [&](auto cut) __attribute__((always_inline)) {
    for (int i = item0; i < item1; ++i) {
      if ((i - item0) % 2 == 0) publish(i);
      f32x16 s[kSub];
      logits((i - item0) % kRing, s);
      statistics(s, i, cut);
    }
  };
  if (key0 + kWaveKeys <= n_cand) all_items(std::false_type{});
  else all_items(std::true_type{});
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  fold(item0 + (item1 - 1 - item0) / 2 * 2);
}

// lse2[h][row] from the partials of all key blocks, folded in block order; kFoldBatch of them are on their way together
constexpr int kFoldBatch = 16;
__global__ void __launch_bounds__(256)
rowstat_fold_kernel(const RowstatArgs a) {
  // grid (blocks of 256 rows, layers of the group)
  const int i = blockIdx.x * 256 + threadIdx.x, li = blockIdx.y;
  have_arguments(a.lse2, a.part_m, a.part_l, a.g.first_set, a.g.n_sets, a.g.set_stride, a.n, a.n_q_heads, a.n_kv_blocks, a.lse_stride,
                 a.rows_magic, a.scale_log2);
  const int rows = a.n_q_heads * a.n;
  if (i >= rows) return;
  const float* const part_m = in_set_of(a.part_m, a.g, li) + i;
  const float* const part_l = in_set_of(a.part_l, a.g, li) + i;
  // two passes over the partials, the maximum first; up to a batch of them stays in registers for the second
  float pm[kFoldBatch], pl[kFoldBatch], m = -INFINITY, l = 0.f;
  auto fetch = [&](int first) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < kFoldBatch; ++u) {
      // (past the end: the last one again, with weight 0; a load under a condition would be waited for on the spot)
      const size_t at = (size_t)min(first + u, a.n_kv_blocks - 1) * rows;
      pm[u] = part_m[at];
      pl[u] = part_l[at];
    }
  };
  for (int first = 0; first < a.n_kv_blocks; first += kFoldBatch) {
    fetch(first);
#pragma unroll
    for (int u = 0; u < kFoldBatch; ++u) m = fmaxf(m, pm[u]);
  }
  for (int first = 0; first < a.n_kv_blocks; first += kFoldBatch) {
    if (a.n_kv_blocks > kFoldBatch) fetch(first);
#pragma unroll
    for (int u = 0; u < kFoldBatch; ++u) {
      const float f = __builtin_amdgcn_exp2f((pm[u] - m) * a.scale_log2);
      l = __builtin_fmaf(pl[u], first + u < a.n_kv_blocks ? f : 0.f, l);
    }
  }
  const int h = (int)quotient((unsigned)i, a.rows_magic), row = i - h * a.n;    // (fewer than 8192 rows, n_obs 8192 at most)
  in_set_of(a.lse2, a.g, li)[(size_t)h * a.lse_stride + row] = m * a.scale_log2 + __builtin_log2f(l);
}

}  // namespace

hipError_t launch_rowstat(RowstatArgs a, int head_dim, hipStream_t s) {
  a.n_kv_blocks = rowstat_key_blocks(a.c + a.n_keys);
  if (a.g.n_layers < 1 || a.g.n_layers > kMaxGroupLayers) return hipErrorInvalidValue;
  // Items (32-row tiles x query heads of a KV group) per workgroup: a workgroup's keys cost it as much as about six
  // items, up to two workgroups per CU more of them cost nothing, and beyond that the launch takes as long as the CUs with
  // one workgroup more than the others (8 layers of 28/4 heads, 128 queries over 1536 keys: three workgroups for every CU
  // instead of two or three 31.3 -> 30.2 us with the fold, 64 queries 22.3 -> 21.1).
  const int n_items = (a.n_q_heads / a.n_kv_heads) * ((a.n + 31) / 32);
  const long long blocks = (long long)a.n_kv_blocks * a.n_kv_heads * a.g.n_layers;
  long long best = 0;
  for (int splits = 1; splits <= n_items; ++splits) {
    const int per = (n_items + splits - 1) / splits;
    const long long workgroups = blocks * splits, cost = (workgroups <= 512 ? 2 : (workgroups + 255) / 256) * (per + 6);
    if (splits == 1 || cost < best) {
      best = cost;
      a.items_per_wg = per;
    }
  }
  a.item_splits = (n_items + a.items_per_wg - 1) / a.items_per_wg;
  if ((long long)a.n_kv_heads * a.item_splits > 65535) return hipErrorInvalidValue;
  a.group = a.n_q_heads / a.n_kv_heads;
  // (n_obs * n_q_heads < 8192 here: fewer than 8192 items and rows, fewer than 65536 workgroups along y, products below 2^31)
  a.splits_magic = divisor_magic((unsigned)a.item_splits);
  a.tiles_magic = divisor_magic((unsigned)((a.n + 31) / 32));
  a.rows_magic = divisor_magic((unsigned)a.n);
  const dim3 grid(a.n_kv_blocks, a.n_kv_heads * a.item_splits, a.g.n_layers);
  if (head_dim == 128) hipLaunchKernelGGL(rowstat_kernel<128>, grid, dim3(kThreads), 0, s, a);
  else hipLaunchKernelGGL(rowstat_kernel<64>, grid, dim3(kThreads), 0, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int total = a.n_q_heads * a.n;
  hipLaunchKernelGGL(rowstat_fold_kernel, dim3((total + 255) / 256, a.g.n_layers), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace kvp
