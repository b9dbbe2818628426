// Attention of one block of queries over cache U block (Eq. 1) with its scores (Eq. 4), for blocks too
// small to fill the chip with the tiles of attention.hip: the KEYS are split over the waves.
//
// A workgroup of eight waves takes 32 QW query rows of one head (QW = 1 or 2); the KS = 8 / QW waves
// of a 32-row tile take every KS-th block of 32 keys.  The products are those of attention.hip
// (S^T = K Q^T, O^T = V^T P^T, one query row per lane), but a wave works entirely by itself: its K
// and V blocks go straight from global memory into two strips of LDS that belong to the wave, and there
// is no barrier until the KS partial results of a row are added up.  What bounds a block of this
// size is the chain of one workgroup -- launch, first keys from memory, the wave's share of the keys,
// the merge, the second sweep -- and eight short chains replace two or four long ones.
//
// Everything comes through LDS, although a wave could load K and Q fragments straight into registers
// in operand layout: there neighbouring lanes read different rows, and the address path of a CU takes
// such a load at 16 bytes a clock, against 60 when four neighbouring lanes share 64 bytes (measured,
// from L2).
//
// A wave's loop over its key blocks i, with one row tile per workgroup:
//   S = K(i) Q^T from the K strip, then the load of K(i + 1) into it; P = exp(S - m);
//   O += P V(i) from the V strip, then the load of V(i + 1).
// With two row tiles (one from the front of the head, one from the back, for equal work) the waves of a pair need the
// same blocks: one wave of the pair brings in K and the other V, a round ahead, with one barrier per round.  In round i the
// products S(i + 1) carry the exponentials of S(i) and the loads between them, and the products with V(i) the maxima of S(i + 1).
// A round of 64 rows over 128 keys takes 0.94 us (1.2 before that; 28/4 heads, d 128, 512 rows over 1536 keys: 27.0 -> 25.6 us, a launch
// without scores 14.9 -> 13.6 us, 28/4 heads of d 64 19.0 -> 17.0 us).  The second sweep laid out this way was 2 % slower.  (A software pipeline
// as in attention.hip, the products with V a round later still, was slower with one row tile; a touch of all the head's cache lines up
// front gave nothing: the blocks do not wait for memory.)
//
// What a wave does for a block beside its products counts as much as they do: it issues one instruction in about five
// cycles.  Blocks therefore come through buffer descriptors, whose end takes care of a block's missing rows, and their addresses, the
// blocks that need a mask and the reference's margin are carried along instead of being worked out for each; and all fragments of a product
// are asked for before the first of them is used.  16/4 heads, d 64, 333 rows over 1444 keys: 11.2 -> 10.4 us; 28/4 heads, d 128, 256 rows over
// 768 keys: 10.6 -> 10.3 us.  From one whole block to the next a descriptor only moves on, and four loads go out in one statement with one
// setting of M0 (Feed: a block of d 64 had 56 scalar instructions, now 19): 16/4 heads, d 64, 333 rows over 1444 keys 9.06 -> 8.78 us, 28/4
// heads, d 128, 256 rows over 768 keys 8.55 -> 8.37, 16 layers of 28/4 heads, 512 rows over 1536 keys 4863 -> 4646 us a prefix.  What bounds the
// 32-row launches beside that is the path into the CU: the blocks of a round are 64 KiB at d 64 and 128 at d 128, 1024 and 2048 of its 1270 and
// 2000 cycles.
//
// The partial results of a row meet in LDS as they lie in the accumulators; a wave's own are written over its own strips, with no barrier
// in front, and with kept weights a wave puts together one slice of the channels of the rows that its lanes have anyway: 0.3 us of each
// of these launches, 0.1 us of the 64-row ones, against whole padded rows behind a barrier.
//
// Two waves share a SIMD: one has matrix work while the other has vector work.  They start together and would stay
// in step, both at the same kind of work; a wave therefore raises its priority once its products S are on their way and
// lowers it at the end of the block, so that the one that is ahead stays ahead (16/4 heads, d 64, 333 rows over 1444
// keys: 13.6 -> 13.3 us; 28/4 heads, d 128, 256 rows over 768 keys: 9.3 -> 9.0 us per layer of a grouped launch;
// 28/4 heads, 512 rows over 1536 keys, second sweep only: 26.1 -> 25.7 us).  Not with two row tiles in the first sweep,
// whose barrier per round keeps the waves together anyhow.  Leaving out the maximum of every later block, with a
// check of the row sums instead, was slower (25.7 -> 26.7 us): the waves of a SIMD fall into step again.
//
// Softmax reference.  A row's reference is the maximum of its first visible block; a later logit more
// than 2^30 above it (fp32 has room for 2^127) sends the wave through a branch that brings O and the
// row sum onto a new reference.  Ordinary logits never take it.
//
// Scores (Eq. 4), one row tile per workgroup: a wave has few key blocks (three at 768 keys), so the fp32 weights
// exp(S - m) of all of them stay in its registers.  When the rows' normalisers are known, a lane's factor exp(m - lse) turns
// them into the softmax weights of its row, and the column sums run over the lanes: some 50 vector instructions per block,
// where a second sweep takes the keys from L2, the products and the exponentials again.  The kernel is built for each
// number of kept blocks that its registers have room for (16 each: up to 6 at d 128, 8 at d 64; the unrolled loop also
// spares the rest).  16/4 heads, d 64, 333 rows over 1444 keys, when it was built: 13.6 -> 11.4 us per launch; 28/4 heads, d 128, 256 rows over
// 768 keys: 9.6 -> 8.4 us per layer of a grouped launch; 32/32 heads, 128 rows over 384 keys: 8.4 -> 7.8 us.  The
// scores' error against 64 bits is the same (2e-7 in the root mean square).
//
// Second sweep (longer lists; two row tiles, whose waves have more blocks): as in attention.hip, S = Q K^T again
// with the final normalisers, one key per lane, one partial array of column sums per workgroup.  Query fragments
// are, register for register, the A operand of this product.  With two row tiles the weights of the first two rounds (four at d 64) stay in
// registers all the same, the sums of the two tiles meet in LDS, and the second sweep begins behind them (28/4 heads, d 128,
// 512 rows over 1536 keys, with no round kept, two, three, four: 26.6, 25.8, 25.8, 26.8 us; more than two spill).
//
// plan.cpp has the rule that picks this kernel and what it measured against the tiles of attention.hip.
#include <type_traits>

#include "key_scores.h"
#include "kvp_internal.h"
#include "mfma_tools.h"

namespace kvp {
namespace {

constexpr float kRescueLog2 = 30.f;

// Two row tiles per workgroup: rounds whose weights stay in registers.
template <int D, int QW> constexpr int kKeptRounds = QW == 1 ? 0 : D == 64 ? 4 : 2;

template <int D, int QW>
struct Split {
  static constexpr int kWaves = 8;
  static constexpr int KS = kWaves / QW;              // waves that share a 32-row tile
  static constexpr int kThreads = 64 * kWaves;
  static constexpr int kRows = 32 * QW;
  static constexpr int kStrip = 32 * D;               // bf16 elements of a strip: 32 rows of K or V
  static constexpr int kMainBytes = 2 * kWaves * kStrip * 2;       // strips; later the partial outputs, a wave's in as much
  static constexpr int kStatBytes = 2 * kWaves * 32 * 4;           // maximum and sum per wave and row
  static constexpr int kQBytes = kRows * D * 2;       // the workgroup's query rows
  static constexpr int kKeptBytes = kWaves * kKeptRounds<D, QW> * 32 * 4;     // sums of a wave's rows over its kept blocks
  static constexpr int kLdsBytes = kMainBytes + kStatBytes + kQBytes + kRows * 4 + kKeptBytes;
  static_assert(kLdsBytes <= 160 * 1024, "LDS of a CU");
};

// Sums of v times the lane's factor over the 32 lanes of each half of the wave; lane l ends up with that of
// v[8 b4 + 4 b3 + 2 b2 + b1], b0 .. b4 the bits of l: at every step a lane hands the half of its values that its
// partner keeps to that partner.
__device__ __forceinline__ float sum_over_half(float (&v)[16], float factor, int lane) {
  float even = factor, odd = factor;                       // of the rows of sixteen lanes that the swapped values come from
  swap_lanes<16>(even, odd);
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    swap_lanes<16>(v[i], v[i + 8]);
    v[i] = __builtin_fmaf(v[i], even, v[i + 8] * odd);
  }
  // (each step adds twice, the second time in the banks of four lanes that keep the other value alone: with the choices of
  // what to keep and what to hand on there were three instructions for two.  24 layers of 16/4 heads of d 64, 333 rows over 1444
  // keys 6948 -> 6900 us.  The waits are those between a vector instruction and one that reads its result from other lanes, which
  // the compiler does not see to here.)
  float w[4], x[2];
  asm("s_nop 1\n\t"
      "v_add_f32_dpp %0, %4, %4 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %1, %5, %5 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %2, %6, %6 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %3, %7, %7 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %0, %8, %8 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %1, %9, %9 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %2, %10, %10 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %3, %11, %11 row_ror:8 row_mask:0xf bank_mask:0xc"
      : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3])
      : "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "v"(v[4]), "v"(v[5]), "v"(v[6]), "v"(v[7]));
  asm("s_nop 1\n\t"
      "v_add_f32_dpp %0, %2, %2 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %1, %3, %3 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %0, %4, %4 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
      "v_add_f32_dpp %1, %5, %5 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
      "s_nop 1"
      : "=&v"(x[0]), "=&v"(x[1])
      : "v"(w[0]), "v"(w[1]), "v"(w[2]), "v"(w[3]));
  const bool b1 = lane & 2;
  const float mine = b1 ? x[1] : x[0], theirs = b1 ? x[0] : x[1];
  const float two = mine + dpp_lane<0x4E>(theirs);         // lane ^ 2
  return two + dpp_lane<0xB1>(two);                        // lane ^ 1
}

// kKept: key blocks of a wave whose softmax weights stay in registers; 0: the scores take a second sweep;
// kScoreByKeys: no scores from the queries, and the first workgroups of the launch score by the keys alone
constexpr int kScoreByKeys = -1;
//
// Without scores a workgroup at d 64 has 112 (one row tile) or 124 (two) registers a lane, and two of them fit on a CU.  With two row tiles
// that takes the second sweep out (launches with scores keep weights) and the loop over the rounds in one piece: the first rounds
// taken apart from the others, as the compiler would, had 138 and one workgroup per CU.  Whole prefixes, 8 layers per launch: 16/4
// heads, 640 rows over 1920 keys, proxy queries 969 -> 812 us, 1300 over 3900 1141 -> 978; 32/32 heads, 512 rows over 1536 keys 1954 -> 1647;
// 28/4 heads, 512 rows over 1536 keys, scored by the keys 1199 -> 1006.  At d 128, where one workgroup fits either way, the first rounds
// apart are the faster way: 16 layers of 28/4 heads, 512 rows over 1536 keys, proxy queries, a prefix 3710 us, in one piece 3726, with the
// second sweep left in 3723.
template <int D, int QW, int kKept>
__global__ void __launch_bounds__((Split<D, QW>::kThreads))
attention_split_kernel(const AttnArgs args) {
  using S = Split<D, QW>;
  constexpr bool kScores = kKept > 0 || (kKept == 0 && QW == 1);      // where launches with scores come
  constexpr int KS = S::KS;
  constexpr int kNK = D / 16;                // K fragments (and MFMAs) of a 32-key block
  constexpr int kND = D / 32;                // channel tiles of O
  constexpr int kChunks = D / 8;             // 16-byte chunks per row
  constexpr int kRowsPerLoad = 64 / kChunks; // rows one wave instruction brings in
  constexpr int kLoads = 32 / kRowsPerLoad;  // instructions for a 32-row block
  extern __shared__ __align__(16) unsigned char lds_raw[];
  float* const stat_m = reinterpret_cast<float*>(lds_raw + S::kMainBytes);       // [kWaves][32]
  float* const stat_l = stat_m + S::kWaves * 32;
  u16* const q_lds = reinterpret_cast<u16*>(stat_l + S::kWaves * 32);            // [kRows][D], chunks swizzled like K's
  float* const lse_lds = reinterpret_cast<float*>(q_lds + S::kRows * D);         // [kRows]
  float* const kept_lds = lse_lds + S::kRows;                                    // [kWaves][kKeptRounds][32]

  const int li = blockIdx.y;
  AttnPlan a = args;
  const u16* const q_rows = args.layer[li].q;
  u16* const out_rows = args.layer[li].out;
  have_arguments(q_rows, out_rows, args.layer[li].k_new, args.layer[li].v_new, a.k_cache, a.v_cache, a.lse2, a.partial, a.g.first_set,
                 a.g.n_sets, a.g.set_stride, a.g.kv_stride, a.n, a.c, a.work_per_xcd, a.total_work, a.tiles_magic, a.group_magic);
  // (loaded again where they are used, eight waits on a wave's way: a whole prefix of 16/4 heads, d 64, 333 rows over
  // 1444 keys, a layer per launch 7866 -> 7741 us; of 28/4 heads, d 128, 256 rows over 768 keys, eight layers per launch 851 -> 837 us)
  keep_arguments(a.n_q_heads, a.n_kv_heads, a.n_keys, a.n_row_tiles, a.budget, a.shift, a.group, a.scale_log2, a.lse_stride,
                 a.partial_stride, a.cand_stride);
  int block = (int)blockIdx.x;
  if constexpr (kKept == kScoreByKeys) {
    // They start with the launch and take about as long as an attention workgroup.
    static_assert(S::kThreads == kKeyScoreThreads && (S::kWaves + 1) * D * 4 <= S::kMainBytes);
    block -= a.key_score_wgs;
    if (block < 0) {
      const int hk = (int)blockIdx.x;
      if (hk < a.n_kv_heads)
        score_head_by_keys<D>(a.k_cache + (size_t)li * a.g.kv_stride + (size_t)hk * a.budget * D, args.layer[li].k_new + (size_t)hk * D,
                              a.n_kv_heads, a.c, a.c + a.n_keys, reinterpret_cast<float*>(lds_raw),
                              in_set_of(a.partial, a.g, li) + (size_t)hk * a.partial_stride);
      return;
    }
  }
  // XCD-aware order: consecutive work items (same KV head) land on one die
  const int w = (block % kXcds) * a.work_per_xcd + block / kXcds;
  if (w >= a.total_work) return;
  float* const lse2 = in_set_of(a.lse2, a.g, li);
  const int group = a.group;
  const int h = (int)quotient((unsigned)w, a.tiles_magic);
  const int rt = a.n_row_tiles - 1 - (w - h * a.n_row_tiles);    // long rows first
  const int hk = (int)quotient((unsigned)h, a.group_magic);

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qw = wave / KS, ks = wave % KS;
  const int l32 = lane & 31;
  const int g = lane >> 5;

  const int n = a.n, c = a.c, shift = a.shift;
  // Row tiles.  Two of a workgroup are one from the front of the head and one from the back, so that all workgroups see
  // about as many keys; and since waves w and w + 4 share a SIMD, the late tile's wave has the SIMD to itself
  // when the early tile has run out of visible keys.
  auto tile_row = [&](int t) __attribute__((always_inline)) {
    return 32 * (QW == 1 || t == 0 ? rt : 2 * a.n_row_tiles - 1 - rt);
  };
  const int q0 = tile_row(qw);                             // first query row of this wave
  const u16* const kc = a.k_cache + (size_t)li * a.g.kv_stride + (size_t)hk * a.budget * D;
  const u16* const vc = a.v_cache + (size_t)li * a.g.kv_stride + (size_t)hk * a.budget * D;
  const u16* const kn = args.layer[li].k_new + (size_t)hk * D;
  const u16* const vn = args.layer[li].v_new + (size_t)hk * D;
  const int new_stride = a.n_kv_heads * D;
  const float sl2 = a.scale_log2;

  // ---- key blocks: 32 keys of the cache first, then those among the block's own keys (each part is cut
  // into 32s by itself, so a block lies in one or the other)
  const int c_blk = (c + 31) / 32;
  struct Block {
    bool cached;
    int first, rows;                         // first row within the cache or the block's keys; real rows
  };
  auto block_of = [&](int b) __attribute__((always_inline)) -> Block {
    const bool cached = b < c_blk;
    const int first = 32 * (cached ? b : b - c_blk);
    return Block{cached, first, min(32, (cached ? c : a.n_keys) - first)};
  };

  // ---- global memory -> LDS, 16 bytes per lane.  Instruction j brings in rows kRowsPerLoad j + (0 ..
  // kRowsPerLoad - 1) of a 32-row strip; the 16-byte chunks of a row are XOR-swizzled on the way so that the
  // fragment reads are free of bank conflicts (K and Q: by the row, V: v_swizzle).  Inline assembly for the
  // reasons given in attention.hip; the waits are this kernel's own.  (s_nop 3: a load may read a scalar register five wait states after a
  // vector instruction, such as one that reads the first lane, has written it, and the compiler does not see to that here.)
  u16* const k_strip = reinterpret_cast<u16*>(lds_raw) + wave * S::kStrip;
  u16* const v_strip = k_strip + S::kWaves * S::kStrip;
  const unsigned lds_base =
      __builtin_amdgcn_readfirstlane((unsigned)(size_t)(__attribute__((address_space(3))) void*)lds_raw);
  auto lds_addr = [&](const u16* p) __attribute__((always_inline)) -> unsigned {
    return lds_base + 2u * (unsigned)(p - reinterpret_cast<u16*>(lds_raw));
  };
  auto load_row16 = [&](const u16* base, unsigned lane_bytes, unsigned to) __attribute__((always_inline)) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 3\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(lane_bytes), "s"(base), "s"(to)
                 : "m0", "memory");
  };
  const int ld_sub = lane / kChunks, ld_pos = lane % kChunks;
  const int ld_chunk_k = ld_pos ^ ld_sub, ld_chunk_v = ld_pos ^ v_swizzle<D>(ld_sub);
  // rows [0, rows) at `base`, `stride` elements apart; rows past the end: the last one again
  auto load_strip = [&](const u16* base, int stride, int rows, u16* strip, int j) __attribute__((always_inline)) {
    // row kRowsPerLoad j + ld_sub of the strip: its swizzle is the lane's, with bits of j where a row has 16 chunks
    const int chunk = ld_chunk_k ^ ((kRowsPerLoad * j) % kChunks);
    const int row = min(kRowsPerLoad * j + ld_sub, rows - 1);
    load_row16(base, 2u * (unsigned)(row * stride + 8 * chunk), lds_addr(strip + j * kRowsPerLoad * D));
  };
  auto wait_older_than = [&](auto newest) __attribute__((always_inline)) {   // all but the `newest` latest loads have landed
    constexpr int k = decltype(newest)::value;
    static_assert(k <= 16, "fits the two fields of the wait");
    __builtin_amdgcn_s_waitcnt(0x0F70 | (k & 15) | (k >> 4 << 14));
    asm volatile("" ::: "memory");
  };
  typedef std::integral_constant<int, 0> None;
  typedef std::integral_constant<int, kLoads> OneBlock;
  typedef std::integral_constant<int, 2 * kLoads> TwoBlocks;

  // ---- per-lane LDS read offsets (bf16 elements), as in attention.hip
  int k_off[kNK];
#pragma unroll
  for (int st = 0; st < kNK; ++st) k_off[st] = l32 * D + 8 * ((2 * st) ^ (g ^ (l32 % kChunks)));
  int v_off[kND];
  {
    const int rsub = 4 * g + ((lane & 15) >> 2);
#pragma unroll
    for (int dt = 0; dt < kND; ++dt)
      v_off[dt] = rsub * D + 8 * ((4 * dt + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) ^ v_swizzle<D>(rsub)) + 4 * (lane & 1);
  }

  // ---- first sweep
  const int rows_end = min(n, q0 + 32);
  const int n_blk = c_blk + (min(a.n_keys, rows_end + shift) + 31) / 32;     // blocks some row of the tile sees
  const int my_blk = q0 < n && n_blk > ks ? (n_blk - ks + KS - 1) / KS : 0;   // (a tile may lie past the end)
  auto mine = [&](int i) __attribute__((always_inline)) { return block_of(ks + KS * i); };
  const int wg_rows_end = min(n, tile_row(QW - 1) + 32);
  const int n_kb = c_blk + (min(a.n_keys, wg_rows_end + shift) + 31) / 32;   // blocks some row of the workgroup sees
  // A block comes in through a buffer descriptor that ends with it: rows past its end come as zeros, and so does a block that
  // does not exist.  Two row tiles share their blocks: of the waves (0, ks) and (1, ks) one brings in K and the other V for both, a
  // round of KS blocks ahead, into the strips that the round before has left.
  constexpr bool kShared = QW == 2;
  const u16* const k_mine = reinterpret_cast<const u16*>(lds_raw) + ks * S::kStrip;      // [2][KS][kStrip], then V's
  const u16* const v_mine = k_mine + 2 * KS * S::kStrip;
  const unsigned my_to = lds_addr(qw == 0 ? k_mine : v_mine);
  const unsigned new_bytes = 2u * (unsigned)new_stride;
  // What brings in a wave's blocks, every `step` blocks of the list.  From one whole block to the next of the cache, or of the block's
  // own rows, the addresses move on and nothing else changes; the rest is worked out where the kind of block changes.  Load j brings in
  // rows kRowsPerLoad j .. of a block; its immediate offset moves both of its addresses, that in memory and that in LDS, by 1 KiB from load
  // to load, and the lane's part of an address takes that back where the rows lie further apart.  A lane keeps its part for each load
  // of four, or only that of the first where registers are short.
  constexpr int kLaneParts = (D == 64 && kKept == 0) || (D == 128 && kKept == 6) ? 1 : 4;
  struct Feed {
    u32x4 k, v;                              // descriptors: from the block's first row to its last one's end
    int whole;                               // blocks after this one that only move on
    bool cached;
    unsigned by;                             // bytes to the next block
    unsigned k_lane[kLaneParts], v_lane[kLaneParts];       // lanes' parts of an address
    unsigned further;                        // bytes in memory from a load to the load four on; or to the next one, beyond the 1 KiB
  };
  typedef std::true_type Yes;
  typedef std::false_type No;
  // `two`: K and V; else one tensor, in the place of K, whose chunks are K's or V's (`like_k`)
  auto feed_lanes = [&](Feed& f, auto two, bool like_k) __attribute__((always_inline)) {
    const unsigned row_bytes = f.cached ? 2u * D : new_bytes;
    f.further = kLaneParts == 4 ? 4 * kRowsPerLoad * row_bytes : kRowsPerLoad * row_bytes - 1024u;
#pragma unroll
    for (int j = 0; j < kLaneParts; ++j) {
      const unsigned row = (unsigned)(kRowsPerLoad * j + ld_sub) * row_bytes - 1024u * j;
      const int chunk_k = ld_chunk_k ^ ((kRowsPerLoad * j) % kChunks);
      f.k_lane[j] = row + 16u * (unsigned)(like_k ? chunk_k : ld_chunk_v);
      if constexpr (decltype(two)::value) f.v_lane[j] = row + 16u * (unsigned)ld_chunk_v;
    }
  };
  auto buffer_at = [&](unsigned long long at, unsigned bytes) __attribute__((always_inline)) -> u32x4 {
    return u32x4{(unsigned)at, (unsigned)(at >> 32) & 0xFFFFu, bytes, 0x00020000u};
  };
  struct Tensors {
    const u16 *kc, *kn, *vc, *vn;            // (one tensor: in the place of K)
    int end;                                 // blocks from this one on are not wanted
  };
  auto feed_at = [&](Feed& f, const Tensors& of, int b, int step, auto two) __attribute__((always_inline)) {
    f.cached = b < c_blk;
    const int first = 32 * (f.cached ? b : b - c_blk), after = (f.cached ? c : min(a.n_keys, 32 * (of.end - c_blk))) - first - 32;
    const unsigned row_bytes = f.cached ? 2u * D : new_bytes;
    const unsigned long long at = (unsigned long long)(unsigned)first * row_bytes;
    unsigned long long ka = (unsigned long long)of.kc, kb = (unsigned long long)of.kn;
    asm("" : "+s"(ka), "+s"(kb));            // (choices between values, no branch)
    const int rows = min(after + 32, 32);
    const unsigned bytes = rows > 0 ? (unsigned)(rows - 1) * row_bytes + 2u * D : 0u;
    f.k = buffer_at((f.cached ? ka : kb) + at, bytes);
    if constexpr (decltype(two)::value) {
      unsigned long long va = (unsigned long long)of.vc, vb = (unsigned long long)of.vn;
      asm("" : "+s"(va), "+s"(vb));
      f.v = buffer_at((f.cached ? va : vb) + at, bytes);
    }
    f.by = 32u * (unsigned)step * row_bytes;
    f.whole = after > 0 && row_bytes < 1u << 23 ? (int)((unsigned)after / (32u * (unsigned)step)) : 0;       // (`by` is a 32-bit number)
  };
  auto move_on = [&](u32x4& buffer, unsigned by) __attribute__((always_inline)) {
    const unsigned long long at = ((unsigned long long)buffer.y << 32 | buffer.x) + by;
    buffer.x = (unsigned)at;
    buffer.y = (unsigned)(at >> 32);
  };
  // On to block b, `step` blocks after the one that the feed is at.
  auto feed_moves = [&](Feed& f, auto two) __attribute__((always_inline)) {
    --f.whole;
    move_on(f.k, f.by);
    if constexpr (decltype(two)::value) move_on(f.v, f.by);
  };
  auto feed_anew = [&](Feed& f, const Tensors& of, int b, int step, auto two, bool like_k) __attribute__((always_inline)) {
    const bool was = f.cached;
    feed_at(f, of, b, step, two);
    if (f.cached != was) feed_lanes(f, two, like_k);
  };
  auto feed_on = [&](Feed& f, const Tensors& of, int b, int step, auto two, bool like_k) __attribute__((always_inline)) {
    if (f.whole > 0) feed_moves(f, two);
    else feed_anew(f, of, b, step, two, like_k);
  };
  // Loads 4 i .. 4 i + 3 of a block, in one statement: what sets M0 and what reads it stay together.  k_bits: all ones for K, whose
  // chunks are swizzled by the row, zero for V.
  auto load_four = [&](const u32x4& from, const unsigned (&lane_at)[kLaneParts], unsigned further, int i, unsigned to, unsigned k_bits)
      __attribute__((always_inline)) {
    unsigned at[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if constexpr (kLaneParts == 4) at[j] = lane_at[j] + (unsigned)i * further;
      else at[j] = (lane_at[0] ^ (16u * ((kRowsPerLoad * j) % kChunks) & k_bits)) + (unsigned)(4 * i + j) * further + 4096u * i;
    }
    // (through the first lane: the compiler would carry the descriptor from block to block in vector registers)
    const u32x4 buffer = {(unsigned)__builtin_amdgcn_readfirstlane(from.x), (unsigned)__builtin_amdgcn_readfirstlane(from.y),
                          (unsigned)__builtin_amdgcn_readfirstlane(from.z), 0x00020000u};
    asm volatile("s_mov_b32 m0, %5\n\ts_nop 3\n\t"
                 "buffer_load_dwordx4 %0, %4, 0 offen lds\n\t"
                 "buffer_load_dwordx4 %1, %4, 0 offen offset:1024 lds\n\t"
                 "buffer_load_dwordx4 %2, %4, 0 offen offset:2048 lds\n\t"
                 "buffer_load_dwordx4 %3, %4, 0 offen offset:3072 lds" ::"v"(at[0]), "v"(at[1]), "v"(at[2]), "v"(at[3]), "s"(buffer), "s"(to + 4096u * i)
                 : "m0", "memory");
  };
  auto load_all = [&](const Feed& f, const u32x4& from, const unsigned (&lane_at)[kLaneParts], unsigned to, unsigned k_bits) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < kLoads / 4; ++i) load_four(from, lane_at, f.further, i, to, k_bits);
  };
  const unsigned my_bits = qw == 0 ? ~0u : 0u;

  // the workgroup's query rows (each wave brings in its share), the wave's first block
  for (int j = wave; j < QW * kLoads; j += S::kWaves) {
    const int first_row = tile_row(j / kLoads);                // rows past the block are computed, not stored
    load_strip(q_rows + ((size_t)min(first_row, n - 1) * a.n_q_heads + h) * D, a.n_q_heads * D, max(min(32, n - first_row), 1),
               q_lds + (j / kLoads) * S::kStrip, j % kLoads);
  }
  Feed feed;                                 // one row tile: of block i and then i + 1; two: of the block that comes in next
  const Tensors tensors = kShared ? Tensors{qw == 0 ? kc : vc, qw == 0 ? kn : vn, nullptr, nullptr, n_kb} : Tensors{kc, kn, vc, vn, n_blk};
  typedef std::integral_constant<bool, !kShared> Both;
  auto next_shared = [&](int i) __attribute__((always_inline)) { feed_on(feed, tensors, ks + KS * i, KS, No{}, qw == 0); };
  feed_at(feed, tensors, ks, KS, Both{});
  feed_lanes(feed, Both{}, kShared ? qw == 0 : true);
  if constexpr (kShared) {
    load_all(feed, feed.k, feed.k_lane, my_to, my_bits);                       // K(0) or V(0)
    next_shared(1);
    if (qw == 0) {
      load_all(feed, feed.k, feed.k_lane, my_to + 2u * (unsigned)(KS * S::kStrip), my_bits);        // K(1)
      next_shared(2);
    }
    wait_older_than(OneBlock{});
  } else {
    load_all(feed, feed.k, feed.k_lane, lds_addr(k_strip), ~0u);
    load_all(feed, feed.v, feed.v_lane, lds_addr(v_strip), 0u);
    wait_older_than(TwoBlocks{});
  }
  __builtin_amdgcn_s_barrier();              // the query rows are in LDS
  asm volatile("" ::: "memory");
  bf16x8 qf[kNK];
#pragma unroll
  for (int st = 0; st < kNK; ++st) qf[st] = lds_read_b128(q_lds + qw * S::kStrip + k_off[st]);
  f32x16 o[kND];
  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int dt = 0; dt < kND; ++dt) o[dt] = zero;
  float m_ref = -INFINITY, l_run = 0.f;
  // the margin in units of the raw dot product; finite, whatever the scale, so that a row without a reference keeps its limit
  const float rescue_raw = fminf(kRescueLog2 / sl2, __FLT_MAX__);
  float limit = -INFINITY, neg = 0.f;        // m_ref + rescue_raw; -m_ref in the exponent, 0 while the row has seen nothing
  // of this wave's blocks: the part block of the cache, if it has that one; the first of which some row may not see some key
  const int part_blk = c % 32 != 0 && (c_blk - 1 - ks) % KS == 0 ? (c_blk - 1 - ks) / KS : -1;
  const int edge = c_blk + min((q0 + shift + 1) / 32, a.n_keys / 32) - ks;
  const int edge_blk = edge > 0 ? (edge + KS - 1) / KS : 0;
  auto max_of = [&](const f32x16& x) __attribute__((always_inline)) {
    float m = x[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) m = fmaxf(m, x[r]);
    return max_with_other_half(m);
  };
  // hides what the rows of the tile may not see of block i
  auto hide = [&](int i, f32x16& s) __attribute__((always_inline)) {
    const Block b = mine(i);
    const int last = b.cached ? b.rows - 1 : min(b.rows - 1, q0 + l32 + shift - b.first);
    const int lim = last - 4 * g;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = (8 * (r >> 2) + (r & 3) <= lim) ? s[r] : -INFINITY;
  };
  // a new reference at block i for rows whose maximum is far above it, or which see their first key
  auto new_reference = [&](int i, float mx) __attribute__((always_inline)) {
    const float m_new = fmaxf(m_ref, mx);
    if (i > 0) {
      const float f = m_ref == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m_ref - m_new) * sl2);
      l_run *= f;
#pragma unroll
      for (int dt = 0; dt < kND; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[dt][r] *= f;
    }
    m_ref = m_new;
    limit = m_ref + rescue_raw;
    neg = -(m_ref == -INFINITY ? 0.f : m_ref) * sl2;
  };

  auto p_frag = [](const unsigned (&p)[8], int mm) __attribute__((always_inline)) {
    const u32x4 pw = {p[4 * mm], p[4 * mm + 1], p[4 * mm + 2], p[4 * mm + 3]};
    return __builtin_bit_cast(bf16x8, pw);
  };
  // block i of this wave, K and V in LDS; k_read runs when K has been read, v_wait before V is
  auto attend = [&](int i, const u16* k_from, const u16* v_from, float (&p)[16], auto&& k_read, auto&& v_wait) __attribute__((always_inline)) {
    f32x16 s;
    bf16x8 kf[kNK];
#pragma unroll
    for (int st = 0; st < kNK; ++st) kf[st] = lds_read_b128(k_from + k_off[st]);
    __builtin_amdgcn_sched_barrier(0);       // all on their way before the first product
#pragma unroll
    for (int st = 0; st < kNK; ++st) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[st], qf[st], st == 0 ? zero : s, 0, 0, 0);
    __builtin_amdgcn_s_setprio(1);
    k_read();
    if (i >= edge_blk || i == part_blk) hide(i, s);
    const float mx = max_of(s);
    if (__any(mx > limit)) new_reference(i, mx);
    unsigned pw[8];
    float sum = 0.f;
    auto weigh_pair = [&](int k) __attribute__((always_inline)) {
      p[2 * k] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[2 * k], sl2, neg));
      p[2 * k + 1] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[2 * k + 1], sl2, neg));
      sum += p[2 * k] + p[2 * k + 1];
      pw[k] = pack_bf16(p[2 * k], p[2 * k + 1]);
    };
#pragma unroll
    for (int k = 0; k < 4; ++k) weigh_pair(k);
    v_wait();
    bf16x8 vf[2 * kND];
#pragma unroll
    for (int dt = 0; dt < kND; ++dt) {
      vf[dt] = lds_read_vt(v_from + v_off[dt], 8 * D);
      vf[kND + dt] = lds_read_vt(v_from + v_off[dt] + 16 * D, 8 * D);
    }
    __builtin_amdgcn_sched_barrier(0);
    // the products with the first sixteen keys run beside the exponentials of the other sixteen
#pragma unroll
    for (int dt = 0; dt < kND; ++dt) o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[dt], p_frag(pw, 0), o[dt], 0, 0, 0);
#pragma unroll
    for (int k = 4; k < 8; ++k) weigh_pair(k);
#pragma unroll
    for (int dt = 0; dt < kND; ++dt) o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[kND + dt], p_frag(pw, 1), o[dt], 0, 0, 0);
    l_run += sum;
    __builtin_amdgcn_s_setprio(0);
  };
  float kept[kKept > 0 ? kKept : 1][16], kept_m[kKept > 0 ? kKept : 1];      // weights against the references kept_m
  if constexpr (kShared) {
    // Round i: S(i + 1) = K(i + 1) Q^T with the exponentials of S(i) between the products, then O += P(i) V(i).
    constexpr int kNV = 2 * kND;
    constexpr int kAhead = D / 32;           // fragments read ahead of their product
    // The feed moves on among the products with V, a branch and all: 16 layers of 28/4 heads, d 128, 512 rows over 1536 keys, a layer
    // per launch 4764 us a prefix with the feed behind the products, 4734 with it here.  (Set anew for every block, without a branch, with the
    // loop in one piece or not: 16 layers per launch without scores 0.8 % slower.)
    //
    // The loads go out four at a time beside two of the products with K, which ones was measured.  The same prefix, a layer per launch with
    // scores: 4867 us with a load beside each product, 4788 with four beside products 0 and 4, 4883 with 2 and 10.  16 layers per launch without
    // scores, where a CU has one workgroup after the other: 3940 us with a load beside each, 3920 with 0 and 4, 3900 with 1 and 6; 0 and 1
    // were 1.6 % slower than 0 and 4.
    constexpr int kLoadsWith[2] = {kKept > 0 ? 0 : 1, kKept > 0 ? 5 : 6};
    f32x16 s2[2];
    float mx;                                // of the row's logits in the block that comes next
    static_assert(kLoads == kNK);
    auto shared_loads = [&](int k, auto parity) __attribute__((always_inline)) {           // four loads of the block that comes in
      constexpr int par = decltype(parity)::value;
      load_four(feed.k, feed.k_lane, feed.further, k, my_to + 2u * (unsigned)((qw == 0 ? par : par ^ 1) * KS * S::kStrip), my_bits);
    };
    auto phase = [&](int i, auto parity, float (&p)[16]) __attribute__((always_inline)) {
      constexpr int par = decltype(parity)::value;
      f32x16& s = s2[par];
      f32x16& s_new = s2[par ^ 1];
      unsigned pw[8];
      const u16* const kt = k_mine + (par ^ 1) * KS * S::kStrip;
      const u16* const vt = v_mine + par * KS * S::kStrip;
      bf16x8 kfr[kNK], vfr[kNV];
      auto read_k = [&](int st) __attribute__((always_inline)) { kfr[st] = lds_read_b128(kt + k_off[st]); };
      auto read_v = [&](int vi) __attribute__((always_inline)) { vfr[vi] = lds_read_vt(vt + v_off[vi % kND] + 16 * (vi / kND) * D, 8 * D); };
#pragma unroll
      for (int st = 0; st < kAhead; ++st) read_k(st);
      __builtin_amdgcn_sched_barrier(0);
      if (i >= edge_blk || i == part_blk) {
        hide(i, s);
        mx = max_of(s);
      }
      if (__any(mx > limit)) new_reference(i, mx);
      __builtin_amdgcn_sched_barrier(0);
      float sum = 0.f, arg = __builtin_fmaf(s[0], sl2, neg), pe1 = 0.f, pe2 = 0.f;
      auto finish_element = [&](int e) __attribute__((always_inline)) {      // element e: pe1, the one before: pe2
        sum += pe1;
        asm volatile("" : "+v"(sum));
        p[e] = pe1;
        if (e & 1) pw[e >> 1] = pack_bf16(pe2, pe1);
      };
      auto weigh = [&](int from, int end) __attribute__((always_inline)) {
#pragma unroll
        for (int e = from; e < end; ++e) {
          const float pe = __builtin_amdgcn_exp2f(arg);
          if (e + 1 < 16) arg = __builtin_fmaf(s[e + 1], sl2, neg);
          if (e >= 1) finish_element(e - 1);
          pe2 = pe1;
          pe1 = pe;
        }
      };
#pragma unroll
      for (int st = 0; st < kNK; ++st) {
        if (st + kAhead < kNK) read_k(st + kAhead);
        else read_v(st + kAhead - kNK);
        s_new = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kfr[st], qf[st], st == 0 ? zero : s_new, 0, 0, 0);
        weigh(10 * st / kNK, 10 * (st + 1) / kNK);
#pragma unroll
        for (int k = 0; k < kLoads / 4; ++k)
          if (st == kLoadsWith[k]) shared_loads(k, parity);
        __builtin_amdgcn_sched_barrier(0);
      }
      float m = -INFINITY;
#pragma unroll
      for (int vi = 0; vi < kNV; ++vi) {
        if (vi + kAhead < kNV) read_v(vi + kAhead);
        o[vi % kND] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vfr[vi], p_frag(pw, vi / kND), o[vi % kND], 0, 0, 0);
        if (vi < kND) {                      // beside the products with the first sixteen keys
          weigh(10 + 6 * vi / kND, 10 + 6 * (vi + 1) / kND);
          if (vi == kND - 1) finish_element(15);
        } else {
          if (vi == kND) next_shared(i + (qw == 0 ? 3 : 2));
#pragma unroll
          for (int r = 16 * (vi - kND) / kND; r < 16 * (vi - kND + 1) / kND; r += 2) m = fmaxf(fmaxf(m, s_new[r]), s_new[r + 1]);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      l_run += sum;
      mx = max_with_other_half(m);
    };
    const int n_rounds = (n_kb + KS - 1) / KS;
    auto round = [&](int i, auto parity, float (&p)[16]) __attribute__((always_inline)) {
      wait_older_than(None{});               // this wave's share of the blocks has landed
      __builtin_amdgcn_s_barrier();          // everybody's has, and everybody is done with round i - 1
      asm volatile("" ::: "memory");
      if (i < my_blk) {
        phase(i, parity, p);
      } else {
#pragma unroll
        for (int k = 0; k < kLoads / 4; ++k) shared_loads(k, parity);
        next_shared(i + (qw == 0 ? 3 : 2));
      }
    };
    typedef std::integral_constant<int, 0> Even;
    typedef std::integral_constant<int, 1> Odd;
    {                                        // S(0), with nothing beside it
      bf16x8 kfr[kNK];
#pragma unroll
      for (int st = 0; st < kNK; ++st) kfr[st] = lds_read_b128(k_mine + k_off[st]);
#pragma unroll
      for (int st = 0; st < kNK; ++st) s2[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kfr[st], qf[st], st == 0 ? zero : s2[0], 0, 0, 0);
      mx = max_of(s2[0]);
    }
#pragma unroll
    for (int i = 0; i < kKept; ++i)
      if (i < n_rounds) {
        if (i & 1) round(i, Odd{}, kept[i]);
        else round(i, Even{}, kept[i]);
        kept_m[i] = m_ref;
      }
    constexpr int kFrom = kKept > 0 ? kKept : 0;
    float p[16];
    auto two_rounds = [&](int i) __attribute__((always_inline)) {
      round(i, std::integral_constant<int, kFrom & 1>{}, p);
      if (i + 1 < n_rounds) round(i + 1, std::integral_constant<int, (kFrom & 1) ^ 1>{}, p);
    };
    if constexpr (D == 64 && kKept == 0) {
#pragma nounroll
      for (int i = kFrom; i < n_rounds; i += 2) two_rounds(i);
    } else {
      for (int i = kFrom; i < n_rounds; i += 2) two_rounds(i);
    }
    wait_older_than(None{});
  } else {
    auto step = [&](int i, float (&p)[16]) __attribute__((always_inline)) {
      const bool more = i + 1 < my_blk;
      wait_older_than(OneBlock{});           // K(i) is in its strip; V(i) may still be on its way
      attend(i, k_strip, v_strip, p,
             [&]() __attribute__((always_inline)) {
               __builtin_amdgcn_s_waitcnt(0xC07F);         // the strip has been read
               if (more) {
                 feed_on(feed, tensors, ks + KS * (i + 1), KS, Yes{}, true);
                 load_all(feed, feed.k, feed.k_lane, lds_addr(k_strip), ~0u);
               }
             },
             [&]() __attribute__((always_inline)) {
               if (more) wait_older_than(OneBlock{});      // V(i) is in its strip; K(i + 1) may still be on its way
               else wait_older_than(None{});
             });
      __builtin_amdgcn_s_waitcnt(0xC07F);    // the strip has been read
      if (more) load_all(feed, feed.v, feed.v_lane, lds_addr(v_strip), 0u);
    };
    if constexpr (kKept > 0) {
#pragma unroll
      for (int i = 0; i < kKept; ++i)
        if (i < my_blk) {
          step(i, kept[i]);
          kept_m[i] = m_ref;
        }
    } else {
      float p[16];
      for (int i = 0; i < my_blk; ++i) step(i, p);
    }
  }

  // ---- merge the KS partial results of every row through LDS, as they lie in the accumulators: the channels are cut into KS
  // slices, every wave leaves its part of all of them (one row tile: in its own strips, with nobody to wait for) and adds up one
  // slice over the waves of its tile
  constexpr int kSlice = 16 * kND / KS;      // registers of a slice
  wait_older_than(None{});                   // (the block after the last one does not exist, but is asked for)
  auto slice_at = [&](int of_wave, int sl) __attribute__((always_inline)) {
    return reinterpret_cast<f32x4*>(reinterpret_cast<u16*>(lds_raw) + (of_wave + (sl < KS / 2 ? 0 : S::kWaves)) * S::kStrip) +
           (sl % (KS / 2)) * (kSlice / 4) * 64 + lane;
  };
  l_run = sum_with_other_half(l_run);        // lanes l and l + 32 each summed half of the keys of a row
  if constexpr (kShared) __syncthreads();    // nobody needs the strips any more
#pragma unroll
  for (int sl = 0; sl < KS; ++sl) {
    f32x4* const to = slice_at(wave, sl);
#pragma unroll
    for (int k = 0; k < kSlice / 4; ++k) {
      const int r = sl * kSlice + 4 * k;
      to[64 * k] = f32x4{o[r / 16][r % 16], o[r / 16][r % 16 + 1], o[r / 16][r % 16 + 2], o[r / 16][r % 16 + 3]};
    }
  }
  if (g == 0) {
    stat_m[wave * 32 + l32] = m_ref;
    stat_l[wave * 32 + l32] = l_run;
  }
  const bool score = kScores && a.partial != nullptr;
  __syncthreads();
  float lse_row;                             // of row l32 of the wave's tile
  {
    float m = -INFINITY, l = 0.f, f[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) m = fmaxf(m, stat_m[(qw * KS + s) * 32 + l32]);
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      f[s] = __builtin_amdgcn_exp2f((stat_m[(qw * KS + s) * 32 + l32] - m) * sl2);       // 0 for a wave that saw nothing
      l += stat_l[(qw * KS + s) * 32 + l32] * f[s];
    }
    lse_row = m * sl2 + __builtin_log2f(l);
    f32x4 acc[kSlice / 4];
#pragma unroll
    for (int k = 0; k < kSlice / 4; ++k) acc[k] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const f32x4* const from = slice_at(qw * KS + s, ks);
#pragma unroll
      for (int k = 0; k < kSlice / 4; ++k) {
        const f32x4 v = from[64 * k];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[k][e] += f[s] * v[e];
      }
    }
    const int orow = q0 + l32;
    if (ks == 0 && g == 0) {
      lse_lds[32 * qw + l32] = lse_row;
      if (orow < n) lse2[(size_t)h * a.lse_stride + orow] = lse_row;
    }
    if (out_rows != nullptr) {
      // registers 4 k .. 4 k + 3 of the slice are channels 8 k + 4 g .. + 3 of its 2 kSlice; of two neighbouring fours the
      // halves of the wave exchange one, and each lane has eight channels in a row
      const float inv = 1.f / l;
      u16* const dst = out_rows + ((size_t)min(orow, n - 1) * a.n_q_heads + h) * D + 2 * kSlice * ks;
      u32x2 pk[kSlice / 4];
#pragma unroll
      for (int k = 0; k < kSlice / 4; ++k) pk[k] = u32x2{pack_bf16(acc[k][0] * inv, acc[k][1] * inv), pack_bf16(acc[k][2] * inv, acc[k][3] * inv)};
      if constexpr (kSlice == 4) {
        if (orow < n) *reinterpret_cast<u32x2*>(dst + 4 * g) = pk[0];
      } else {
#pragma unroll
        for (int k = 0; k < kSlice / 4; k += 2) {
          const auto x = __builtin_amdgcn_permlane32_swap(pk[k].x, pk[k + 1].x, false, false);
          const auto y = __builtin_amdgcn_permlane32_swap(pk[k].y, pk[k + 1].y, false, false);
          if (orow < n) *reinterpret_cast<u32x4*>(dst + 8 * (k + g)) = u32x4{x[0], y[0], x[1], y[1]};
        }
      }
    }
  }
  if (!score) return;
  const int split = (h - hk * group) * a.n_row_tiles + rt;
  float* const part = in_set_of(a.partial, a.g, li) + (size_t)hk * a.partial_stride + (size_t)split * a.cand_stride;
  // keys that none of this workgroup's rows see: zeros (the selection adds every partial array)
  for (int k = 32 * (n_kb - c_blk) + tid; k < a.n_keys; k += S::kThreads) part[c + k] = 0.f;

  // ---- column sums (Eq. 4) of the workgroup's rows, from the weights in registers: a lane's factor brings those of its row
  // onto the final normaliser, and the sums run over the lanes
  const int kept_r = 8 * ((lane >> 4) & 1) + 4 * ((lane >> 3) & 1) + 2 * ((lane >> 2) & 1) + ((lane >> 1) & 1);
  const int my_key = 8 * (kept_r >> 2) + 4 * g + (kept_r & 3);               // this lane's, and its neighbour's
  auto kept_sum = [&](int i, float lse_row) __attribute__((always_inline)) {
    if (q0 + 32 > n && q0 + l32 >= n) {      // a row past the end of the block
#pragma unroll
      for (int e = 0; e < 16; ++e) kept[i][e] = 0.f;
      kept_m[i] = -INFINITY;
    }
    return sum_over_half(kept[i], __builtin_amdgcn_exp2f(__builtin_fmaf(kept_m[i], sl2, -lse_row)), lane);    // (0 where the wave saw nothing)
  };
  // A row's factor has to leave the weight 0 of a key that the row does not see.  Where the normaliser of some row is not finite, or
  // so large that its rounding alone could make the factor infinite, the weights are brought onto the normalisers here, key by
  // key, and the factors are 1.  (Out of the way of the others, which pay for the question: 0.3 % of a launch of 8 to 11 us.)
  auto settle_odd_rows = [&](float& lse_row) __attribute__((always_inline)) {
    if (__builtin_expect(__all(__builtin_fabsf(lse_row) < 0x1p30f), 1)) return;
#pragma unroll
    for (int i = 0; i < kKept; ++i) {
      if (i >= my_blk) continue;
      const Block b = mine(i);
      float f = __builtin_amdgcn_exp2f(__builtin_fmaf(kept_m[i], sl2, -lse_row));
      f = f > __FLT_MAX__ ? __FLT_MAX__ : f;               // (a NaN stays one)
      const int last = b.cached ? 31 : q0 + l32 + shift - b.first;           // of the block's keys, the last that the row sees
#pragma unroll
      for (int e = 0; e < 16; ++e) kept[i][e] = 8 * (e >> 2) + 4 * g + (e & 3) <= last ? kept[i][e] * f : 0.f;
      kept_m[i] = 0.f;
    }
    lse_row = 0.f;
  };
  if constexpr (kKept > 0 && QW == 1) {
    settle_odd_rows(lse_row);
#pragma unroll
    for (int i = 0; i < kKept; ++i) {
      if (i >= my_blk) continue;
      const float tot = kept_sum(i, lse_row);
      const Block b = mine(i);
      if ((lane & 1) == 0 && my_key < b.rows) part[(b.cached ? 0 : c) + b.first + my_key] = tot;
    }
    return;
  }

  // ---- second sweep: column sums (Eq. 4) of the workgroup's rows; wave w takes key blocks w, w + 8, ...,
  // its two strips in turn
  __syncthreads();                           // the rows' statistics are in LDS, the partial outputs have been read
  constexpr int kFirst = kKept > 0 ? kKept * KS : 0;       // (two row tiles: those before it are in registers)
  const Tensors keys = {kc, kn, nullptr, nullptr, n_kb};
  feed_at(feed, keys, kFirst + wave, S::kWaves, No{});
  feed_lanes(feed, No{}, true);
  load_all(feed, feed.k, feed.k_lane, lds_addr(k_strip), ~0u);
  if constexpr (kKept > 0) {
    settle_odd_rows(lse_row);
#pragma unroll
    for (int i = 0; i < kKept; ++i) {
      const float tot = i < my_blk ? kept_sum(i, lse_row) : 0.f;
      if ((lane & 1) == 0) kept_lds[(wave * kKept + i) * 32 + my_key] = tot;
    }
    __syncthreads();
    for (int t = tid; t < kFirst * 32; t += S::kThreads) {
      const int b = t / 32, at = ((b % KS) * kKept + b / KS) * 32 + t % 32;
      const Block kb = block_of(b);
      if (b < n_kb && t % 32 < kb.rows) part[(kb.cached ? 0 : c) + kb.first + t % 32] = kept_lds[at] + kept_lds[KS * kKept * 32 + at];
    }
  }
  bf16x8 qs[QW][kNK];
#pragma unroll
  for (int t = 0; t < QW; ++t)
#pragma unroll
    for (int st = 0; st < kNK; ++st) qs[t][st] = lds_read_b128(q_lds + t * S::kStrip + k_off[st]);
  float ls[QW][16];                          // register r is row 8 (r / 4) + 4 g + r % 4 of its tile
#pragma unroll
  for (int t = 0; t < QW; ++t)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(&lse_lds[32 * t + 8 * j + 4 * g]);
#pragma unroll
      for (int e = 0; e < 4; ++e) ls[t][4 * j + e] = v[e];
    }
  // The wave's blocks from b up to `end`, by row tiles T0 .. QW - 1 (those before T0 see none of them); returns its first
  // block after those.  (No software pipeline: with the exponentials of one block among the matrix instructions of the
  // next it was a few per cent slower; the two waves of a SIMD fill each other's gaps.)
  int turn = 0;                              // which strip holds the block
  auto sweep = [&](int from, int end, auto tiles_from) __attribute__((always_inline)) -> int {
    constexpr int T0 = decltype(tiles_from)::value;
    int at = from;
    for (; at < end; at += S::kWaves, ++turn) {
      // (wave-uniform, which the compiler does not see through two loops in a row)
      const int b = __builtin_amdgcn_readfirstlane(at), odd = __builtin_amdgcn_readfirstlane(turn) & 1;
      u16* const strip = k_strip + odd * S::kWaves * S::kStrip;          // k_strip or v_strip
      feed_on(feed, keys, b + S::kWaves, S::kWaves, No{}, true);
      load_all(feed, feed.k, feed.k_lane, lds_addr(k_strip + (1 - odd) * S::kWaves * S::kStrip), ~0u);
      wait_older_than(OneBlock{});
      bf16x8 kf[kNK];
#pragma unroll
      for (int st = 0; st < kNK; ++st) kf[st] = lds_read_b128(strip + k_off[st]);
      f32x16 s[QW];
#pragma unroll
      for (int st = 0; st < kNK; ++st)
#pragma unroll
        for (int t = T0; t < QW; ++t)
          s[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qs[t][st], kf[st], st == 0 ? zero : s[t], 0, 0, 0);
      __builtin_amdgcn_s_setprio(1);
      const Block kb = block_of(b);
      float sum[2] = {0.f, 0.f};
      // every row sees every key and all are real
      if (kb.rows == 32 && (kb.cached || kb.first + 31 <= tile_row(T0) + shift) && tile_row(QW - 1) + 32 <= n) {
#pragma unroll
        for (int t = T0; t < QW; ++t)
#pragma unroll
          for (int r = 0; r < 16; ++r) sum[r & 1] += __builtin_amdgcn_exp2f(__builtin_fmaf(s[t][r], sl2, -ls[t][r]));
      } else {
        // this lane's key counts for the row at offset off = 8 (r / 4) + r % 4 from row0 iff first <= off < rows left
#pragma unroll
        for (int t = T0; t < QW; ++t) {
          const int row0 = tile_row(t) + 4 * g;
          const int first = kb.cached ? 0 : max(kb.first + l32 - shift - row0, 0);
          const unsigned span = (unsigned)max(n - row0 - first, 0);
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[t][r], sl2, -ls[t][r]));
            sum[r & 1] += (unsigned)(8 * (r >> 2) + (r & 3) - first) < span ? p : 0.f;
          }
        }
      }
      const float tot = sum_with_other_half(sum[0] + sum[1]);  // lanes l and l + 32 hold the two halves of the rows
      if (g == 0 && l32 < kb.rows) part[(kb.cached ? 0 : c) + kb.first + l32] = tot;
      __builtin_amdgcn_s_setprio(0);
    }
    return at;
  };
  if constexpr (QW == 1) {
    sweep(kFirst + wave, n_kb, std::integral_constant<int, 0>{});
  } else {
    // blocks that rows of both tiles see, then those that only the late tile's do
    const int n_both = c_blk + (min(a.n_keys, min(n, tile_row(0) + 32) + shift) + 31) / 32;
    const int b = sweep(kFirst + wave, min(n_both, n_kb), std::integral_constant<int, 0>{});
    sweep(b, n_kb, std::integral_constant<int, 1>{});
  }
  wait_older_than(None{});                   // no load into LDS outlives the workgroup
}

template <int D, int QW, int kKept>
hipError_t launch_shape(const AttnArgs& a, hipStream_t s) {
  using S = Split<D, QW>;
  hipLaunchKernelGGL((attention_split_kernel<D, QW, kKept>), dim3(kXcds * a.work_per_xcd + a.key_score_wgs, a.g.n_layers), dim3(S::kThreads),
                     S::kLdsBytes, s, a);
  return hipGetLastError();
}

template <int D, int QW, int kKept>
hipError_t prepare_shape() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(attention_split_kernel<D, QW, kKept>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, Split<D, QW>::kLdsBytes);
}

// 32-row workgroups: as many kept blocks per wave as the list needs, where registers have room for them (d 128: all 256
// with six; d 64: 228 with eight).  A launch without scores keeps none.
template <int D>
hipError_t launch_split32(const AttnArgs& a, hipStream_t s) {
  if (a.key_score_wgs > 0) return launch_shape<D, 1, kScoreByKeys>(a, s);
  const int blocks = (a.c + 31) / 32 + (a.n_keys + 31) / 32;
  const int need = a.partial != nullptr ? (blocks + Split<D, 1>::KS - 1) / Split<D, 1>::KS : 0;
  if (need >= 1 && need <= 2) return launch_shape<D, 1, 2>(a, s);
  if (need == 3) return launch_shape<D, 1, 3>(a, s);
  if (need == 4) return launch_shape<D, 1, 4>(a, s);
  if (need == 5) return launch_shape<D, 1, 5>(a, s);
  if (need == 6) return launch_shape<D, 1, 6>(a, s);
  if constexpr (D == 64) {
    if (need == 7 || need == 8) return launch_shape<D, 1, 8>(a, s);
  }
  return launch_shape<D, 1, 0>(a, s);
}
template <int D>
hipError_t launch_split64(const AttnArgs& a, hipStream_t s) {
  if (a.key_score_wgs > 0) return launch_shape<D, 2, kScoreByKeys>(a, s);
  return a.partial != nullptr ? launch_shape<D, 2, kKeptRounds<D, 2>>(a, s) : launch_shape<D, 2, 0>(a, s);
}
template <int D>
hipError_t prepare_split32() {
  hipError_t e;
  if ((e = prepare_shape<D, 1, 0>()) != hipSuccess) return e;
  if ((e = prepare_shape<D, 1, kScoreByKeys>()) != hipSuccess) return e;
  if ((e = prepare_shape<D, 1, 2>()) != hipSuccess) return e;
  if ((e = prepare_shape<D, 1, 3>()) != hipSuccess) return e;
  if ((e = prepare_shape<D, 1, 4>()) != hipSuccess) return e;
  if ((e = prepare_shape<D, 1, 5>()) != hipSuccess) return e;
  if ((e = prepare_shape<D, 1, 6>()) != hipSuccess) return e;
  if constexpr (D == 64) e = prepare_shape<D, 1, 8>();
  return e;
}

}  // namespace

hipError_t prepare_attention_split() {
  hipError_t e;
  if ((e = prepare_split32<128>()) != hipSuccess) return e;
  if ((e = prepare_split32<64>()) != hipSuccess) return e;
  if ((e = prepare_shape<128, 2, 0>()) != hipSuccess) return e;
  if ((e = prepare_shape<128, 2, kKeptRounds<128, 2>>()) != hipSuccess) return e;
  if ((e = prepare_shape<64, 2, kKeptRounds<64, 2>>()) != hipSuccess) return e;
  if ((e = prepare_shape<128, 2, kScoreByKeys>()) != hipSuccess) return e;
  if ((e = prepare_shape<64, 2, 0>()) != hipSuccess) return e;
  return prepare_shape<64, 2, kScoreByKeys>();
}

hipError_t launch_attention_split(const AttnArgs& a, int head_dim, hipStream_t s) {
  if (head_dim == 128) return a.variant == kAttnSplit32 ? launch_split32<128>(a, s) : launch_split64<128>(a, s);
  return a.variant == kAttnSplit32 ? launch_split32<64>(a, s) : launch_split64<64>(a, s);
}

}  // namespace kvp
