// Attention of one block of queries over cache U block (Eq. 1 of the paper),
// for gfx950: bf16 MFMA 32x32x16, wave64, K and V tiles staged through LDS.
//
// Formulation.  Every wave owns QT tiles of 32 query rows and works on the
// TRANSPOSED problem: S^T = K Q^T (A operand = K tile from LDS, B operand = Q
// held in registers for the whole kernel) and O^T = V^T P^T (A operand = V^T
// from LDS, B operand = P^T).  In the 32x32 accumulator layout a lane holds one
// column, so with the transposed problem a lane holds ONE query row: the
// softmax reference and the running sum are one scalar per lane, and the
// exponentiated S^T accumulators are, register for register, the B operand of
// the second product.  P never touches LDS and is never shuffled between lanes.
//
// The contraction index of an MFMA may be permuted freely as long as A and B
// agree.  For O^T the index is the key position: accumulator register r of lane
// (g = lane / 32) holds key  8 (r / 4) + 4 g + r % 4  of the 32-key block, so
// registers 8 m .. 8 m + 7 are fed to MFMA m of the block, and the V^T operand
// is gathered in exactly that key order.
//
// Staging.  K and V tiles go from global memory straight into LDS
// (buffer_load ... lds through descriptors that move on by a tile; global_load_lds where a tile straddles
// the cache and the block or ends past the last key; 16 bytes per lane, no registers, no LDS store
// instructions), row-major as they are in memory.  A wave instruction fills
// 1 KiB of consecutive LDS, so rows cannot be padded; instead the 16-byte chunks
// of a row are XOR-swizzled by the row number on the way in, each tensor with
// the pattern that makes its own fragment reads conflict-free.  The K operand is
// one ds_read_b128 per fragment; the V^T operand is two ds_read_b64_tr_b16:
// within 16 lanes, lane j receives element j % 4 of the 8-byte chunks addressed
// by lanes j / 4, j / 4 + 4, j / 4 + 8, j / 4 + 12, i.e. four keys of one channel.
//
// A workgroup is QW x KS waves: QW groups of query rows times a KS-way split of
// every staged key tile.  A wave takes 64 keys of each tile as two 32-key
// blocks X and Y; the KS partial results of a row are merged through LDS at the
// end.  The split keeps all 1024 SIMDs busy when a block of the prefix has
// fewer than 1024 wave-sized row tiles.  The library picks 4 x 2 waves of 32 rows (two
// waves per SIMD, 256 registers each); blocks too small to fill the chip with its 128-row workgroups
// go to attention_split.hip.  2 x 2 waves of 64 rows (one wave per SIMD, 512 registers) and 2 x 2 waves of 32 rows
// run where a caller forces them (kvp_set_attention_shape).
//
// Schedule.  Matrix and vector work of one wave are made to overlap in program
// order.  With S_X(t) = scores of block X of tile t, the loop body is
//   phase 1   MFMA: S_Y(t), O += P_Y(t-1) V     | VALU: P_X(t) = exp(S_X(t) - m)
//   barrier
//   phase 2   MFMA: S_X(t+1), O += P_X(t) V     | VALU: P_Y(t) = exp(S_Y(t) - m)
//             and, first thing after the barrier, the loads of K(t+2) and
//             V(t+1) into the buffers whose last readers were in phase 1.
// LDS holds two K tiles and two V tiles; one barrier per tile is enough because
// a buffer is only overwritten in the phase after its last reader.  The first K fragments of a phase 1 are read at
// the end of the phase before it.
//
// What stands between the products is kept out of the loop: the tiles come through descriptors that move on by a tile, a load's
// place in its tile is a scalar, and how many tiles go which way is worked out once (as a search, tile by tile, it took 4500 of a
// workgroup's 115,000 cycles).  A plain tile takes 2640 cycles, 41 for each matrix instruction of a SIMD, of which the pipe needs 33 (2940 with
// 110 scalar instructions a tile; 1.80 instead of 1.92 us; a tile with a mask 448 instructions instead of 587).  32/8 heads, d 128, 1024 rows over 3072 keys, one
// layer: 57.0 -> 53.9 us without scores, 78 -> 75 us with them.  The clock gives part of it back: with
// ordinary data launches of 16 layers run at 1.6 to 1.9 of 2.4 GHz (zeros for data, one layer: 46.6 -> 42.6 and 59.2 -> 55.5 us).
//
// Softmax reference.  exp(S - m) is exact for ANY per-row reference m as long as
// nothing overflows, so the fast loop fixes m at the maximum of the row's first
// visible block and never touches O again: no rescaling, no branch.  Every block
// maximum is still computed; should one exceed m by more than 2^64 (fp32 would
// overflow near 2^127) the workgroup raises a flag, throws its result away and
// redoes its rows with the textbook online softmax in a plain loop.  Real
// attention logits never get there; adversarial inputs stay correct.
//
// Layers.  One launch takes the block of up to sixteen layers (grid y), for callers that have them
// all in hand (kvp_prefill_block).  One layer's block is 96 to 256 workgroups, a single round of the
// chip at best: every launch pays the dispatch, the first tiles and the wait for its slowest
// workgroup, and small blocks leave CUs idle.  Per layer, scores included: 74 -> 68 us at 32/8 heads, d 128,
// 1024 rows over 3072 keys (16 layers per launch).
#include <type_traits>

#include "key_tiles.h"
#include "kvp_internal.h"
#include "mfma_tools.h"

namespace kvp {

namespace {

constexpr float kRedoLog2 = 64.f;   // redo a row tile when a block maximum exceeds the reference by 2^64

template <int D, int QT, int QW, int KS>
struct Shape {
  static constexpr int kWaves = QW * KS;
  static constexpr int kThreads = 64 * kWaves;
  static constexpr int kRows = QW * QT * 32;          // query rows per workgroup
  static constexpr int kTk = KS * 64;                 // keys per staged tile
  static constexpr int kChunks = D / 8;               // 16-byte chunks per row
  static constexpr int kRowsPerLoad = 64 / kChunks;   // rows one wave instruction brings in
  static constexpr int kRowGroup = kWaves * kRowsPerLoad;  // rows the waves bring in per step
  static constexpr int kLoadsPerWave = kTk / kRowGroup;            // per tensor and tile
  static constexpr int kTile = kTk * D;               // bf16 elements of a K or V tile, unpadded
  static constexpr int kTileBytes = 4 * kTile * 2;    // two K and two V buffers
  // at the end of the tile buffers, when the tiles are done with: the finished row statistics of the workgroup's
  // rows for the score sweep, and before them a word per wave (does it want its rows redone)
  static constexpr int kScoreBytes = QW * QT * 32 * 4;
  static constexpr int kFlagBytes = kWaves * 4;
  // in the K buffers what the waves leave for each other of their partial results, and the key strips of the score sweep, one block
  // of 32 keys per wave; at the front of the V buffers the waves' row maxima and sums and the half rows that they store
  static constexpr int kStrip = 32 * D;
  static_assert(kWaves * QT * kStrip * 2 <= kTileBytes / 2, "what the waves leave for each other");
  static_assert(kWaves * QT * 64 * 4 + kWaves * 32 * D + kScoreBytes + kFlagBytes <= kTileBytes / 2, "statistics and rows");
  static constexpr int kQBytes = kRows * D * 2;       // behind the tiles: the workgroup's query rows, for both sweeps
  static constexpr int kLdsBytes = kTileBytes + kQBytes;
  static_assert(kLdsBytes <= 160 * 1024, "LDS of a CU");
  static_assert(kWaves == 4 || kWaves == 8, "four or eight waves per workgroup");
  static_assert(kTk == 128, "the staging map assumes 128-key tiles");
};

template <int D, int QT, int QW, int KS>
__global__ void __launch_bounds__((Shape<D, QT, QW, KS>::kThreads))
attention_kernel(const AttnArgs args) {
  using S = Shape<D, QT, QW, KS>;
  constexpr int kThreads = S::kThreads;
  extern __shared__ __align__(16) unsigned char lds_raw[];
  u16* const lds_k = reinterpret_cast<u16*>(lds_raw);              // [2][kTile]
  u16* const lds_v = lds_k + 2 * S::kTile;                         // [2][kTile]
  u16* const q_lds = lds_v + 2 * S::kTile;                         // [QW][QT][32][D], chunks swizzled like K's
  float* const lse_lds = reinterpret_cast<float*>(lds_raw + S::kTileBytes - S::kScoreBytes);   // [QW][QT][32]
  unsigned* const flag_lds = reinterpret_cast<unsigned*>(lse_lds) - S::kWaves;

  const int li = blockIdx.y;                         // layer of the group
  AttnPlan a = args;
  const u16* const q_rows = args.layer[li].q;
  u16* const out_rows = args.layer[li].out;
  have_arguments(q_rows, out_rows, args.layer[li].k_new, args.layer[li].v_new, a.k_cache, a.v_cache, a.lse2, a.partial, a.g.first_set,
                 a.g.n_sets, a.g.set_stride, a.g.kv_stride, a.n, a.c, a.work_per_xcd, a.total_work, a.tiles_magic, a.group_magic,
                 a.tiles_shift, a.group_shift);
  // (a whole prefix of 32/8 heads, d 128, 1024 rows over 3072 keys, a layer per launch 30192 -> 30124 us)
  keep_arguments(a.n_q_heads, a.n_kv_heads, a.n_keys, a.n_row_tiles, a.budget, a.shift, a.group, a.scale_log2, a.lse_stride,
                 a.partial_stride, a.cand_stride);
  // XCD-aware order: consecutive work items (same KV head) land on one die
  const int xcd = blockIdx.x % kXcds;
  const int w = xcd * a.work_per_xcd + blockIdx.x / kXcds;
  if (w >= a.total_work) return;
  float* const lse2 = in_set_of(a.lse2, a.g, li);
  const int group = a.group;
  const int h = (int)quotient((unsigned)w, Divisor{a.tiles_magic, a.tiles_shift});
  const int rt = a.n_row_tiles - 1 - (w - h * a.n_row_tiles);    // long rows first
  const int hk = (int)quotient((unsigned)h, Divisor{a.group_magic, a.group_shift});

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  // the same number in a scalar register: what a wave derives from it (its rows, its tile counts,
  // its branches, addresses of its loads) is then uniform for the compiler as well
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);
  const int qw = wave_s / KS;
  const int ks = wave_s % KS;
  const int l32 = lane & 31;
  const int g = lane >> 5;

  const int n = a.n, c = a.c, n_cand = c + a.n_keys, shift = a.shift;
  // Rows.  A head's rows are cut into blocks of QT * 32 (one per group of KS waves); later rows
  // see more of the block's keys.  A workgroup takes QW / 2 blocks from the front of the head
  // and QW / 2 from the back, so every workgroup has the same amount of work; and since waves w
  // and w + 4 of a workgroup share a SIMD, every SIMD of the eight-wave shape gets one early and
  // one late block: when the early one has run out of visible keys the late one has the SIMD to
  // itself.  first_row_of(q) is the first row of the block the waves with qw = q work on.
  auto first_row_of = [&](int q) __attribute__((always_inline)) -> int {
    constexpr int kHalf = QW / 2;
    const int blocks = a.n_row_tiles * QW;
    const int b = q < kHalf ? rt * kHalf + q : blocks - (rt + 1) * kHalf + (q - kHalf);
    return b * QT * 32;
  };
  const int q0 = first_row_of(qw);                   // first query row of this wave
  // the workgroup as a whole: the last block is the latest; tiles are staged for everybody
  const int wg_rows_end = min(n, first_row_of(QW - 1) + QT * 32);
  const int n_tiles = (min(n_cand, c + wg_rows_end + shift) + S::kTk - 1) / S::kTk;
  // this wave: the tiles its rows can see, and those among them visible in full to all its rows
  const int my_rows_end = min(n, q0 + QT * 32);      // = n for a block that lies past the end: computed, not stored
  const int my_tiles = (min(n_cand, c + my_rows_end + shift) + S::kTk - 1) / S::kTk;
  const int n_plain = min(my_tiles, (min(c + q0 + shift + 1, n_cand)) / S::kTk);
  const u16* kc = a.k_cache + (size_t)li * a.g.kv_stride + (size_t)hk * a.budget * D;
  const u16* vc = a.v_cache + (size_t)li * a.g.kv_stride + (size_t)hk * a.budget * D;
  const u16* kn = args.layer[li].k_new + (size_t)hk * D;
  const u16* vn = args.layer[li].v_new + (size_t)hk * D;
  const int new_stride = a.n_kv_heads * D;
  const float sl2 = a.scale_log2;

  // ---- staging: global -> LDS, 16 bytes per lane, chunks swizzled by row.
  // Instruction j of wave w brings in rows kRowGroup j + kRowsPerLoad w + (0 .. kRowsPerLoad-1)
  // of the tile; a lane always handles the same row residue, so its swizzle is a constant.
  const int ld_sub = lane / S::kChunks, ld_pos = lane % S::kChunks;
  const int ld_row = S::kRowsPerLoad * wave + ld_sub;          // + kRowGroup j
  const int ld_chunk_k = ld_pos ^ (ld_row % S::kChunks);
  const int ld_chunk_v = ld_pos ^ v_swizzle<D>(ld_row);
  // LDS destination of instruction j into `tile`, as the byte address M0 wants: wave-uniform and
  // all scalar arithmetic (the wave number is read into a scalar register once)
  const unsigned lds_base =
      __builtin_amdgcn_readfirstlane((unsigned)(size_t)(__attribute__((address_space(3))) void*)lds_raw);
  auto lds_dst = [&](const u16* tile, int j) __attribute__((always_inline)) -> unsigned {
    return lds_base + 2u * (unsigned)((int)(tile - lds_k) + (S::kRowGroup * j + S::kRowsPerLoad * wave_s) * D);
  };
  // Issued as inline assembly on purpose: the compiler then does not know that these loads write
  // LDS and does not make every later LDS read wait for them.  Ordering is this kernel's job:
  // wait_loads() before the barrier that publishes a tile.
  // Three address forms: a 64-bit address per lane (tiles that straddle the cache and the block or
  // run past the end), a scalar base with a 32-bit offset per lane (key strips of the score sweep), and
  // a buffer descriptor (load_fed below: the uniform tiles, in the cache or in the block as a whole).
  auto load16 = [&](const u16* src, unsigned lds_addr) __attribute__((always_inline)) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(lds_addr)
                 : "m0", "memory");
  };
  auto load16_scalar_base = [&](const u16* base, unsigned lane_bytes, unsigned lds_addr) __attribute__((always_inline)) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(lane_bytes), "s"(base),
                 "s"(lds_addr)
                 : "m0", "memory");
  };
  auto wait_loads = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_s_waitcnt(0x0F70);    // vmcnt(0), nothing else
  };
  // A uniform tile: the scalar address of the first row this wave brings in, the row stride, and
  // which of the lane offsets goes with it.  The lane part of an address is
  // (ld_sub rows + the swizzled chunk) in bytes, one value per tensor and per stride.
  struct UniformSrc {
    const u16* base;
    int stride;
    bool cached;
  };
  auto uniform_src = [&](const u16* cache, const u16* fresh, int t) __attribute__((always_inline)) -> UniformSrc {
    const int base = t * S::kTk;
    const bool cached = base < c;
    const int stride = cached ? D : new_stride;
    const u16* p = cached ? cache + (size_t)base * D : fresh + (size_t)(base - c) * new_stride;
    return UniformSrc{p + (size_t)(S::kRowsPerLoad * wave_s) * stride, stride, cached};
  };
  const unsigned lane_k_cache = 2u * (unsigned)(ld_sub * D + 8 * ld_chunk_k);
  const unsigned lane_k_new = 2u * (unsigned)(ld_sub * new_stride + 8 * ld_chunk_k);
  const unsigned lane_v_cache = 2u * (unsigned)(ld_sub * D + 8 * ld_chunk_v);
  const unsigned lane_v_new = 2u * (unsigned)(ld_sub * new_stride + 8 * ld_chunk_v);
  auto issue_any_one = [&](const u16* cache, const u16* fresh, u16* tile, int t, int chunk, int j)
      __attribute__((always_inline)) {
    const int kv = min(t * S::kTk + S::kRowGroup * j + ld_row, n_cand - 1);   // past the end: any finite row
    const u16* src = kv < c ? cache + (size_t)kv * D : fresh + (size_t)(kv - c) * new_stride;
    load16(src + 8 * chunk, lds_dst(tile, j));
  };
  auto issue_any = [&](const u16* cache, const u16* fresh, u16* tile, int t, int chunk)
      __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < S::kLoadsPerWave; ++j) issue_any_one(cache, fresh, tile, t, chunk, j);
  };

  // ---- per-lane LDS read offsets (bf16 elements), swizzle folded in
  // K operand, d-slice st: row (block + l32), chunk (2 st + g) ^ (row % kChunks)
  int k_off[D / 16];
  {
    const int q = g ^ (l32 % S::kChunks);
#pragma unroll
    for (int st = 0; st < D / 16; ++st) k_off[st] = l32 * D + 8 * ((2 * st) ^ q);
  }
  // V^T operand, channel tile dt: this lane addresses key row 4 g + (lane % 16) / 4 (+ block + 16 mm
  // + 8 h) and the 8-byte half (lane % 4) & 1 of chunk 4 dt + 2 ((lane / 16) % 2) + (lane % 4) / 2
  int v_off[D / 32];
  {
    const int rsub = 4 * g + ((lane & 15) >> 2);
    const int z = v_swizzle<D>(rsub);
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt) {
      const int chunk = (4 * dt + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) ^ z;
      v_off[dt] = rsub * D + 8 * chunk + 4 * (lane & 1);
    }
  }

  // ---- the score sweep's key blocks, blocks of 32 keys that some row of the workgroup sees: they come in whole rows through a strip
  // of LDS of the wave's own, block i + 1 on its way into it while block i is worked on from registers.  (In operand layout straight from
  // memory they took a CU's address path at a quarter of its rate.  Statistics to the last sum, 32/8 heads, 1024 rows over 3072
  // keys: 27.3 -> 24.5 us, a quarter of that from the query rows that are there already; a prefill of 16640 tokens through 32
  // such layers 36.3 -> 35.1 ms.)
  const int n_kb = (min(n_cand, c + wg_rows_end + shift) + 31) / 32;
  u16* const k_strip = lds_k + wave_s * QT * S::kStrip;
  constexpr int kStripLoads = 32 / S::kRowsPerLoad;
  const int strip_chunk = ld_pos ^ ld_sub;             // of load 0; load j: bits of j where a row has 16 chunks
  const unsigned lane_cache = 2u * (unsigned)(ld_sub * D + 8 * strip_chunk);
  const unsigned lane_new = 2u * (unsigned)(ld_sub * new_stride + 8 * strip_chunk);
  auto load_keys = [&](int kbi) __attribute__((always_inline)) {
    const int kb0 = kbi * 32;
    const bool cached = kb0 + 32 <= c;
    if (cached || (kb0 >= c && kb0 + 32 <= n_cand)) {
      const int stride = cached ? D : new_stride;
      const u16* const base = cached ? kc + (size_t)kb0 * D : kn + (size_t)(kb0 - c) * new_stride;
      const unsigned lane_off = cached ? lane_cache : lane_new;
#pragma unroll
      for (int j = 0; j < kStripLoads; ++j)
        load16_scalar_base(base + (size_t)(S::kRowsPerLoad * j) * stride, lane_off ^ (16u * ((S::kRowsPerLoad * j) % S::kChunks)),
                           lds_base + 2u * (unsigned)((int)(k_strip - lds_k) + S::kRowsPerLoad * j * D));
    } else {
#pragma unroll
      for (int j = 0; j < kStripLoads; ++j) {
        const int kv = min(kb0 + S::kRowsPerLoad * j + ld_sub, n_cand - 1);      // past the end: any real row, never stored
        const u16* src = kv < c ? kc + (size_t)kv * D : kn + (size_t)(kv - c) * new_stride;
        load16(src + 8 * (strip_chunk ^ ((S::kRowsPerLoad * j) % S::kChunks)),
               lds_base + 2u * (unsigned)((int)(k_strip - lds_k) + S::kRowsPerLoad * j * D));
      }
    }
  };

  // ================================================================ fast path
  bool redo = false;
  {
    // ---- the workgroup's query rows, whole rows into LDS (they stay there for the second sweep), and the first
    // tiles behind them: one trip to memory for all.  (The fragments straight from memory in operand layout, where
    // neighbouring lanes read different rows, go through the CU's address path at a quarter of its rate, and the tiles
    // had to wait for them.)  Entry to the first tile's products at 32/8 heads, d 128, 1024 rows: 5.5 -> 4.6 us.
    constexpr int kQLoads = S::kRows / S::kRowGroup;
    static_assert(32 % S::kRowsPerLoad == 0 && S::kRows % S::kRowGroup == 0, "whole loads per row tile");
#pragma unroll
    for (int j = 0; j < kQLoads; ++j) {
      const int r0 = S::kRowGroup * j + S::kRowsPerLoad * wave_s;        // first row of this load; 32-row tiles in a row
      const int ti = r0 / 32, r = r0 % 32 + ld_sub;
      const int row = min(first_row_of(ti / QT) + 32 * (ti % QT) + r, n - 1);   // rows past the block are computed, not stored
      load16(q_rows + ((size_t)row * a.n_q_heads + h) * D + 8 * (ld_pos ^ (r % S::kChunks)),
             lds_base + 2u * (unsigned)((int)(q_lds - lds_k) + r0 * D));
    }
    issue_any(kc, kn, lds_k, 0, ld_chunk_k);
    issue_any(vc, vn, lds_v, 0, ld_chunk_v);
    issue_any(kc, kn, lds_k + S::kTile, 1, ld_chunk_k);
    bf16x8 qf[QT][D / 16];        // Q fragments: B operand, lane holds Q[q0 + 32 t + l32][16 s + 8 g .. + 7]
    f32x16 o[QT][D / 32];
    float m_ref[QT], l_run[QT];
#pragma unroll
    for (int t = 0; t < QT; ++t) {
      m_ref[t] = -INFINITY;
      l_run[t] = 0.f;
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[t][dt][r] = 0.f;
    }
    const float redo_raw = kRedoLog2 / sl2;       // the margin in units of the raw dot product
    const int blk_off = 64 * ks * D;               // this wave's 64 keys inside a tile

    // Hide block keys a row may not see, fix the reference at the first visible block, and
    // watch for a block maximum far above the reference.
    // `track` is off for the tiles after the first plain one: every row has its reference by
    // then, and a logit far above it shows up in the row sum instead (checked after the loop).
    auto prepare = [&](f32x16 (&s)[QT], int kb, auto mask, auto track) __attribute__((always_inline)) {
#pragma unroll
      for (int t = 0; t < QT; ++t) {
        if constexpr (decltype(mask)::value) {
          // key kb + 8 (r / 4) + 4 g + r % 4 is visible when cached, or a block key not after the row
          const int lim = min(q0 + 32 * t + l32 + shift + c, n_cand - 1) - kb - 4 * g;
#pragma unroll
          for (int r = 0; r < 16; ++r) s[t][r] = (8 * (r >> 2) + (r & 3) <= lim) ? s[t][r] : -INFINITY;
        }
        if constexpr (decltype(track)::value) {
          float v = s[t][0];
#pragma unroll
          for (int r = 1; r < 16; ++r) v = fmaxf(v, s[t][r]);
          const float mx = max_with_other_half(v);
          m_ref[t] = (m_ref[t] == -INFINITY) ? mx : m_ref[t];
          redo |= mx > m_ref[t] + redo_raw;
        }
      }
    };

    // One phase, as one basic block: MFMA i is followed by the exponentials of 128 / D elements
    // of the S block computed in the previous phase, and LDS fragment reads run kAhead operands
    // ahead of their use.  The source is written in exactly that order and a scheduling fence after
    // every MFMA's share keeps the compiler from regrouping it (left to itself it bunches the
    // MFMAs and piles the exponentials up behind them).
    //   s_exp -> p_out   P = exp2((S - m) * scale) for the block whose scores are ready
    //   s_new            S^T of the next block = K[kt rows] Q^T
    //   p_pend, vt       O^T += V^T P^T for the block exponentiated one phase ago
    //   first            the first K fragments, read already where kHave; with kNext those of the next phase at the end
    constexpr int kAhead = D / 32;
    bf16x8 first[kAhead];
    auto phase_core = [&](const f32x16 (&s_exp)[QT], unsigned (&p_out)[QT][8], f32x16 (&s_new)[QT],
                          const u16* kt, const unsigned (&p_pend)[QT][8], const u16* vt, auto have, auto next, const u16* next_kt,
                          auto&& after_mfma) __attribute__((always_inline)) {
      constexpr bool kHave = decltype(have)::value, kNext = decltype(next)::value;
      constexpr int kNK = D / 16;            // K fragments
      constexpr int kNV = (D / 32) * 2;      // V^T fragments
      float neg[QT], sum[QT];
#pragma unroll
      for (int t = 0; t < QT; ++t) {
        const float m_use = (m_ref[t] == -INFINITY) ? 0.f : m_ref[t];   // row has seen nothing yet
        neg[t] = -m_use * sl2;
        sum[t] = 0.f;
      }
      bf16x8 kfr[kNK], vfr[kNV];
      auto read_k = [&](int st) __attribute__((always_inline)) { kfr[st] = lds_read_b128(kt + k_off[st]); };
      auto read_v = [&](int vi) __attribute__((always_inline)) {
        vfr[vi] = lds_read_vt(vt + v_off[vi / 2] + 16 * (vi % 2) * D, 8 * D);
      };
      // The vector work of an element is a chain (scale-and-shift, exponential, add to the row sum,
      // pack) and an instruction that needs the result of the one before it stalls the wave, the
      // exponential most of all.  So the chain is skewed over the MFMAs: each call computes the
      // argument of the next element, the exponential of this one, and adds and packs the one before.
      constexpr int kElems = QT * 16, kMfmas = QT * (kNK + kNV);
      int ei = 0;   // next element to exponentiate
      float arg = __builtin_fmaf(s_exp[0][0], sl2, neg[0]), pe1 = 0.f, pe2 = 0.f;
      auto finish_element = [&](int e) __attribute__((always_inline)) {      // element e: pe1, the one before: pe2
        const int t = e / 16, r = e % 16;
        sum[t] += pe1;
        // the sums are only needed after the loop, and left alone the compiler gathers the
        // additions of several phases in one place, keeping every exponential alive until then
        asm volatile("" : "+v"(sum[t]));
        if (r & 1) p_out[t][r >> 1] = pack_bf16(pe2, pe1);
      };
      auto exp_until = [&](int end) __attribute__((always_inline)) {
#pragma unroll
        for (; ei < end; ++ei) {
          const float pe = __builtin_amdgcn_exp2f(arg);
          if (ei + 1 < kElems) arg = __builtin_fmaf(s_exp[(ei + 1) / 16][(ei + 1) % 16], sl2, neg[(ei + 1) / 16]);
          if (ei >= 1) finish_element(ei - 1);
          pe2 = pe1;
          pe1 = pe;
        }
      };
      const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int st = 0; st < kAhead; ++st) {
        if constexpr (kHave) kfr[st] = first[st];
        else read_k(st);
      }
      __builtin_amdgcn_sched_barrier(0);     // all of them before the first MFMA
      auto share = [&](int i) __attribute__((always_inline)) { exp_until(kElems * (i + 1) / kMfmas); };    // of MFMA i
#pragma unroll
      for (int st = 0; st < kNK; ++st) {
        if (st + kAhead < kNK) read_k(st + kAhead);
        else read_v(st + kAhead - kNK);
#pragma unroll
        for (int t = 0; t < QT; ++t) {
          s_new[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kfr[st], qf[t][st], st == 0 ? zero : s_new[t], 0, 0, 0);
          share(st * QT + t);
          after_mfma(std::integral_constant<int, 0>{}, st * QT + t);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
#pragma unroll
      for (int vi = 0; vi < kNV; ++vi) {
        if (vi + kAhead < kNV) read_v(vi + kAhead);
        else if constexpr (kNext) first[vi + kAhead - kNV] = lds_read_b128(next_kt + k_off[vi + kAhead - kNV]);
        const int dt = vi / 2, mm = vi % 2;
#pragma unroll
        for (int t = 0; t < QT; ++t) {
          const u32x4 pw = {p_pend[t][4 * mm], p_pend[t][4 * mm + 1], p_pend[t][4 * mm + 2], p_pend[t][4 * mm + 3]};
          o[t][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vfr[vi], __builtin_bit_cast(bf16x8, pw), o[t][dt], 0, 0, 0);
          share((kNK + vi) * QT + t);
          after_mfma(std::integral_constant<int, 1>{}, vi * QT + t);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      finish_element(kElems - 1);
#pragma unroll
      for (int t = 0; t < QT; ++t) l_run[t] += sum[t];
    };

    // ---- prologue: Q and K(0) in LDS, S_X(0) computed (V(0) and K(1) may still be on their way: the first
    // body waits for them)
    f32x16 sx[QT], sy[QT];
    unsigned px[QT][8], py[QT][8];
#pragma unroll
    for (int t = 0; t < QT; ++t)
#pragma unroll
      for (int r = 0; r < 8; ++r) { px[t][r] = 0u; py[t][r] = 0u; }
    // V buffer 1 is read as "V(-1)" with P = 0 in the first phase: make it finite
    for (int i = tid; i < S::kTile / 8; i += kThreads)
      reinterpret_cast<u32x4*>(lds_v + S::kTile)[i] = u32x4{0u, 0u, 0u, 0u};
    static_assert(2 * S::kLoadsPerWave < 32, "fits the two fields of the wait");
    __builtin_amdgcn_s_waitcnt(0x0F70 | (2 * S::kLoadsPerWave & 15) | (2 * S::kLoadsPerWave >> 4 << 14));
    __syncthreads();
#pragma unroll
    for (int t = 0; t < QT; ++t)
#pragma unroll
      for (int s = 0; s < D / 16; ++s) qf[t][s] = lds_read_b128(q_lds + (qw * QT + t) * 32 * D + k_off[s]);
    {
      // S_X(0) without anything to overlap with
#pragma unroll
      for (int t = 0; t < QT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) sx[t][r] = 0.f;
#pragma unroll
      for (int st = 0; st < D / 16; ++st) {
        const bf16x8 ka = lds_read_b128(lds_k + blk_off + k_off[st]);
#pragma unroll
        for (int t = 0; t < QT; ++t) sx[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, qf[t][st], sx[t], 0, 0, 0);
      }
    }

    // The steady-state tiles that this wave brings in come through descriptors that move on by a tile at a time: K of tile t + 2 and V of
    // tile t + 1, in the cache or among the block's rows.  A load has its place in the tile in a scalar register.
    struct TileFeed {
      u32x4 buffer;
      unsigned lane, group_bytes;            // the lane's part of an address; bytes from a load's rows to the next load's
    };
    auto feed_at = [&](const u16* cache, const u16* fresh, unsigned lane_cache, unsigned lane_new, int t) __attribute__((always_inline)) -> TileFeed {
      const UniformSrc src = uniform_src(cache, fresh, t);
      const unsigned long long base = (unsigned long long)src.base;
      return TileFeed{u32x4{(unsigned)base, (unsigned)(base >> 32) & 0xFFFFu, 0xFFFFFFFFu, 0x00020000u}, src.cached ? lane_cache : lane_new,
                      2u * (unsigned)(S::kRowGroup * src.stride)};
    };
    auto move_on = [&](TileFeed& f) __attribute__((always_inline)) {
      const unsigned long long at = ((unsigned long long)f.buffer.y << 32 | f.buffer.x) + (unsigned long long)f.group_bytes * (S::kTk / S::kRowGroup);
      f.buffer.x = (unsigned)at;
      f.buffer.y = (unsigned)(at >> 32);
    };
    auto load_fed = [&](const TileFeed& f, int j, unsigned lds_addr) __attribute__((always_inline)) {
      asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds" ::"v"(f.lane), "s"(f.buffer),
                   "s"(f.group_bytes * (unsigned)j), "s"(lds_addr)
                   : "m0", "memory");
    };
    TileFeed k_feed, v_feed;

    // kTag = t & 1 as a compile-time constant in the steady-state loop, -1 for "use t & 1".
    // The steady-state loop also knows that the tiles it prefetches are uniform, and has the first K fragments of its first phase.
    auto body = [&](int t, auto buf_tag, auto fed, auto mask, auto track) __attribute__((always_inline)) {
      constexpr int kTag = decltype(buf_tag)::value;
      constexpr bool kSteady = kTag >= 0, kFed = decltype(fed)::value;
      const int buf = kTag >= 0 ? kTag : (t & 1);
      const int kb = t * S::kTk + ks * 64;
      u16* k_cur = lds_k + buf * S::kTile;
      u16* k_nxt = lds_k + (buf ^ 1) * S::kTile;
      u16* v_cur = lds_v + buf * S::kTile;
      u16* v_prv = lds_v + (buf ^ 1) * S::kTile;
      typedef std::integral_constant<bool, kSteady> Steady;
      // ---- phase 1: P_X(t), S_Y(t), O += P_Y(t-1) V(t-1)
      prepare(sx, kb, mask, track);
      phase_core(sx, px, sy, k_cur + blk_off + 32 * D, py, v_prv + blk_off + 32 * D, Steady{}, std::false_type{}, nullptr, [](auto, int) {});
      // P_X is only read in phase 2, and the compiler would gladly take its exponentials there,
      // all in a lump behind the barrier: make them due here, in the shadow of this phase's MFMAs
#pragma unroll
      for (int tq = 0; tq < QT; ++tq)
#pragma unroll
        for (int r = 0; r < 8; ++r) asm volatile("" ::"v"(px[tq][r]));
      __builtin_amdgcn_sched_barrier(0);
      wait_loads();               // the loads this wave issued in the last phase 2 have landed
      __syncthreads();
      // ---- phase 2: P_Y(t), S_X(t+1), O += P_X(t) V(t); the loads of K(t+2) and V(t+1) are spread
      // over the matrix instructions so that their issue does not stall the wave in one burst
      prepare(sy, kb + 32, mask, track);
      constexpr int kPerHalf = QT * (D / 16);              // MFMAs in each half of a phase
      constexpr int kEvery = kPerHalf / S::kLoadsPerWave;  // one load every kEvery MFMAs
      static_assert(kEvery >= 1 && kPerHalf % S::kLoadsPerWave == 0, "loads must fit the phase");
      // (behind the last fragments of this phase the first of the next one's, of the tile that the barrier has just published)
      phase_core(sy, py, sx, k_nxt + blk_off, px, v_cur + blk_off, std::false_type{}, Steady{}, k_nxt + blk_off + 32 * D,
                 [&](auto half, int i) __attribute__((always_inline)) {
                   if (i % kEvery != 0) return;
                   const int j = i / kEvery;
                   if constexpr (kFed) {
                     if (decltype(half)::value == 0) load_fed(k_feed, j, lds_dst(k_cur, j));
                     else load_fed(v_feed, j, lds_dst(v_prv, j));
                   } else {
                     if (decltype(half)::value == 0) issue_any_one(kc, kn, k_cur, t + 2, ld_chunk_k, j);
                     else issue_any_one(vc, vn, v_prv, t + 1, ld_chunk_v, j);
                   }
                 });
    };
    typedef std::integral_constant<int, 0> Even;
    typedef std::integral_constant<int, 1> Odd;
    typedef std::integral_constant<int, -1> Any;
    // The steady body of tile t needs the tiles that it prefetches (V of t + 1, K of t + 2) uniform, in the cache or in the block as a
    // whole, or past the workgroup's last tile (then it fetches an earlier tile again, into a buffer nobody reads any more).
    const int first_new = (c + S::kTk - 1) / S::kTk;
    int n_fed = min(my_tiles, fed_tiles(c, n_cand, S::kTk, n_tiles));      // tiles the steady bodies take
    if (new_stride >= 1 << 23) n_fed = 0;        // (bytes within a tile are 32-bit numbers)
    const int n_fast = min(n_plain, n_fed) & ~1;      // of these the ones that every row of the wave sees in full, two at a time
    // the feed of tile `t`: from the one before it, or, where the block's own rows begin, anew
    auto next_feed = [&](TileFeed& f, const u16* cache, const u16* fresh, unsigned lane_cache, unsigned lane_new, int t) __attribute__((always_inline)) {
      if (t >= n_tiles) return;
      if (t == first_new) f = feed_at(cache, fresh, lane_cache, lane_new, t);
      else move_on(f);
    };
    typedef std::true_type Yes;
    typedef std::false_type No;
    int t = 0;
    auto fed_body = [&](auto buf_tag, auto mask, auto track) __attribute__((always_inline)) {
      body(t, buf_tag, Yes{}, mask, track);
      ++t;
      next_feed(k_feed, kc, kn, lane_k_cache, lane_k_new, t + 2);
      next_feed(v_feed, vc, vn, lane_v_cache, lane_v_new, t + 1);
    };
    if (n_fed > 0) {
      k_feed = feed_at(kc, kn, lane_k_cache, lane_k_new, 2 < n_tiles ? 2 : 0);
      v_feed = feed_at(vc, vn, lane_v_cache, lane_v_new, 1 < n_tiles ? 1 : 0);
    }
    if (n_fast > 0) {
#pragma unroll
      for (int st = 0; st < kAhead; ++st) first[st] = lds_read_b128(lds_k + blk_off + 32 * D + k_off[st]);
      // tile 0 is plain: it gives every row its reference, and no plain tile after it looks at maxima
      fed_body(Even{}, No{}, Yes{});
      fed_body(Odd{}, No{}, No{});
    }
    while (t < n_fast) {
      fed_body(Even{}, No{}, No{});
      fed_body(Odd{}, No{}, No{});
    }
    while (t < n_fed) fed_body(Any{}, Yes{}, Yes{});       // masking a fully visible tile is harmless
    for (; t < my_tiles; ++t) body(t, Any{}, No{}, Yes{}, Yes{});
    {
      // O += P_Y V of this wave's last tile.  That V was published by the barrier inside the last
      // body and is overwritten only after the barrier of the next tile, which this wave has
      // not reached.
      const u16* vt = lds_v + ((my_tiles + 1) & 1) * S::kTile + blk_off + 32 * D;
#pragma unroll
      for (int vi = 0; vi < (D / 32) * 2; ++vi) {
        const int dt = vi / 2, mm = vi % 2;
        const bf16x8 va = lds_read_vt(vt + v_off[dt] + 16 * mm * D, 8 * D);
#pragma unroll
        for (int tq = 0; tq < QT; ++tq) {
          const u32x4 pw = {py[tq][4 * mm], py[tq][4 * mm + 1], py[tq][4 * mm + 2], py[tq][4 * mm + 3]};
          o[tq][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, __builtin_bit_cast(bf16x8, pw), o[tq][dt], 0, 0, 0);
        }
      }
    }
    // The workgroup's later tiles, which no row of this wave sees: keep in step with the others
    // (one barrier per tile) and bring in this wave's share of the tiles they read.
    for (; t < n_tiles; ++t) {
      wait_loads();
      __syncthreads();
      issue_any(kc, kn, lds_k + (t & 1) * S::kTile, t + 2, ld_chunk_k);
      issue_any(vc, vn, lds_v + ((t & 1) ^ 1) * S::kTile, t + 1, ld_chunk_v);
    }
    wait_loads();
    __syncthreads();               // nothing is on its way into LDS any more
    // a logit more than 2^64 above its row's reference in a tile that did not track maxima has
    // pushed the row sum past 2^64 (or to infinity or NaN)
#pragma unroll
    for (int tq = 0; tq < QT; ++tq) redo |= !(l_run[tq] <= 0x1p64f);
    if (__any(redo)) redo = true;
    if (lane == 0) flag_lds[wave] = redo ? 1u : 0u;
    // ---- merge the two partial results of every row through LDS and store it.  Of a row tile's two waves each finishes half of
    // the channels: it leaves its part of the other half with the other wave, as it lies in the accumulators.  Where a wave finds what
    // was left for it its key strip lies too: the first block of the score sweep is on its way while the rows are stored.
    // (One wave of the two with all of the channels, in single words, and the keys after that: 6870 cycles from the last tile to the
    // score sweep; this way 5500.)
    static_assert(KS == 2, "two waves to a row tile");
    constexpr int kHalf = D / 64;                // channel tiles of a half
    float* const stat_lds = reinterpret_cast<float*>(lds_v);     // [kWaves][QT][2][32]
    auto left_for = [&](int w, int tq, int k) __attribute__((always_inline)) {       // fours k of a half
      return reinterpret_cast<f32x4*>(lds_k + (w * QT + tq) * S::kStrip) + 64 * k + lane;
    };
    auto half_of = [&](int tq, int half, int k) __attribute__((always_inline)) -> f32x4 {
      const f32x16& x = o[tq][half * kHalf + k / 4];
      const int r = 4 * (k % 4);
      return f32x4{x[r], x[r + 1], x[r + 2], x[r + 3]};
    };
#pragma unroll
    for (int tq = 0; tq < QT; ++tq) {
      l_run[tq] = sum_with_other_half(l_run[tq]);            // lanes l and l + 32 each summed half of the keys of a row
#pragma unroll
      for (int k = 0; k < 4 * kHalf; ++k) {
        const f32x4 lo = half_of(tq, 0, k), hi = half_of(tq, 1, k);
        *left_for(wave_s ^ 1, tq, k) = ks == 0 ? hi : lo;
      }
      if (g == 0) {
        stat_lds[(wave_s * QT + tq) * 64 + l32] = m_ref[tq];
        stat_lds[(wave_s * QT + tq) * 64 + 32 + l32] = l_run[tq];
      }
    }
    __syncthreads();
    redo = false;                  // workgroup-uniform from here on
#pragma unroll
    for (int w2 = 0; w2 < S::kWaves; ++w2) redo |= flag_lds[w2] != 0u;

    if (!redo) {
      f32x4 sum[QT][4 * kHalf];
      float l_row[QT];
#pragma unroll
      for (int tq = 0; tq < QT; ++tq) {
        const float m_other = stat_lds[((wave_s ^ 1) * QT + tq) * 64 + l32], l_other = stat_lds[((wave_s ^ 1) * QT + tq) * 64 + 32 + l32];
        const float m0 = ks == 0 ? m_ref[tq] : m_other, m1 = ks == 0 ? m_other : m_ref[tq];
        const float mt = fmaxf(m0, m1), m_use = mt == -INFINITY ? 0.f : mt;
        const float f0 = __builtin_amdgcn_exp2f((m0 - m_use) * sl2), f1 = __builtin_amdgcn_exp2f((m1 - m_use) * sl2);
        l_row[tq] = (ks == 0 ? l_run[tq] : l_other) * f0;
        l_row[tq] += (ks == 0 ? l_other : l_run[tq]) * f1;
#pragma unroll
        for (int k = 0; k < 4 * kHalf; ++k) {
          const f32x4 other = *left_for(wave_s, tq, k), lo = half_of(tq, 0, k), hi = half_of(tq, 1, k);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            sum[tq][k][e] = (ks == 0 ? lo[e] : other[e]) * f0;
            sum[tq][k][e] += f1 * (ks == 0 ? other[e] : hi[e]);
          }
        }
        const float lse_row = mt * sl2 + __builtin_log2f(l_row[tq]);
        const int row = q0 + 32 * tq + l32;
        if (ks == 0 && g == 0) {
          lse_lds[(qw * QT + tq) * 32 + l32] = lse_row;
          if (row < n) lse2[(size_t)h * a.lse_stride + row] = lse_row;
        }
      }
#pragma unroll
      for (int tq = 0; tq < QT; ++tq)
#pragma unroll
        for (int k = 0; k < 4 * kHalf; ++k) asm volatile("" : "+v"(sum[tq][k]));       // what was left has been read
      if (a.partial != nullptr && wave_s < n_kb) load_keys(wave_s);
      if (out_rows != nullptr) {
        // fours k of the half are its channels 8 k + 4 g .. + 3: of two neighbouring ones the halves of the wave exchange one, and each
        // lane has eight channels in a row; then through LDS, so that the global stores are whole rows of the half.
        constexpr int kRowChunks = D / 16;         // 16-byte chunks of a half row, swizzled by the row
        u32x4* const rows = reinterpret_cast<u32x4*>(lds_v) + S::kWaves * QT * 16 + wave_s * 32 * kRowChunks;      // (behind the statistics)
#pragma unroll
        for (int tq = 0; tq < QT; ++tq) {
          const float inv = 1.f / l_row[tq];
#pragma unroll
          for (int k = 0; k < 4 * kHalf; k += 2) {
            const f32x4 x = sum[tq][k], y = sum[tq][k + 1];
            const auto lo = __builtin_amdgcn_permlane32_swap(pack_bf16(x[0] * inv, x[1] * inv), pack_bf16(y[0] * inv, y[1] * inv), false, false);
            const auto hi = __builtin_amdgcn_permlane32_swap(pack_bf16(x[2] * inv, x[3] * inv), pack_bf16(y[2] * inv, y[3] * inv), false, false);
            rows[l32 * kRowChunks + ((k + g) ^ (l32 % kRowChunks))] = u32x4{lo[0], hi[0], lo[1], hi[1]};
          }
#pragma unroll
          for (int it = 0; it < kRowChunks / 2; ++it) {
            const int r = (64 * it + lane) / kRowChunks, ch = lane % kRowChunks, row = q0 + 32 * tq + r;
            const u32x4 val = rows[r * kRowChunks + (ch ^ (r % kRowChunks))];
            if (row < n) *reinterpret_cast<u32x4*>(out_rows + ((size_t)row * a.n_q_heads + h) * D + (D / 2) * ks + 8 * ch) = val;
          }
        }
      }
    }
  }

  // ================================================================ careful path
  // Textbook online softmax, one 32-row tile per wave, one tile buffer, no overlap.
  // Only reached when a logit exceeded its row's reference by more than 2^64.
  if (redo) {
    const bool active = wave < S::kRows / 32;
    const int qs = active ? first_row_of(wave / QT) + 32 * (wave % QT) : 0;
    bf16x8 qf[D / 16];
    {
      const int row = min(qs + l32, n - 1);
      const u16* src = q_rows + ((size_t)row * a.n_q_heads + h) * D + 8 * g;
#pragma unroll
      for (int s = 0; s < D / 16; ++s)
        qf[s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(src + 16 * s));
    }
    f32x16 o[D / 32];
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[dt][r] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;
    for (int t = 0; t < n_tiles; ++t) {
      __syncthreads();                                   // the tile buffer is free
      issue_any(kc, kn, lds_k, t, ld_chunk_k);
      issue_any(vc, vn, lds_v, t, ld_chunk_v);
      wait_loads();
      __syncthreads();                                   // and full again
      if (!active) continue;
      for (int blk = 0; blk < S::kTk / 32; ++blk) {
        const int kb = t * S::kTk + 32 * blk;
        if (kb >= n_cand || (kb >= c && kb - c > qs + 31 + shift)) continue;    // nothing visible
        f32x16 s;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
        for (int st = 0; st < D / 16; ++st)
          s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_read_b128(lds_k + 32 * blk * D + k_off[st]), qf[st], s, 0, 0, 0);
        const int lim = min(qs + l32 + shift + c, n_cand - 1) - kb - 4 * g;
        float mx = -INFINITY;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          s[r] = (8 * (r >> 2) + (r & 3) <= lim) ? s[r] : -INFINITY;
          mx = fmaxf(mx, s[r]);
        }
        mx = max_with_other_half(mx);
        const float m_new = fmaxf(m_run, mx);
        const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
        const float alpha = __builtin_amdgcn_exp2f((m_run - m_use) * sl2);
        const float neg = -m_use * sl2;
        unsigned pb[8];
        float sum = 0.f;
#pragma unroll
        for (int r = 0; r < 8; ++r) {
          const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[2 * r], sl2, neg));
          const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[2 * r + 1], sl2, neg));
          sum += p0 + p1;
          pb[r] = pack_bf16(p0, p1);
        }
        l_run = l_run * alpha + sum;
        m_run = m_new;
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt) {
#pragma unroll
          for (int r = 0; r < 16; ++r) o[dt][r] *= alpha;
#pragma unroll
          for (int mm = 0; mm < 2; ++mm) {
            const bf16x8 va = lds_read_vt(lds_v + 32 * blk * D + v_off[dt] + 16 * mm * D, 8 * D);
            const u32x4 pw = {pb[4 * mm], pb[4 * mm + 1], pb[4 * mm + 2], pb[4 * mm + 3]};
            o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, __builtin_bit_cast(bf16x8, pw), o[dt], 0, 0, 0);
          }
        }
      }
    }
    if (active) {
      l_run = sum_with_other_half(l_run);
      const int row = qs + l32;
      if (row < n) {
        const float inv = 1.f / l_run;
        if (out_rows != nullptr) {
          u16* dstp = out_rows + ((size_t)row * a.n_q_heads + h) * D + 4 * g;
#pragma unroll
          for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              u32x2 pk;
              pk.x = pack_bf16(o[dt][4 * j] * inv, o[dt][4 * j + 1] * inv);
              pk.y = pack_bf16(o[dt][4 * j + 2] * inv, o[dt][4 * j + 3] * inv);
              *reinterpret_cast<u32x2*>(dstp + 32 * dt + 8 * j) = pk;
            }
        }
        if (g == 0) lse2[(size_t)h * a.lse_stride + row] = m_run * sl2 + __builtin_log2f(l_run);
      }
      // wave w worked on row group w / QT, tile w % QT: the same order as the fast path's
      if (g == 0) lse_lds[wave * 32 + l32] = m_run * sl2 + __builtin_log2f(l_run);
    }
  }

  // ================================================================ scores
  // Eq. 4 needs every row's FINAL normaliser, so the column sums are a second sweep over the
  // workgroup's keys, now that its rows have their log-sum-exp.  The roles change: the workgroup's
  // query rows are in LDS (row tiles of 32), and every wave takes every kWaves-th block of
  // 32 keys and keeps it in registers as the B operand while the row tiles pass by as the A
  // operand.  S = Q K^T then has one KEY column per lane and 16 rows of it in the lane's
  // registers: exp2(S - lse) is the exact softmax weight, the column sum is a running add inside
  // the lane, and after the last row tile the lane pair holds the sum over all of the workgroup's
  // rows.  No barrier, no exchange between waves, no atomics: one partial array per workgroup,
  // and the selection adds the arrays of a KV head in a fixed order.
  if (a.partial == nullptr) return;
  {
    constexpr int kNK = D / 16;
    constexpr int kRowTiles = QW * QT;
    static_assert(kRowTiles % 2 == 0, "the two accumulator sets alternate over the row tiles");
    __syncthreads();               // the statistics are in LDS; nobody needs the tile buffers any more
    const int split = (h - hk * group) * a.n_row_tiles + rt;
    float* const part = in_set_of(a.partial, a.g, li) + (size_t)hk * a.partial_stride + (size_t)split * a.cand_stride;
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

    // the block in the strip into registers, the next one on its way
    auto next_keys = [&](bf16x8 (&kf)[kNK], int next_kbi) __attribute__((always_inline)) {
      wait_loads();
      asm volatile("" ::: "memory");
#pragma unroll
      for (int st = 0; st < kNK; ++st) kf[st] = lds_read_b128(k_strip + k_off[st]);
#pragma unroll
      for (int st = 0; st < kNK; ++st) asm volatile("" : "+v"(kf[st]));      // the strip has been read
      if (next_kbi < n_kb) load_keys(next_kbi);
    };
    // The scale behind an opaque copy for every variant of the stage below, made here, where all
    // lanes are active: the variants then share no subexpression, and the compiler cannot lift the
    // scale-and-shift of all sixteen elements above the branch that picks the variant, out of the
    // MFMAs' shadow.
    float sl2_copy[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) asm volatile("v_mov_b32 %0, %1" : "=v"(sl2_copy[i]) : "s"(sl2));
    // A slot is one key block against kR consecutive row tiles (64 rows when a workgroup has four
    // row tiles: its first two tiles are neighbours, and so are its last two): kR independent
    // chains of matrix instructions, and the costs a slot pays once -- the wait for its first
    // fragments, picking its variant, the distance to the first read of its result -- are shared
    // by twice the work.
    constexpr int kR = kRowTiles == 4 ? 2 : 1;
    constexpr int kSlots = kRowTiles / kR;
    static_assert(kSlots % 2 == 0, "the two accumulator sets alternate over the slots");
    // The slot before the current one: its logits wait in the other accumulator set.
    bool p_vis = false, p_plain = false;
    int p_kb0 = 0, p_row0 = 0, p_tile = 0;

    // One slot: the MFMAs of (key block, row tiles) into s_new among the exponentials of the slot
    // before it from s_exp, laid out MFMA by MFMA as in the first sweep.  Returns this lane's sum
    // of the exponentiated slot over its 16 kR rows.
    auto stage = [&](const f32x16 (&s_exp)[kR], f32x16 (&s_new)[kR], const u16* qt, const bf16x8 (&kf)[kNK],
                     auto do_mfma, auto do_exp, auto mask) __attribute__((always_inline)) -> float {
      constexpr bool kMfma = decltype(do_mfma)::value, kExp = decltype(do_exp)::value, kMask = decltype(mask)::value;
      constexpr int kElems = 16 * kR;
      constexpr int kPer = kMfma ? 16 / kNK : kElems;      // elements per matrix instruction
      constexpr int kAhead = kNK < 4 ? kNK : 4;
      bf16x8 qfr[kR][kNK];
      float ls[kR][16];
      float sum[2] = {0.f, 0.f};
      int first[kR];
      unsigned span[kR];
      if constexpr (kExp) {
        // statistics of the previous slot's rows: register r is row 8 (r / 4) + 4 g + r % 4 of its tile
#pragma unroll
        for (int t = 0; t < kR; ++t)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const f32x4 v = *reinterpret_cast<const f32x4*>(&lse_lds[(p_tile + t) * 32 + 8 * j + 4 * g]);
            ls[t][4 * j] = v[0]; ls[t][4 * j + 1] = v[1]; ls[t][4 * j + 2] = v[2]; ls[t][4 * j + 3] = v[3];
          }
        if constexpr (kMask) {
          // key p_kb0 + l32 counts for the row at offset off = 8 (r / 4) + r % 4 from the tile's row
          // 4 g iff first <= off < rows left in the block
#pragma unroll
          for (int t = 0; t < kR; ++t) {
            const int row0 = p_row0 + 32 * t + 4 * g;
            first[t] = p_kb0 + l32 - c - shift - row0;            // negative for a cached key
            span[t] = (unsigned)max(n - row0 - first[t], 0);
          }
        }
      }
      const float sl2_here = sl2_copy[(kMfma ? 0 : 2) + (kMask ? 1 : 0)];
      int ei = 0;
      float arg = 0.f, pe1 = 0.f;
      if constexpr (kExp) arg = __builtin_fmaf(s_exp[0][0], sl2_here, -ls[0][0]);
      auto finish_element = [&](int e) __attribute__((always_inline)) {      // element e is in pe1
        float p = pe1;
        if constexpr (kMask) p = (unsigned)(8 * ((e % 16) >> 2) + (e & 3) - first[e / 16]) < span[e / 16] ? p : 0.f;
        sum[e & 1] += p;
        asm volatile("" : "+v"(sum[e & 1]));
      };
      auto exp_some = [&]() __attribute__((always_inline)) {
        if constexpr (kExp) {
#pragma unroll
          for (int k = 0; k < kPer; ++k, ++ei) {
            const float pe = __builtin_amdgcn_exp2f(arg);
            if (ei + 1 < kElems)
              arg = __builtin_fmaf(s_exp[(ei + 1) / 16][(ei + 1) % 16], sl2_here, -ls[(ei + 1) / 16][(ei + 1) % 16]);
            if (ei >= 1) finish_element(ei - 1);
            pe1 = pe;
          }
        }
      };
      if constexpr (kMfma) {
#pragma unroll
        for (int st = 0; st < kAhead; ++st)
#pragma unroll
          for (int t = 0; t < kR; ++t) qfr[t][st] = lds_read_b128(qt + t * 32 * D + k_off[st]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int st = 0; st < kNK; ++st) {
#pragma unroll
          for (int t = 0; t < kR; ++t) {
            if (st + kAhead < kNK) qfr[t][st + kAhead] = lds_read_b128(qt + t * 32 * D + k_off[st + kAhead]);
            s_new[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qfr[t][st], kf[st], st == 0 ? zero : s_new[t], 0, 0, 0);
            exp_some();
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      } else {
        exp_some();
      }
      if constexpr (kExp) finish_element(kElems - 1);
      if constexpr (kMfma) {
        // A vector instruction may read the result of a 32x32x16 matrix instruction only twelve wait
        // states after it was issued.  The next reader of s_new sits in another basic block (the next
        // slot's variant, or a register copy the compiler puts at a block boundary), and measured
        // results show that nobody counts the distance across that boundary: a slot that consists
        // of matrix instructions only was read too early.  So every slot pays the distance itself.
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_nop 7\n\ts_nop 3");
        __builtin_amdgcn_sched_barrier(0);
      }
      return sum[0] + sum[1];
    };
    typedef std::true_type Yes;
    typedef std::false_type No;
    // the slot as it stands: is the current pair visible at all, was the previous one, did it need the mask
    auto slot = [&](const f32x16 (&s_exp)[kR], f32x16 (&s_new)[kR], const u16* qt, const bf16x8 (&kf)[kNK], bool vis)
        __attribute__((always_inline)) -> float {
      if (vis) {
        if (!p_vis) return stage(s_exp, s_new, qt, kf, Yes{}, No{}, No{});
        return p_plain ? stage(s_exp, s_new, qt, kf, Yes{}, Yes{}, No{}) : stage(s_exp, s_new, qt, kf, Yes{}, Yes{}, Yes{});
      }
      if (!p_vis) return 0.f;
      return p_plain ? stage(s_exp, s_new, qt, kf, No{}, Yes{}, No{}) : stage(s_exp, s_new, qt, kf, No{}, Yes{}, Yes{});
    };
    auto store_block = [&](int kbi, float mine) __attribute__((always_inline)) {
      const float tot = sum_with_other_half(mine);       // lanes l and l + 32 hold the two halves of the rows
      const int kv = kbi * 32 + l32;
      if (g == 0 && kv < n_cand) part[kv] = tot;
    };

    f32x16 sa[kR], sb[kR];
#pragma unroll
    for (int t = 0; t < kR; ++t) { sa[t] = zero; sb[t] = zero; }
    float carry = 0.f;             // sums of the block before the current one, its last slot still to come
    int carry_kb = -1;
    // all row tiles against one key block; the next block of this wave is fetched meanwhile
    auto do_block = [&](const bf16x8 (&kf)[kNK], int kbi) __attribute__((always_inline)) {
      const int kb0 = kbi * 32;
      float acc = 0.f;
#pragma unroll
      for (int i = 0; i < kSlots; ++i) {
        // the slot's rows: row0 .. row0 + 32 kR - 1 (row tiles kR i .. kR i + kR - 1 are neighbours)
        const int tile = kR * i;
        const int row0 = first_row_of(tile / QT) + 32 * (tile % QT);
        // some row of the slot sees some key of the block; every row sees every key and all are real
        const bool vis = row0 < n && (kb0 < c || kb0 - c <= row0 + 32 * kR - 1 + shift);
        const bool plain = kb0 + 31 < n_cand && (kb0 + 31 < c || kb0 + 31 - c <= row0 + shift) && row0 + 32 * kR <= n;
        const float got = (i & 1) ? slot(sa, sb, q_lds + tile * 32 * D, kf, vis) : slot(sb, sa, q_lds + tile * 32 * D, kf, vis);
        if (i == 0) {
          if (carry_kb >= 0) store_block(carry_kb, carry + got);   // the last slot of the block before
        } else {
          acc += got;
        }
        p_vis = vis; p_plain = plain; p_kb0 = kb0; p_row0 = row0; p_tile = tile;
      }
      carry = acc;
      carry_kb = kbi;
    };
    // This wave's key blocks are wave, wave + kWaves, ...
    bf16x8 kf[kNK];
    if (redo && wave_s < n_kb) load_keys(wave_s);      // (else it is on its way)
    for (int kbi = wave_s; kbi < n_kb; kbi += S::kWaves) {
      next_keys(kf, kbi + S::kWaves);
      do_block(kf, kbi);
    }
    if (carry_kb >= 0) {
      // the last slot of the last block: its logits are in the second accumulator set
      const float got = slot(sb, sa, q_lds, kf, false);
      store_block(carry_kb, carry + got);
    }
    // keys that none of this workgroup's rows see: zeros (the selection adds every partial array)
    for (int kv = n_kb * 32 + tid; kv < n_cand; kv += kThreads) part[kv] = 0.f;
  }
}

template <int D, int QT, int QW, int KS>
hipError_t launch_shape(const AttnArgs& a, hipStream_t s) {
  using S = Shape<D, QT, QW, KS>;
  const int grid = kXcds * a.work_per_xcd;
  hipLaunchKernelGGL((attention_kernel<D, QT, QW, KS>), dim3(grid, a.g.n_layers), dim3(S::kThreads), S::kLdsBytes, s, a);
  return hipGetLastError();
}

template <int D, int QT, int QW, int KS>
hipError_t prepare_shape() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(attention_kernel<D, QT, QW, KS>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, Shape<D, QT, QW, KS>::kLdsBytes);
}

}  // namespace

// Every shape needs more dynamic LDS than a kernel gets by default.  The attribute belongs to the
// function on the current device, so this runs once per cache creation, on the cache's device.
hipError_t prepare_attention() {
  hipError_t e;
  if ((e = prepare_shape<128, 2, 2, 2>()) != hipSuccess) return e;
  if ((e = prepare_shape<128, 1, 4, 2>()) != hipSuccess) return e;
  if ((e = prepare_shape<128, 1, 2, 2>()) != hipSuccess) return e;
  if ((e = prepare_shape<64, 2, 2, 2>()) != hipSuccess) return e;
  if ((e = prepare_shape<64, 1, 4, 2>()) != hipSuccess) return e;
  if ((e = prepare_shape<64, 1, 2, 2>()) != hipSuccess) return e;
  return prepare_attention_split();
}

hipError_t launch_attention(const AttnArgs& a, int head_dim, hipStream_t s) {
  if (a.variant == kAttnSplit32 || a.variant == kAttnSplit64) return launch_attention_split(a, head_dim, s);
  if (head_dim == 128) {
    if (a.variant == kAttnWide4) return launch_shape<128, 2, 2, 2>(a, s);
    if (a.variant == kAttnTile128) return launch_shape<128, 1, 4, 2>(a, s);
    return launch_shape<128, 1, 2, 2>(a, s);
  }
  if (a.variant == kAttnWide4) return launch_shape<64, 2, 2, 2>(a, s);
  if (a.variant == kAttnTile128) return launch_shape<64, 1, 4, 2>(a, s);
  return launch_shape<64, 1, 2, 2>(a, s);
}

}  // namespace kvp
