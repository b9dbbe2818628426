// Host-side planning of the launches: workgroup shapes, grids, splits and scratch sizes.  Nothing
// here touches the device; the file is also part of the host-only build that runs the state
// machine under the address and undefined-behaviour sanitizers.
#include "kvp_internal.h"

namespace kvp {

// ---- attention
// 128-row workgroups of attention.hip when a layer's block has about one of them for every CU (from
// three quarters on: every key tile then serves 128 rows, and the shape that splits the keys would need
// three rounds of the chip); below that the split-key shapes of attention_split.hip: 32-row workgroups
// while all of them fit on the chip at once, 64-row ones (half as many) beyond.  Per launch with scores,
// against the four-wave 64-row tiles that used to serve these blocks:
//   16/4 heads, d 64, 333 rows over 1444 keys   28.4 ->  9.7 us
//   28/4 heads, d 128, 256 rows over 768 keys   22.7 ->  7.3 us (eight layers per launch)
//   32/32 heads, d 128, 128 rows over 384 keys  15.1 ->  7.5 us
//   28/4 heads, d 128, 512 rows over 1536 keys  34.6 -> 25.6 us (64-row workgroups)
// The lines, whole prefixes with the shape on this side and on the other, one layer per launch (8 layers):
//   at 192 workgroups of 128 rows, 64-row ones instead: 28/4 heads, d 128, 896 rows (196) 4318 -> 4683 us (2616 -> 2752), 32/8 heads, 768 rows
//     (192) 3930 -> 4654 (2415 -> 2769); 28/4 heads, 800 rows (196) 4166 -> 4525 (2706 -> 2639); at d 64 they are ahead, 16/4 heads, 1500 rows (192)
//     2329 -> 2210 (1250 -> 1183);
//   above 256 workgroups of 32 rows, 32-row ones instead: 28/4 heads, d 128, 320 rows (280) 5235 -> 6008 (1979 -> 2419), 32/8 heads, 512 rows (512)
//     4445 -> 5072 (2754 -> 3279), 16/4 heads, d 64, 600 rows (304) 2907 -> 2962 (1064 -> 1117); 32/8 heads, 288 rows (288) 5990 -> 5788 (2462 -> 2335);
//   up to 256, 64-row ones instead: 28/4 heads, d 128, 256 rows (224) 4440 -> 5461 (1658 -> 1710), 32/32 heads, 256 rows (256) 4678 -> 5836 (2200 -> 2131),
//     16/4 heads, d 64, 500 rows (256) 2613 -> 3242 (963 -> 1004).
// The choice depends on one layer's block alone, never on how many layers a launch takes, so that
// grouped and single launches leave the same bits.
static int shape_for(int n, int n_q_heads) {
  if (((n + 127) / 128) * n_q_heads >= 192) return kAttnTile128;
  return ((n + 31) / 32) * n_q_heads <= 256 ? kAttnSplit32 : kAttnSplit64;
}

// The most partial score arrays per KV head (query heads of the group x row tiles) that a block of
// up to chunk_max rows leaves when the library picks the shape itself.  A forced shape may need
// more; such a launch then scores with the separate kernel.
int attention_max_partials(int group, int n_q_heads, int chunk_max) {
  int most = 0;
  for (int n = 1; n <= chunk_max; ++n) {
    const int rows = kAttnRowsOfShape[shape_for(n, n_q_heads)];
    const int tiles = (n + rows - 1) / rows;
    most = tiles > most ? tiles : most;
  }
  return group * most;
}

void plan_attention(AttnArgs& a, int /*head_dim*/, int forced_shape) {
  a.variant = shape_for(a.n, a.n_q_heads);
  if (forced_shape >= 0 && forced_shape <= 2) a.variant = forced_shape;      // kvp_set_attention_shape
  const int rows = kAttnRowsOfShape[a.variant];
  a.n_row_tiles = (a.n + rows - 1) / rows;
  a.total_work = a.n_row_tiles * a.n_q_heads;
  a.group = a.n_q_heads / a.n_kv_heads;
  const Divisor by_tiles = divisor_of((unsigned)a.n_row_tiles, (unsigned)a.total_work);
  const Divisor by_group = divisor_of((unsigned)a.group, (unsigned)a.n_q_heads);
  a.tiles_magic = by_tiles.magic; a.tiles_shift = by_tiles.shift;
  a.group_magic = by_group.magic; a.group_shift = by_group.shift;
  a.work_per_xcd = (a.total_work + kXcds - 1) / kXcds;
}


// ---- column sums
int colsum_max_partials(int /*group*/, int /*chunk_max*/) { return kColsumMaxRowSplits; }

// Key blocks of 32 * nt * kColsumWaves keys, each with as many row splits as it takes to give a workgroup `tau` of the
// query tiles that see it.
static void colsum_work(ColsumArgs& a, int nt, int tau) {
  const int n_qt = (a.n + 31) / 32;
  const int block_keys = 32 * nt * kColsumWaves;
  a.subtiles = nt;
  a.n_kv_blocks = (a.c + a.n_keys + block_keys - 1) / block_keys;
  int total = 0, most = 0;
  for (int k = 0; k < a.n_kv_blocks; ++k) {
    const int blk0 = k * block_keys;
    const int first_tile = blk0 - a.c > a.shift ? (blk0 - a.c - a.shift) / 32 : 0;
    const int visible = n_qt - first_tile > 0 ? n_qt - first_tile : 1;
    const int splits = (visible + tau - 1) / tau;
    a.split_prefix[k] = total;
    total += splits;
    most = splits > most ? splits : most;
  }
  a.split_prefix[a.n_kv_blocks] = total;
  a.wgs_per_head = total;
  a.n_partials = most;
}

void plan_colsum(ColsumArgs& a, int n_layers) {
  const int n_cand = a.c + a.n_keys;
  const int n_qt = (a.n + 31) / 32;
  // 64 keys per wave, or 32 when that is what it takes to spread a small launch over the chip
  const int wide_blocks = (n_cand + 64 * kColsumWaves - 1) / (64 * kColsumWaves) * a.n_kv_heads;
  const int most_splits = n_qt < kColsumMaxRowSplits ? n_qt : kColsumMaxRowSplits;
  const int nt = wide_blocks * most_splits < kColsumTargetWorkgroups / 2 ? 1 : 2;
  // tiles per row split: the fewest that keep the launch within one round (and the row splits of
  // a block within the partial count)
  int tau = (n_qt + kColsumMaxRowSplits - 1) / kColsumMaxRowSplits;
  for (;; ++tau) {
    colsum_work(a, nt, tau);
    if (a.wgs_per_head * a.n_kv_heads <= kColsumTargetWorkgroups || tau >= n_qt) break;
  }
  // A launch for several layers has workgroups enough without the row splits, and a workgroup pays for its keys
  // as much as for two or three of its steps.  Grouped and single launches must leave the same bits, so the
  // sums stay cut where they are: a workgroup takes several splits one after the other, and 64 keys per wave.
  // Only for proxy queries, where every split of every key block has as much work.
  a.splits_per_wg = 1;
  if (a.shift >= a.n_keys && n_layers > 1) {
    const int splits = a.n_partials;
    if (nt == 1 && wide_blocks * splits * n_layers >= kColsumTargetWorkgroups) colsum_work(a, 2, tau);
    const int all = a.n_kv_blocks * a.n_kv_heads * n_layers;
    while (a.splits_per_wg < splits && all * ((splits + a.splits_per_wg) / (a.splits_per_wg + 1)) >= kColsumTargetWorkgroups)
      ++a.splits_per_wg;
    a.wgs_per_head = a.n_kv_blocks * ((splits + a.splits_per_wg - 1) / a.splits_per_wg);
  }
  a.total_work = a.wgs_per_head * a.n_kv_heads;
  a.wgs_magic = divisor_magic((unsigned)a.wgs_per_head);
  a.group = a.n_q_heads / a.n_kv_heads;
  a.work_per_xcd = (a.total_work + kXcds - 1) / kXcds;
}


// ---- selection and compaction
// key, cnt, evicted, free_slot; the histogram; the token table; the source lists or, before them, the score
// sums (up to 4096 candidates; beyond that the lists are in the scratch set and the sums lie elsewhere)
size_t select_lds_bytes(const SelectArgs& a) {
  const size_t cand_pad = (size_t)a.items * a.threads;
  const size_t lists = a.items > 4 ? 0 : cand_pad * kNeighbours * 2, 
               sums = a.items > 4 ? 0 : (size_t)a.groups * a.quads * 16 + (a.keydiff ? (a.threads / 64 + 1) * (size_t)a.head_dim * 4 : 0);
  return cand_pad * (8 + 1 + 2 + 2) + kSelectBins * 4 + (size_t)a.table_size * 2 + (lists > sums ? lists : sums);
}

// A workgroup has 512 threads up to 1024 candidates (and where it holds the keys in registers), 1024 beyond.  Most of its phases are
// what every wave does for itself (scans, the search of the histogram) on four SIMDs, so that fewer waves are done sooner,
// until there are too few for the rows.  Per launch with 512 threads, with 1024: 4 heads of d 64, 192 candidates 7.7,
// 9.3 us; 4 heads of d 128, 768 candidates 12.4, 13.2 us, 8 layers of them 12.9, 13.8 us; 1536 candidates 19.4, 16.8 us, 16 layers
// of them 23.0, 20.3 us.  (With 256 threads, in an earlier kernel, the first two took half a microsecond more, and 8 layers of 768
// candidates 3 us.)
// A thread owns ceil(n_cand / threads) neighbouring candidates.  For the sums of the partial arrays the threads
// form groups of 64, 128 or 256 (the fewest that cover the candidates in fours, 256 at most) that take
// every groups-th array, so that all of them have loads in flight whatever the number of candidates.
// The token table has an entry for every token before the block where LDS has room for that.
void plan_select(SelectArgs& a) {
  const int n_cand = a.c + a.n;
  a.threads = n_cand <= 1024 || a.keydiff ? 512 : kSelectThreads;
  a.items = (n_cand + a.threads - 1) / a.threads;
  a.quads = (n_cand + 3) / 4;
  a.width = a.items > 4 ? a.threads : a.quads <= 64 ? 64 : a.quads <= 128 ? 128 : 256;
  a.groups = a.score_override || a.keydiff ? 1 : a.threads / a.width;
  if (a.groups > a.n_partials) a.groups = a.n_partials < 1 ? 1 : a.n_partials;
  a.width_log2 = 0;
  while (1 << a.width_log2 < a.width) ++a.width_log2;
  a.groups_magic = divisor_magic((unsigned)a.groups);
  a.direct = 1;
  a.table_size = ((a.t0 > n_cand ? a.t0 : n_cand) + 7) / 8 * 8;       // (it becomes the list of destinations, too)
  if (!a.merge || select_lds_bytes(a) > kSelectLdsLimit) {
    a.direct = 0;
    a.table_size = 8;
    while (a.merge && a.table_size < 2 * n_cand) a.table_size <<= 1;
  }
}

// Keys that the threads of one workgroup can hold in registers: the compaction then scores by the keys alone itself.
bool keydiff_in_compaction(int n_cand, int head_dim) {
  return n_cand <= kKeydiffRowsPerThread * (512 / (head_dim / 8));
}

// The attention launch of the split-key shapes has workgroups that score such heads by the keys, one per KV head (up to a multiple
// of kXcds), where they cost less than the compaction's own scoring, 6 us in front of its other phases.  Prefixes scored in the
// compaction, and beside the attention, one layer per launch unless said otherwise:
//   32-row workgroups are as many as CUs at most, one round of the chip.  While the scoring ones fit into it, too:
//     28/4 heads, d 128, 256 rows over 768 keys (224 + 8 workgroups) 819 -> 636 us, 8 layers per launch 628 -> 623 us;
//     16/4 heads, d 64, 333 rows over 1444 keys (176 + 8) 914 -> 712 us.
//   Beyond, as many attention workgroups wait for a second round: 64/64 heads, 128 rows over 384 keys (256 + 64) 725 -> 772 us,
//     64/8 heads, 128 rows over 640 keys (256 + 8) 838 -> 863, 32/8 heads, 256 rows over 768 keys (256 + 8) 806 -> 817 us
//     (32/32 heads, 256 rows over 768 keys, 256 + 32, 893 -> 881 us).
//   64-row workgroups take two or three times as long as a scoring one: 40/8 heads, d 128, 512 rows over 1024 keys (320 + 8)
//     1461 -> 1207 us, 8 layers per launch 1305 -> 1267 us.
//   At d 64 the kernel that scores keys holds one workgroup per CU, the other two.  That shows in launches of many
//     rounds: 28/4 heads, 512 rows over 1536 keys (232 workgroups a layer), 2 layers per launch 1971 -> 1821 us, 3 layers 1200 -> 1154,
//     4 layers 1377 -> 1380, 8 layers 993 -> 1131; 16/4 heads, 333 rows over 1444 keys (184 a layer), 3 layers 1366 -> 1210 us,
//     4 layers 1477 -> 1293, 8 layers 988 -> 970.
// Both ways leave the same bits, so that this may depend on the layers of a launch.
bool scores_keys_beside_attention(const AttnArgs& a, int n_layers, int n_cand, int head_dim) {
  if (a.variant != kAttnSplit32 && a.variant != kAttnSplit64) return false;
  if (!keydiff_in_compaction(n_cand, head_dim)) return false;
  const int workgroups = a.total_work + key_score_workgroups(a.n_kv_heads);
  if (a.variant == kAttnSplit32 && workgroups > 256) return false;
  return head_dim == 128 || workgroups * n_layers <= 3 * 256;
}
int key_score_workgroups(int n_kv_heads) { return (n_kv_heads + kXcds - 1) / kXcds * kXcds; }

// ---- compaction: row pairs (K row and V row of a slot, 16 bytes per lane) a workgroup carries
int rows_per_compact_block(int head_dim) { return kCompactThreads / (2 * head_dim / 8); }

// ---- proxy row statistics, key-only scores
int rowstat_key_blocks(int n_cand) { return (n_cand + kRowstatBlockKeys - 1) / kRowstatBlockKeys; }
int keydiff_slices(int n_cand) { return (n_cand + kKeydiffSliceKeys - 1) / kKeydiffSliceKeys; }

// ---- decode step
int decode_max_group() { return kDecodeGroupLimit; }

// workgroups per KV head the step would like: one per 64-key tile, kDecodeMaxSplits at most
int decode_splits_wanted(long long n_keys) {
  const long long want = (n_keys + kDecodeTile - 1) / kDecodeTile;
  return (int)(want > kDecodeMaxSplits ? kDecodeMaxSplits : want);
}

// workgroups per KV head: as many as wanted while their partial results fit the scratch
// (every workgroup then has at least one tile)
int decode_splits(long long n_keys, int head_dim, size_t scratch_floats, int n_q_heads) {
  long long want = decode_splits_wanted(n_keys);
  const long long fit = (long long)(scratch_floats / ((size_t)n_q_heads * (head_dim + 2)));
  if (want > fit) want = fit;
  return want < 1 ? 0 : (int)want;
}

}  // namespace kvp
