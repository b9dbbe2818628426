// Internal declarations shared by the host state machine and the kernel
// launchers of libkvp.  Not part of the public interface.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "divide.h"
#include "key_range.h"
#include "kvp.h"

namespace kvp {

typedef unsigned short u16;  // one bfloat16 bit pattern

constexpr int kXcds = 8;            // MI355X: 8 accelerator dies, each with its own L2
constexpr int kNeighbours = 6;      // 4 in the plane + 2 in time

// Sizes that the kernels and the host-side planning (plan.cpp) must agree on.
// Attention shapes: the three of attention.hip, then the two of attention_split.hip.
enum { kAttnWide4 = 0, kAttnTile64 = 1, kAttnTile128 = 2, kAttnSplit32 = 3, kAttnSplit64 = 4 };
constexpr int kAttnRowsOfShape[5] = {128, 64, 128, 32, 64};   // query rows per workgroup
constexpr int kColsumWaves = 4;                 // waves per workgroup of the column-sum kernel
constexpr int kColsumTargetWorkgroups = 512;    // two per CU, all resident: the launch is a single round
constexpr int kColsumMaxRowSplits = 16;
constexpr int kSelectThreads = 1024;            // the most of the compaction kernel
constexpr int kKeydiffRowsPerThread = 32;       // keys a thread of it can hold a piece of (of 512 threads)
constexpr size_t kSelectLdsLimit = 156 * 1024;  // dynamic LDS of the compaction kernel, beside 3.5 KiB of static LDS
constexpr int kRowstatBlockKeys = 256;          // keys per workgroup of the proxy row-statistics kernel
constexpr int kKeydiffSliceKeys = 64;           // keys per workgroup of the key-sum kernel
constexpr int kDecodeTile = 64;                 // keys per workgroup step of the decode kernel
constexpr int kDecodeMaxSplits = 128;
constexpr int kDecodeGroupLimit = 16;           // query heads per KV head the decode kernel is built for
constexpr int kCompactThreads = 256;
constexpr int kCompactTargetWorkgroups = 4096;  // an append launch is capped at about this many workgroups

// A launch covers a group of consecutive layers that hold the same block (same c, n, t0).  The cache
// and scratch pointers in a kernel's arguments are those of the group's FIRST layer; layer i of the
// group is reached through the strides below.
constexpr int kMaxGroupLayers = 16;
struct GroupStrides {
  int n_layers;
  int first_set, n_sets;        // layer i uses scratch set (first_set + i) % n_sets
  long long set_stride;         // bytes between scratch sets
  long long kv_stride;          // bf16 elements between the K (or V) caches of consecutive layers
  long long meta_stride;        // elements between their token_idx (or weight) arrays
};
struct LayerGroup : GroupStrides {
  const u16* k_new[kMaxGroupLayers];   // the block's keys and values of every layer of the group
  const u16* v_new[kMaxGroupLayers];
};

#if defined(__HIPCC__)
// Kernel arguments come from memory, a line at a time; read where they are first used they are a chain of waits on the
// way to a workgroup's first load.  This asks for all of its operands at once.
template <class T>
__device__ __forceinline__ void have_argument(T x) { asm volatile("" ::"s"(x)); }
template <class... T>
__device__ __forceinline__ void have_arguments(T... x) { (have_argument(x), ...); }

// Values that stay in registers from here on.  The compiler takes an argument for something that it can always load again and
// does so before each later use, with a wait for the load.
template <class T>
__device__ __forceinline__ void keep_argument(T& x) { asm volatile("" : "+s"(x)); }
template <class T>
__device__ __forceinline__ void keep_argument(T*& x) {
  auto global = (__attribute__((address_space(1))) T*)x;     // (it still has to be known as a pointer to global memory)
  asm volatile("" : "+s"(global));
  x = (T*)global;
}
template <class... T>
__device__ __forceinline__ void keep_arguments(T&... x) { (keep_argument(x), ...); }

// Row p of a list in two parts, the first c rows `old_bytes` apart and the others `new_bytes` apart: choices between values and
// one multiplication.  (Written as a choice between two addresses this becomes a branch around two long
// multiplications for every load.)  Offset: unsigned where a part is smaller than 4 GiB (and its rows less than 16 MiB apart).
template <class Offset>
__device__ __forceinline__ const u16* row_of_two(const u16* old_rows, unsigned old_bytes, const u16* new_rows, unsigned new_bytes, int p, int c) {
  const bool old = p < c;
  const unsigned row = (unsigned)(old ? p : p - c), bytes = old ? old_bytes : new_bytes;
  const char* const base = reinterpret_cast<const char*>(old ? old_rows : new_rows);
  if constexpr (sizeof(Offset) == 4) return reinterpret_cast<const u16*>(base + __umul24(row, bytes));
  else return reinterpret_cast<const u16*>(base + (unsigned long long)row * bytes);
}

// the same pointer in scratch set (first_set + li) % n_sets instead of set first_set (a group has at most
// n_sets layers: one subtraction wraps; pointer arithmetic, not integers: the compiler then still
// knows that it points to global memory)
template <class T>
__device__ __forceinline__ T* in_set_of(T* p, const GroupStrides& g, int li) {
  if (p == nullptr) return p;
  const int sets = g.first_set + li < g.n_sets ? li : li - g.n_sets;
  return (T*)((char*)p + sets * g.set_stride);
}
#endif

// One block of a group of layers attending over cache U block (Eq. 1); the layers of a group are
// independent, and one launch for all of them fills the chip where a single layer's rows do not.
struct AttnLayer {
  const u16* q;        // [n, Hq, D]
  const u16* k_new;    // [n_keys, Hkv, D]
  const u16* v_new;
  u16* out;            // [n, Hq, D], or null: only the row statistics are wanted
};
struct AttnPlan {
  // Arguments are read from far memory at every launch, one 64-byte line at a time: what a workgroup
  // needs first lies together, and so do the pointers of a layer.
  int n, c, n_q_heads, n_kv_heads, budget, lse_stride;
  int n_keys;          // block keys (k_new, v_new rows); the query rows are n
  int shift;           // row r sees block key j iff j <= r + shift (0: causal block; >= n_keys: all)
  int n_row_tiles, work_per_xcd, total_work;   // work items of one layer (grid y = layer)
  int group;           // query heads per KV head
  unsigned tiles_magic, group_magic;   // divisor_of n_row_tiles and of group
  float scale_log2;    // softmax scale times log2(e)
  unsigned tiles_shift;                // 0 in the split-key shapes, of which a layer has fewer than 384 workgroups
  int key_score_wgs;   // workgroups in front that score the candidates by the keys alone (split-key shapes): one per KV head, up to a
                       // multiple of kXcds; their scores are the one partial array
  int partial_stride, cand_stride;   // floats from a KV head's partial arrays to the next head's, and from array to array
  unsigned group_shift;
  GroupStrides g;
  const u16* k_cache;  // the group's first layer: [Hkv, M, D]
  const u16* v_cache;
  float* lse2;         // [Hq, lse_stride]  log2-domain log-sum-exp of every row (first layer's scratch set, like partial)
  float* partial;      // null, or [Hkv][query heads of the group x n_row_tiles][candidates], strides above: the launch
                       // also leaves the column sums of its softmax matrix (Eq. 4), one array per workgroup of a KV head
};
struct AttnArgs : AttnPlan {
  AttnLayer layer[kMaxGroupLayers];
  int variant;         // tile shape, chosen by plan_attention (no kernel reads it)
};

// Column sums of the softmax matrix (Eq. 4 summed over rows and over the query
// heads of a KV group), one partial array per row split.
constexpr int kColsumMaxKvBlocks = 64;
struct ScoreLayer {
  const u16* q;        // [n, Hq, D]
  const u16* k_new;    // [n_keys, Hkv, D]
};
struct ColsumArgs {
  // One launch scores a group of layers (grid y = layer): layer i of the group reads the cache
  // g.kv_stride elements further on per layer, and its statistics and partials from scratch set
  // (g.first_set + i) % g.n_sets.  In the order of AttnArgs.
  int n, c, n_q_heads, n_kv_heads, budget, lse_stride, partial_stride, cand_stride;
  int n_keys, shift;   // as in AttnArgs
  int n_kv_blocks;     // blocks of 256 * subtiles keys
  int n_partials;      // the most row splits any key block has; every key gets that many partials
  int subtiles;        // 32-key subtiles per wave, chosen by plan_colsum
  int splits_per_wg;   // row splits a workgroup takes one after the other; more than one only where all blocks have as many
  int wgs_per_head;    // = split_prefix[n_kv_blocks] where that is one
  unsigned wgs_magic;  // its divisor_magic
  int group;           // query heads per KV head
  int work_per_xcd, total_work;
  float scale_log2;
  GroupStrides g;
  const u16* k_cache;  // of the group's first layer
  const float* lse2;   // in the first layer's scratch set, like partial
  float* partial;      // [Hkv][n_partials][candidates], strides as in AttnArgs
  // workgroups [split_prefix[k], split_prefix[k + 1]) of a head share key block k and split the
  // 32-row query tiles that see it evenly among themselves
  int split_prefix[kColsumMaxKvBlocks + 1];
  ScoreLayer layer[kMaxGroupLayers];
};

// Row statistics of a short list of proxy queries over all candidates (rowstat.hip).
struct RowstatArgs {
  int n, c, n_keys, n_q_heads, n_kv_heads, budget, lse_stride;
  int n_kv_blocks;     // set by launch_rowstat, like those up to the magics
  int items_per_wg;    // (query head, 32-row tile) items a workgroup takes
  int item_splits;     // workgroups that share the items of a KV head
  int group;           // query heads per KV head
  unsigned splits_magic, tiles_magic, rows_magic;   // divisor_magic of item_splits, of the row tiles and of n
  float scale_log2;
  GroupStrides g;      // a group of layers per launch, as in ColsumArgs
  const u16* k_cache;  // the group's first layer: [Hkv, M, D]
  float* lse2;         // [Hq, lse_stride] out
  float* part_m;       // [n_kv_blocks, Hq, n] scratch: row maximum per key block (raw logits)
  float* part_l;       // [n_kv_blocks, Hq, n] scratch: sum of exp2 against that maximum
  ScoreLayer layer[kMaxGroupLayers];   // q: the proxy queries
};
int rowstat_key_blocks(int n_cand);
hipError_t launch_rowstat(RowstatArgs a, int head_dim, hipStream_t s);

// Query-agnostic scores of all candidates (keydiff.hip).
struct KeydiffArgs {
  LayerGroup g;        // a group of layers per launch (grid z); g.k_new[i]: [n_keys, Hkv, D]
  const u16* k_cache;  // the group's first layer: [Hkv, M, D]
  float* sums;         // [Hkv][n_slices][D] scratch: column sums of the keys, one per slice
  float* scores;       // [Hkv][candidates] out (both in the first layer's scratch set, heads head_stride floats apart)
  int c, n_keys, n_kv_heads, budget, head_stride;
  int n_slices, keys_per_block;   // set by launch_keydiff
};
int keydiff_slices(int n_cand);
hipError_t launch_keydiff(KeydiffArgs a, int head_dim, hipStream_t s);

// One decode step of one layer (decode.hip).
struct DecodeArgs {
  int c, n_tail, n_q_heads, n_kv_heads, budget, n_splits;
  int group;           // query heads per KV head
  float scale_log2;
  const u16* q;        // [Hq, D]
  const u16* k_tail;   // [n_tail, Hkv, D]
  const u16* v_tail;
  u16* out;            // [Hq, D]
  const u16* k_cache;  // this layer: [Hkv, M, D]
  const u16* v_cache;
  float* partial;      // [Hq, n_splits, D + 2] scratch: unnormalised output, maximum, sum
};
int decode_max_group();
int decode_splits(long long n_keys, int head_dim, size_t scratch_floats, int n_q_heads);
int decode_splits_wanted(long long n_keys);
hipError_t launch_decode(const DecodeArgs& a, int head_dim, hipStream_t s);
// address and size of the file-scope scratch array on the current device (kvp_decode_step_static)
hipError_t decode_static_scratch(float** ptr, size_t* n_floats);

// Device copy of one prefix segment.
struct Seg {
  int begin, n, kind, gh, gw, planes, temporal;
};

struct LayerBlock {
  const u16* k_new;             // [n, Hkv, D] the block's keys and values of one layer
  const u16* v_new;
};

// Compaction of a group of layers whose block does not fit (select.hip); what a workgroup needs first lies
// together, as in AttnArgs.
struct SelectPlan {
  int c, n, t0, budget, partial_stride, cand_stride, chunk_max, n_partials, merge;
  int n_kv_heads, head_dim, n_segs;
  int threads;                  // of a workgroup: 512 or 1024
  int items;                    // candidates per thread
  int direct;                   // the token table has one entry per token before t0, not a hash of them
  int table_size;               // entries, a multiple of 8 (hash: a power of two >= 2 * (c + n))
  int quads;                    // fours of neighbouring candidates
  int keydiff;                  // 1: the kernel scores by the keys alone itself, there are no partial arrays
  int width, groups;            // the threads sum the partial arrays as `groups` groups of `width` (a power of two)
  int width_log2;
  unsigned groups_magic;        // divisor_magic of groups
  GroupStrides g;
  const float* partial;         // [Hkv][n_partials][candidates], strides as in AttnArgs
  const float* score_override;  // [Hkv, n_cand] used instead, or null
  int32_t* token_idx;           // the group's first layer: [Hkv, M]
  float* weight;
  float* scores;                // [Hkv, cand_stride]   scores actually used
  uint8_t* keep;                // [Hkv, cand_stride]
  int32_t* dst;                 // [Hkv, cand_stride]
  const Seg* segs;
  u16* k_cache;                 // the group's first layer: [Hkv, M, D]
  u16* v_cache;
  u16* sources;                 // [Hkv, cand_stride, kNeighbours]: source lists that do not fit into LDS
  u16* stage;                   // K, then V [chunk_max, D] of every head, over that head's partial arrays
  float* stage_w;               // [Hkv, chunk_max]
  unsigned long long* totals;   // [KVP_T_COUNT] running totals of the cache (kvp_debug_totals)
};
struct SelectArgs : SelectPlan {
  LayerBlock layer[kMaxGroupLayers];
};

// The append of a block that fits, for a group of layers (compact.hip).
struct CompactArgs {
  int c, n, t0, budget, n_kv_heads, head_dim;
  GroupStrides g;
  u16* k_cache;                 // the group's first layer
  u16* v_cache;
  int32_t* token_idx;
  float* weight;
  LayerBlock layer[kMaxGroupLayers];
};

// launchers (each returns the hipError_t of the launch)
hipError_t launch_attention(const AttnArgs& a, int head_dim, hipStream_t s);
hipError_t launch_attention_split(const AttnArgs& a, int head_dim, hipStream_t s);
hipError_t launch_colsum(const ColsumArgs& a, int head_dim, hipStream_t s);
hipError_t launch_select(const SelectArgs& a, int n_kv_heads, hipStream_t s);   // grid: heads x a.g.n_layers
hipError_t launch_move(const CompactArgs& a, hipStream_t s);
hipError_t launch_init(int32_t* token_idx, float* weight, size_t n_slots, const Seg* host_segs,
                       int n_segs, Seg* dev_segs, unsigned long long* totals, hipStream_t s);
int rows_per_compact_block(int head_dim);

// host-side planning shared by launchers and the state machine
void plan_attention(AttnArgs& a, int head_dim, int forced_shape);   // forced_shape < 0: chosen from the launch size
int attention_max_partials(int group, int n_q_heads, int chunk_max);   // most partial score arrays per KV head a launch leaves
constexpr int kMaxFusedPartials = 64;                   // beyond that the separate column-sum kernel scores
hipError_t prepare_attention_split();
hipError_t prepare_attention();   // function attributes on the current device; once per cache creation
hipError_t prepare_select();
void plan_colsum(ColsumArgs& a, int n_layers);
int colsum_max_partials(int group, int chunk_max);
size_t select_lds_bytes(const SelectArgs& a);
void plan_select(SelectArgs& a);
bool keydiff_in_compaction(int n_cand, int head_dim);
bool scores_keys_beside_attention(const AttnArgs& a, int n_layers, int n_cand, int head_dim);
int key_score_workgroups(int n_kv_heads);

}  // namespace kvp
