// Compaction of a layer's cache (Alg. 1 lines 8-11): per KV head the selection of the M candidates to keep
// (the lowest importance scores leave first, Sec. 3.2), the slots of the kept block tokens, the
// grid-neighbour merge of the evicted visual tokens, and the rows themselves, in place.
//
// One workgroup of 512 or 1024 threads (plan.cpp) per KV head and layer does all of it.  A head's rows that change are few
// (at 32/8 heads, 1024 new over 2048 cached: 175 merge destinations, 212 sources and 88 moved rows,
// 0.4 MB), so one CU moves them in a few microseconds, and one launch replaces three whose
// plans had to go through memory.  What bounds it is the chain of its phases: memory round trips,
// LDS atomics, block scans, barriers.  With 16 layers in a launch the chains of 128 heads run side by
// side.
//   * scores by the keys alone where the attention launch has not left them (key_scores.h): up to 1024 candidates at head
//     dimension 128 -- a launch pair of 9 us otherwise (keydiff.hip, which serves larger heads).
//   * other scores: the partial column sums of a head are added up by groups of threads, sixteen bytes per
//     load and sixteen loads in flight, each group every G-th array; the groups' sums meet in LDS, in a fixed order.
//   * order: 64-bit key = (score as order-preserving u32) << 32 | ~token, so
//     "higher score first, equal scores by lower token index" is "larger key
//     first" and all keys are distinct: the kept set is unique.  (Token indices that a caller wrote, kvp_set_state, may
//     repeat; the kernel then still ends and stays inside its memory.)
//   * the M-th largest key: one histogram of 2048 bins (512 with 512 threads) over the range the keys really span (a scale on
//     float bits, so roughly logarithmic in the score), the bin that holds it, and then a ranking of
//     the few keys in that bin by every wave for itself.  Should more than 64 keys share the bin
//     (equal scores) the range shrinks to the bin and the histogram is taken again (key_range.h).
//   * block-wide prefix sums rank the free slots and the kept block tokens;
//     the k-th kept block token (ascending token index) gets the k-th free slot.
//   * merge plan: a token -> position table over the cached tokens (block tokens map directly): one entry per
//     token of the prefix so far where that fits into LDS (some tens of thousands), a hash table
//     beyond.  Every evicted visual candidate looks at its grid neighbours, takes the kept one with the
//     largest key and writes itself into that destination's list of at most six sources.
//     (Walking the hash table was 3 of the 4.5 us of this phase: six chains of dependent LDS reads per lane,
//     and the wave waits for its longest.)  With one candidate per thread its owner does that as soon as it knows the
//     threshold, without a list of the evicted and the two barriers around it: 192 candidates, 4 heads of d 64
//     8.8 -> 7.7 us in a kernel trace, with the table's entries asked for together.
//   * merge: destination and sources of a row pair (the K row and the V row of one slot, 16 bytes per lane)
//     are fetched together, four destinations in flight per group of lanes; sources are sorted by
//     candidate position first, so that the fp32 sum is taken in one fixed order.  A destination in the
//     cache is rewritten in place (no other row reads it: sources are evicted rows, destinations kept
//     ones); one among the block's tokens goes to a staging row, because the slot it will get may
//     still be a source.  The staging rows lie over the head's own partial arrays, read by then.
//   * move: kept block rows, or their staging rows, into the free slots.
#include "key_scores.h"
#include "kvp_internal.h"
#include "lane_tools.h"

namespace kvp {

namespace {

constexpr int kMaxItemsAny = KVP_MAX_CANDIDATES / kSelectThreads;   // 8
constexpr unsigned kNone16 = 0xFFFFu;

__device__ __forceinline__ unsigned order_bits(float x) {
  if (x == 0.f) x = 0.f;   // -0 and +0 rank equal
  const unsigned u = __float_as_uint(x);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// x / w from the rounded reciprocal of w (Markstein): q is at most 1.5 units of its last place off, and with q's remainder added
// the last rounding is that of a number within 2^-22 units of x / w.  It goes the way of x / w's own, because w is a whole
// number, a merge multiplicity: for w up to 2^20 no quotient is that near to the middle of two fp32 numbers.
// Below 2^-126, where the remainder is rounded, the last fp32 bit may differ.  The fix-up puts infinities, zeros and NaN right.
__device__ __forceinline__ float divided(float x, float w, float inv) {
  const float q = x * inv;
  return __builtin_amdgcn_div_fixupf(__builtin_fmaf(__builtin_fmaf(-q, w, x), inv, q), w, x);
}

__device__ __forceinline__ unsigned hash_tok(int tok, unsigned mask) {
  unsigned x = (unsigned)tok * 0x9E3779B1u;
  x ^= x >> 15;
  return x & mask;
}

// Wave-wide scans and reductions on the DPP network (rows of 16 lanes, then across rows): a few cycles a
// step, where a shuffle through LDS costs a hundred.
template <int kCtrl, int kRowMask>
__device__ __forceinline__ unsigned dpp(unsigned identity, unsigned x) {
  return (unsigned)__builtin_amdgcn_update_dpp((int)identity, (int)x, kCtrl, kRowMask, 0xF, false);
}
template <class Op>
__device__ __forceinline__ unsigned wave_scan(unsigned x, unsigned identity, Op op) {     // inclusive
  x = op(x, dpp<0x111, 0xF>(identity, x));   // row_shr 1, 2, 4, 8
  x = op(x, dpp<0x112, 0xF>(identity, x));
  x = op(x, dpp<0x114, 0xF>(identity, x));
  x = op(x, dpp<0x118, 0xF>(identity, x));
  x = op(x, dpp<0x142, 0xA>(identity, x));   // the last lane of a row into the next row (rows 1 and 3)
  x = op(x, dpp<0x143, 0xC>(identity, x));   // the last lane of the first half into the second
  return x;
}
struct Add { __device__ __forceinline__ unsigned operator()(unsigned a, unsigned b) const { return a + b; } };
struct Min { __device__ __forceinline__ unsigned operator()(unsigned a, unsigned b) const { return a < b ? a : b; } };
struct Max { __device__ __forceinline__ unsigned operator()(unsigned a, unsigned b) const { return a > b ? a : b; } };
__device__ __forceinline__ unsigned last_lane(unsigned x) { return (unsigned)__builtin_amdgcn_readlane((int)x, 63); }

// word of histogram bin b: kPer neighbouring bins are a lane's, and the lanes of a wave read four of theirs at a
// time from consecutive 16-byte pieces (in bin order the pieces would lie 128 bytes apart, in two of the
// sixteen bank groups: 2 us of the selection)
template <unsigned kPer>
__device__ __forceinline__ unsigned bin_word(unsigned b) {
  static_assert(kPer >= 4 && (kPer & (kPer - 1)) == 0, "a permutation of the 64 kPer bins");
  return ((b % kPer >> 2) << 8) | (b / kPer << 2) | (b & 3u);
}

struct Lds {
  unsigned long long* key;    // [cand_pad] low word ~token, high word order-preserving score bits; at the end the
                              // high word is the staging row of a destination
  unsigned* cnt;              // [cand_pad / 4] one byte per candidate: sources that chose it
  unsigned short* evicted;    // [cand_pad] positions of the evicted candidates; later those of the moved rows
  unsigned short* free_slot;  // [cand_pad] free slots by rank
  unsigned* hist;             // [kBins]
  unsigned* table;    // token -> position of the cached tokens, u16; later the destinations
  float* sums;        // [groups][4 * quads] sums of the partial arrays by group
};

__device__ __forceinline__ void table_insert(unsigned* words, unsigned mask, int tok, unsigned pos) {
  unsigned h = hash_tok(tok, mask);
  for (;;) {
    unsigned* word = words + (h >> 1);
    const unsigned sh = (h & 1u) * 16u;
    unsigned old = *word;
    while (((old >> sh) & 0xFFFFu) == kNone16) {
      const unsigned nv = (old & ~(0xFFFFu << sh)) | (pos << sh);
      const unsigned prev = atomicCAS(word, old, nv);
      if (prev == old) return;
      old = prev;
    }
    h = (h + 1) & mask;
  }
}

__device__ __forceinline__ unsigned table_entry(const Lds& l, unsigned h) {
  return (l.table[h >> 1] >> ((h & 1u) * 16u)) & 0xFFFFu;
}

// position of cached token `tok`, or -1
__device__ __forceinline__ int probe(const Lds& l, unsigned mask, int tok) {
  unsigned h = hash_tok(tok, mask), e = table_entry(l, h);
  for (;;) {
    if (e == kNone16) return -1;
    if ((unsigned)l.key[e] == ~(unsigned)tok) return (int)e;
    h = (h + 1) & mask;
    e = table_entry(l, h);
  }
}

struct SegL {          // a prefix segment in LDS, with reciprocals for the coordinate split
  int begin, n, kind, gh, gw, planes, temporal, per;
  float inv_per, inv_gw;
};

// u / d and u % d for 0 <= u < 2^24, d >= 1, with a float reciprocal and one fix-up step
__device__ __forceinline__ void div_mod(int u, int d, float inv_d, int& q, int& r) {
  q = (int)((float)u * inv_d);
  r = u - q * d;
  if (r < 0) { r += d; --q; }
  if (r >= d) { r -= d; ++q; }
}

// grid neighbours of a visual token: left, right, up, down, previous plane, next plane;
// out[j] = -1 where there is none.  Returns false for a text token.
// (`first` is segs[0], which the caller has in registers: a prefix is mostly one visual segment with text behind it)
__device__ __forceinline__ bool neighbours(const SegL& first, const SegL* segs, int n_segs, int tok, int (&out)[kNeighbours]) {
#pragma unroll
  for (int j = 0; j < kNeighbours; ++j) out[j] = -1;
  SegL sg = first;
  bool found = tok >= first.begin && tok < first.begin + first.n;
  for (int s = 1; s < n_segs && __any(!found); ++s) {
    const int begin = segs[s].begin;
    if (found || tok < begin || tok >= begin + segs[s].n) continue;
    sg = segs[s];
    found = true;
  }
  if (!found || sg.kind != KVP_VISUAL) return false;
  int plane, rem, y, x;
  div_mod(tok - sg.begin, sg.per, sg.inv_per, plane, rem);
  div_mod(rem, sg.gw, sg.inv_gw, y, x);
  if (x > 0) out[0] = tok - 1;
  if (x + 1 < sg.gw) out[1] = tok + 1;
  if (y > 0) out[2] = tok - sg.gw;
  if (y + 1 < sg.gh) out[3] = tok + sg.gw;
  if (sg.temporal) {
    if (plane > 0) out[4] = tok - sg.per;
    if (plane + 1 < sg.planes) out[5] = tok + sg.per;
  }
  return true;
}

// One row pair of `D` channels: 2 D / 8 lanes of 16 bytes, K row then V row.
template <int D, int kThreads>
struct Lanes {
  static constexpr int kPerRow = D / 8;
  static constexpr int kPerPair = 2 * kPerRow;
  static constexpr int kPairs = kThreads / kPerPair;   // row pairs the workgroup carries at a time
};

// kMaxItems: candidates a thread can own (up to 4, i.e. up to 4096 candidates, with the source lists in LDS;
// 8 covers the limit, with the source lists in the scratch set)
template <int D, int kMaxItems, int kThreads>
__global__ void __launch_bounds__(kThreads)
compact_kernel(const SelectArgs args) {
  constexpr int kWaves = kThreads / 64;
  constexpr bool kListsInLds = kMaxItems <= 4;
  // (every wave searches the histogram for itself, and a few candidates need no fine one)
  constexpr int kBinBits = kThreads == 512 ? kSelectFewBinBits : kSelectBinBits, kBins = 1 << kBinBits;
  constexpr unsigned kPer = kBins / 64;
  extern __shared__ __align__(16) unsigned char lds_raw[];
  __shared__ unsigned long long s_members[64];
  __shared__ unsigned s_n_members, s_n_dst, s_n_src;
  __shared__ unsigned s_wave_tot[kWaves], s_wave_ev[kWaves], s_wave_min[kWaves], s_wave_max[kWaves];
  __shared__ SegL s_segs[KVP_MAX_SEGMENTS];

  const int hk = blockIdx.x, li = blockIdx.y;          // grid (KV heads, layers of the group)
  SelectPlan a = args;
  const u16* k_new = args.layer[li].k_new;
  const u16* v_new = args.layer[li].v_new;
  have_arguments(a.token_idx, a.partial, a.segs, a.weight, a.scores, a.k_cache, k_new, a.g.first_set, a.g.n_sets,
                 a.g.set_stride, a.g.kv_stride, a.g.meta_stride, a.c, a.n, a.t0, a.budget, a.partial_stride, a.cand_stride,
                 a.n_partials, a.merge, a.n_kv_heads, a.n_segs, a.items, a.table_size, a.quads, a.keydiff, a.width, a.groups);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int c = a.c, n_cand = c + a.n, budget = a.budget, items = a.items;
  const int cand_pad = items * kThreads;
  const unsigned mask = (unsigned)a.table_size - 1u;
  int* const token_idx = a.token_idx + (long long)li * a.g.meta_stride + (size_t)hk * budget;
  float* const weight = a.weight + (long long)li * a.g.meta_stride + (size_t)hk * budget;

  Lds l;
  unsigned short* sources;                             // [candidate][kNeighbours]
  {
    unsigned char* p = lds_raw;
    l.key = reinterpret_cast<unsigned long long*>(p); p += (size_t)cand_pad * 8;
    l.cnt = reinterpret_cast<unsigned*>(p); p += (size_t)cand_pad;
    l.evicted = reinterpret_cast<unsigned short*>(p); p += (size_t)cand_pad * 2;
    l.free_slot = reinterpret_cast<unsigned short*>(p); p += (size_t)cand_pad * 2;
    l.hist = reinterpret_cast<unsigned*>(p); p += kBins * 4;
    l.table = reinterpret_cast<unsigned*>(p); p += (size_t)a.table_size * 2;
    if constexpr (kListsInLds) {
      l.sums = reinterpret_cast<float*>(p);            // dead when the lists begin
      sources = reinterpret_cast<unsigned short*>(p);
    } else {
      l.sums = reinterpret_cast<float*>(l.evicted);    // one group; dead when those lists begin
      sources = in_set_of(a.sources, a.g, li) + (size_t)hk * a.cand_stride * kNeighbours;
    }
  }
  unsigned* const key_words = reinterpret_cast<unsigned*>(l.key);
  unsigned short* const direct = reinterpret_cast<unsigned short*>(l.table);

  // ---- token indices, the token -> position table of the cached ones, and the sums of the partial arrays:
  // the threads are `groups` groups of `width`; thread t adds up the fours of neighbouring candidates
  // t % width, + width, ... over the arrays t / width, + groups, ...
  {
    // (token indices and segments are asked for first and used last, without a condition: one that is loaded under a
    // condition is waited for on the spot, before the sums are on their way)
    int tokv[kMaxItems];
#pragma unroll
    for (int i = 0; i < kMaxItems; ++i) tokv[i] = token_idx[max(min(tid + i * kThreads, c - 1), 0)];
    const Seg my_seg = a.segs[min(tid, a.n_segs - 1)];
    for (int i = tid; i < kBins; i += kThreads) l.hist[i] = 0u;
    if (tid == 0) { s_n_members = 0u; s_n_dst = 0u; s_n_src = 0u; }
    if (a.merge) {
      for (int i = tid; i < a.table_size / 8; i += kThreads)
        reinterpret_cast<uint4*>(l.table)[i] = make_uint4(0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu);
      for (int i = tid; i < cand_pad / 4; i += kThreads) l.cnt[i] = 0u;
    }
    if (a.score_override) {
      for (int p = tid; p < n_cand; p += kThreads) l.sums[p] = a.score_override[(size_t)hk * n_cand + p];
    } else if (kThreads == 512 && a.keydiff) {
      score_head_by_keys<D>(a.k_cache + (long long)li * a.g.kv_stride + (size_t)hk * budget * D, k_new + (size_t)hk * D,
                            a.n_kv_heads, c, n_cand, l.sums + 4 * a.quads, l.sums);
    } else {
      // (a group is whole waves: what a wave loads is decided by scalar branches)
      const int grp = __builtin_amdgcn_readfirstlane(tid >> a.width_log2), quad0 = tid & (a.width - 1);
      const int n_arrays = grp < a.groups ? (int)quotient((unsigned)(a.n_partials - grp + a.groups - 1), a.groups_magic) : 0;
      // a scalar base per array, lane offsets that never change (past the end: the last four candidates again, not stored)
      const float* part = in_set_of(a.partial, a.g, li) + (size_t)hk * a.partial_stride + grp * a.cand_stride;
      const int step = a.groups * a.cand_stride;
      // (as many passes as the candidates of this kernel need, and sixteen loads in flight with them.  With four passes wherever
      // a group does not cover the candidates at once, half of the loads of 1536 candidates were the last four again: 56 arrays
      // of them 8.3 -> 4.2 us)
      constexpr int kWidth = kMaxItems > 4 ? kThreads : 256, kPasses = (kMaxItems * kThreads / 4 + kWidth - 1) / kWidth;
      constexpr int kBatch = 16 / kPasses;
      float4 acc[kPasses];
      unsigned lane_off[kPasses];
#pragma unroll
      for (int s = 0; s < kPasses; ++s) {
        acc[s] = make_float4(0.f, 0.f, 0.f, 0.f);
        lane_off[s] = 4u * (unsigned)min(quad0 + s * a.width, a.quads - 1);
      }
      for (int first = 0; first < n_arrays; first += kBatch) {
        float4 v[kBatch][kPasses];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
#pragma unroll
          for (int s = 0; s < kPasses; ++s) v[u][s] = make_float4(0.f, 0.f, 0.f, 0.f);
          if (first + u < n_arrays) {
#pragma unroll
            for (int s = 0; s < kPasses; ++s) v[u][s] = *reinterpret_cast<const float4*>(part + lane_off[s]);
            part += step;
          }
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u)
#pragma unroll
          for (int s = 0; s < kPasses; ++s) {
            acc[s].x += v[u][s].x; acc[s].y += v[u][s].y; acc[s].z += v[u][s].z; acc[s].w += v[u][s].w;
          }
      }
#pragma unroll
      for (int s = 0; s < kPasses; ++s)
        if (n_arrays > 0 && quad0 + s * a.width < a.quads)
          *reinterpret_cast<float4*>(l.sums + (size_t)(grp * a.quads + quad0 + s * a.width) * 4) = acc[s];
    }
#pragma unroll
    for (int i = 0; i < kMaxItems; ++i) {
      const int p = tid + i * kThreads;
      if (p >= c) tokv[i] = a.t0 + (p - c);
      if (i < items && p < n_cand) key_words[2 * p] = ~(unsigned)tokv[i];
    }
    if (tid < a.n_segs) {
      SegL sl;
      sl.begin = my_seg.begin; sl.n = my_seg.n; sl.kind = my_seg.kind; sl.gh = my_seg.gh; sl.gw = my_seg.gw;
      sl.planes = my_seg.planes; sl.temporal = my_seg.temporal;
      sl.per = sl.gh * sl.gw;
      sl.inv_per = sl.per > 0 ? 1.f / (float)sl.per : 0.f;
      sl.inv_gw = sl.gw > 0 ? 1.f / (float)sl.gw : 0.f;
      s_segs[tid] = sl;
    }
    __syncthreads();
    if (a.merge) {
#pragma unroll
      for (int i = 0; i < kMaxItems; ++i) {
        const int p = tid + i * kThreads;
        if (i < items && p < c) {
          // (a cache that was loaded from outside may hold any token index: one that is not below t0 has no entry)
          if (!a.direct) table_insert(l.table, mask, tokv[i], (unsigned)p);
          else if ((unsigned)tokv[i] < (unsigned)a.t0) direct[tokv[i]] = (unsigned short)p;
        }
      }
    }
  }

  // (what the phases from here on use; loaded again in each of them, with a wait every time: ten blocks of 64 tokens,
  // 4 heads of d 64, 192 candidates: 126.3 -> 123.3 us.  With the rows' pointers, too, four heads of d 128 and 768 candidates
  // lost 0.3 %)
  keep_arguments(a.scores, a.keep, a.dst, a.g.first_set, a.g.n_sets, a.g.set_stride, a.cand_stride, a.t0, a.merge, a.n_segs, a.direct,
                 c, n_cand, budget, items);

  SegL first_seg;
  if (a.merge) first_seg = s_segs[0];

  // ---- own candidates, blocked: thread t owns positions [t * items, (t + 1) * items)
  float* const scores = in_set_of(a.scores, a.g, li) + (size_t)hk * a.cand_stride;
  unsigned long long key[kMaxItems];
  bool valid[kMaxItems];
  unsigned ob_min = 0xFFFFFFFFu, ob_max = 0u;
#pragma unroll
  for (int i = 0; i < kMaxItems; ++i) {
    const int p = tid * items + i;
    valid[i] = i < items && p < n_cand;
    key[i] = 0ull;
    if (valid[i]) {
      float s = l.sums[p];
      for (int grp = 1; grp < a.groups; ++grp) s += l.sums[(size_t)grp * a.quads * 4 + p];
      scores[p] = s;
      const unsigned ob = order_bits(s);
      key[i] = ((unsigned long long)ob << 32) | key_words[2 * p];
      key_words[2 * p + 1] = ob;
      ob_min = min(ob_min, ob);
      ob_max = max(ob_max, ob);
    }
  }
  ob_min = last_lane(wave_scan(ob_min, 0xFFFFFFFFu, Min{}));
  ob_max = last_lane(wave_scan(ob_max, 0u, Max{}));
  if (lane == 0) { s_wave_min[wave] = ob_min; s_wave_max[wave] = ob_max; }
  __syncthreads();
#pragma unroll
  for (int w2 = 0; w2 < kWaves; ++w2) { ob_min = min(ob_min, s_wave_min[w2]); ob_max = max(ob_max, s_wave_max[w2]); }

  // ---- the budget-th largest key
  unsigned long long threshold;
  {
    KeyRangeOf<kBinBits> range = KeyRangeOf<kBinBits>::over(ob_min, ob_max);
    unsigned want = (unsigned)budget, in_bin = 0;
    for (;;) {
#pragma unroll
      for (int i = 0; i < kMaxItems; ++i)
        if (unsigned bin; valid[i] && range.holds(key[i], bin)) atomicAdd(&l.hist[bin_word<kPer>(bin)], 1u);
      __syncthreads();
      // every wave finds the bin for itself: lane L adds up bins kPer L .. kPer L + kPer - 1, a scan over the lanes finds
      // the lane with the wanted key, and a second one, of that lane's bins, the bin
      unsigned mine = 0;
#pragma unroll
      for (int b = 0; b < kBins / 64; b += 4) {
        const uint4 v = *reinterpret_cast<const uint4*>(&l.hist[64 * b + 4 * lane]);
        mine += v.x + v.y + v.z + v.w;
      }
      const unsigned upto = wave_scan(mine, 0u, Add{});
      const unsigned above = last_lane(upto) - upto;                 // keys in the bins of higher lanes
      const int owner = __builtin_ctzll(__ballot(above < want && want <= above + mine));
      want -= (unsigned)__builtin_amdgcn_readlane((int)above, owner);
      const unsigned one = lane < (int)kPer ? l.hist[bin_word<kPer>(kPer * (unsigned)owner + (unsigned)lane)] : 0u;
      const unsigned upto1 = wave_scan(one, 0u, Add{});
      const unsigned above1 = last_lane(upto1) - upto1;
      const int from = __builtin_ctzll(__ballot(above1 < want && want <= above1 + one));
      const unsigned digit = kPer * (unsigned)owner + (unsigned)from;
      want -= (unsigned)__builtin_amdgcn_readlane((int)above1, from);
      in_bin = (unsigned)__builtin_amdgcn_readlane((int)one, from);
      range.enter(digit);
      // (one key to a bin and still more than 64 of them: cached slots that share score and token index)
      if (in_bin <= 64u || range.shift == 0) break;
      // more than a wave can rank: look into this bin alone
      range.divide();
      __syncthreads();                                 // everybody has read the histogram
      for (int i = tid; i < kBins; i += kThreads) l.hist[i] = 0u;
      __syncthreads();
    }
    if (in_bin > 64u) {
      threshold = range.lo;
    } else {
#pragma unroll
      for (int i = 0; i < kMaxItems; ++i)
        if (unsigned bin; valid[i] && range.holds(key[i], bin)) s_members[atomicAdd(&s_n_members, 1u)] = key[i];
      __syncthreads();
      const unsigned long long k = lane < (int)in_bin ? s_members[lane] : 0ull;
      unsigned rank = 0;
      for (unsigned i = 0; i < in_bin; i += 4) {             // (four reads in flight; past the end: zeros or old keys, not counted)
        unsigned long long other[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) other[u] = s_members[i + u];
#pragma unroll
        for (int u = 0; u < 4; ++u) rank += i + u < in_bin && other[u] > k ? 1u : 0u;
      }
      // (members that are equal share the rank of the first of them: the last rank up to the wanted one that there is)
      unsigned long long at = 0ull;
      for (unsigned r = want; at == 0ull && r > 0u; --r) at = __ballot(lane < (int)in_bin && rank == r - 1u);
      const int from = __builtin_ctzll(at);
      threshold = ((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(k >> 32), from) << 32) |
                  (unsigned)__builtin_amdgcn_readlane((int)(unsigned)k, from);
    }
  }

  // ---- keep flags; rank the free slots, the kept block tokens and the evicted candidates
  // (one candidate per thread: its owner plans the merge of an evicted one, before the barrier that the ranks wait for.  With more
  // of them, an owner would plan one after the other: there the list deals them out to all threads.)
  constexpr bool kOwnPlan = kMaxItems == 1;
  uint8_t* const keep_out = in_set_of(a.keep, a.g, li) + (size_t)hk * a.cand_stride;
  int32_t* const dst_out = in_set_of(a.dst, a.g, li) + (size_t)hk * a.cand_stride;
  // ---- merge plan: evicted candidate p picks its best kept grid neighbour and enters itself there
  auto plan_merge = [&](int p, int tok) __attribute__((always_inline)) {
    int best = -1;
    int nb[kNeighbours];
    if (neighbours(first_seg, s_segs, a.n_segs, tok, nb)) {
      // of cached slots that share a token index the one in the table merges: a destination then has at most
      // one source per neighbour, which is what its list has room for
      // (the two kinds of table are asked in branches of their own, so that the entries of the direct one come together:
      // with the choice inside, each was waited for before the next was asked for, 0.4 us)
      int self = p, r[kNeighbours];
      if (a.direct) {
        const unsigned self_entry = direct[(unsigned)tok < (unsigned)a.t0 ? tok : 0];
        unsigned entry[kNeighbours];
#pragma unroll
        for (int j = 0; j < kNeighbours; ++j) entry[j] = direct[(unsigned)nb[j] < (unsigned)a.t0 ? nb[j] : 0];
#pragma unroll
        for (int j = 0; j < kNeighbours; ++j) r[j] = (unsigned)nb[j] < (unsigned)a.t0 && entry[j] != kNone16 ? (int)entry[j] : -1;
        if (p < c) self = (unsigned)tok < (unsigned)a.t0 ? (int)self_entry : -1;
      } else {
        if (p < c) self = probe(l, mask, tok);
#pragma unroll
        for (int j = 0; j < kNeighbours; ++j) r[j] = (unsigned)nb[j] < (unsigned)a.t0 ? probe(l, mask, nb[j]) : -1;
      }
      // (a token of the block sits at a known position, one after it nowhere)
#pragma unroll
      for (int j = 0; j < kNeighbours; ++j)
        if (nb[j] >= a.t0 && nb[j] < a.t0 + (n_cand - c)) r[j] = c + (nb[j] - a.t0);
      unsigned long long kr[kNeighbours], best_key = 0;
#pragma unroll
      for (int j = 0; j < kNeighbours; ++j) kr[j] = l.key[max(r[j], 0)];
#pragma unroll
      for (int j = 0; j < kNeighbours; ++j)
        if (r[j] >= 0 && kr[j] >= threshold && (best < 0 || kr[j] > best_key)) { best = r[j]; best_key = kr[j]; }
      if (self != p) best = -1;
    }
    dst_out[p] = best;
    if (best >= 0) {
      const unsigned old = atomicAdd(&l.cnt[best >> 2], 1u << (8 * (best & 3)));
      sources[best * kNeighbours + ((old >> (8 * (best & 3))) & 0xFFu)] = (unsigned short)p;
    }
    const unsigned long long merged = __ballot(best >= 0);
    if (merged && lane == __builtin_ctzll(__ballot(true))) atomicAdd(&s_n_src, (unsigned)__builtin_popcountll(merged));
  };
  bool keep[kMaxItems];
  unsigned n_free = 0, n_new = 0, n_ev = 0;
#pragma unroll
  for (int i = 0; i < kMaxItems; ++i) {
    const int p = tid * items + i;
    keep[i] = valid[i] && key[i] >= threshold;
    if (valid[i]) {
      keep_out[p] = keep[i];
      if (!a.merge || keep[i]) dst_out[p] = -1;        // an evicted candidate's is written by the merge plan
      if (p < budget && (p >= c || !keep[i])) ++n_free;
      if (p >= c && keep[i]) ++n_new;
      if (!keep[i]) ++n_ev;
    }
  }
  const unsigned packed = n_free | (n_new << 16);
  const unsigned incl = wave_scan(packed, 0u, Add{});
  unsigned incl_ev = 0;
  if constexpr (!kOwnPlan) incl_ev = wave_scan(n_ev, 0u, Add{});
  if (lane == 63) { s_wave_tot[wave] = incl; s_wave_ev[wave] = incl_ev; }
  if (kOwnPlan && a.merge && valid[0] && !keep[0]) plan_merge(tid, (int)~(unsigned)key[0]);
  __syncthreads();
  unsigned base = incl - packed, base_ev = incl_ev - n_ev;
  unsigned total = 0, total_ev = 0;
#pragma unroll
  for (int w2 = 0; w2 < kWaves; ++w2) {
    const unsigned t = s_wave_tot[w2], te = s_wave_ev[w2];
    if (w2 < wave) { base += t; base_ev += te; }
    total += t; total_ev += te;
  }
  unsigned base_free = base & 0xFFFFu;
  const unsigned base_new = base >> 16;
  // (distinct keys: as many slots as new rows.  Slots that share a key with the threshold all stay, and the last of the
  // block's rows find no slot.)
  const unsigned total_new = min(total >> 16, total & 0xFFFFu);
#pragma unroll
  for (int i = 0; i < kMaxItems; ++i) {
    const int p = tid * items + i;
    if (valid[i]) {
      if (p < budget && (p >= c || !keep[i])) l.free_slot[base_free++] = (unsigned short)p;
      if (!kOwnPlan && !keep[i]) l.evicted[base_ev++] = (unsigned short)p;
    }
  }
  if constexpr (!kOwnPlan) __syncthreads();

  using L = Lanes<D, kThreads>;
  const int sub = tid % L::kPerPair;
  const bool is_v = sub >= L::kPerRow;
  const int piece = sub % L::kPerRow;
  // (both candidates of a choice are formed outside of it: a load of an argument whose address depends on a
  // per-lane condition would push the arguments to memory)
  u16* const k_cache = a.k_cache;
  u16* const v_cache = a.v_cache;
  u16* const stage_k = in_set_of(a.stage, a.g, li) + 2 * (size_t)hk * a.partial_stride;
  u16* const stage_v = stage_k + (size_t)a.chunk_max * D;
  u16* const cache = (is_v ? v_cache : k_cache) + (long long)li * a.g.kv_stride + (size_t)hk * budget * D + 8 * piece;
  const u16* const fresh = (is_v ? v_new : k_new) + (size_t)hk * D + 8 * piece;
  const int fresh_stride = a.n_kv_heads * D;
  u16* const staged = (is_v ? stage_v : stage_k) + 8 * piece;
  float* const staged_w = in_set_of(a.stage_w, a.g, li) + (size_t)hk * a.chunk_max;

  if (a.merge && !kOwnPlan) {
    // (one evicted candidate per thread, whichever threads own them)
    for (unsigned e = tid; e < total_ev; e += kThreads) plan_merge((int)l.evicted[e], (int)~key_words[2 * l.evicted[e]]);
    __syncthreads();
  }

  // ---- the destinations that were chosen, in any order (which staging row one gets is nobody's
  // business), and the block rows to move, by rank
  unsigned short* const dests = reinterpret_cast<unsigned short*>(l.table);
  unsigned short* const moved = l.evicted;
  {
    unsigned rank = base_new;
#pragma unroll
    for (int i = 0; i < kMaxItems; ++i) {
      if (!valid[i]) continue;
      const int p = tid * items + i;
      if (p >= c && keep[i]) moved[rank++] = (unsigned short)p;
      if (a.merge) {
        const unsigned k = (l.cnt[p >> 2] >> (8 * (p & 3))) & 0xFFu;
        if (k) {
          const unsigned at = atomicAdd(&s_n_dst, 1u);
          dests[at] = (unsigned short)p;
          key_words[2 * p + 1] = at;
        }
      }
    }
  }
  __syncthreads();

  // Running totals for the benchmark's byte counts (integer atomics: the order does not matter), a lane of the last wave each, on their way
  // while the rows move.  The heads of all dies add to one line of memory: by one lane after the other, at the kernel's end, that kept it
  // from ending for 0.35 us (4 heads) to 2.8 (128).  4 layers of 32 heads of d 128, 384 candidates, a whole prefix 191.6 -> 178.5 us.
  static_assert(KVP_T_EVICTING_HEADS == 0 && KVP_T_MOVED_ROWS == 1 && KVP_T_MERGE_DESTINATIONS == 2 && KVP_T_MERGE_SOURCES == 3);
  if (const int t = tid - (kThreads - 64); t >= 0 && t < (a.merge ? 4 : 2))
    atomicAdd(&a.totals[t], (unsigned long long)(t == 0 ? 1u : t == 1 ? total_new : t == 2 ? s_n_dst : s_n_src));

  if (a.merge) {
    const int n_dst = (int)s_n_dst;
    auto row_at = [&](int pos) __attribute__((always_inline)) {
      return *reinterpret_cast<const uint4*>(row_of_two<unsigned long long>(cache, 2 * D, fresh, 2 * (unsigned)fresh_stride, pos, c));
    };
    auto weight_at = [&](int pos) __attribute__((always_inline)) { return pos < c ? weight[pos] : 1.f; };
    // sources of destination p in ascending position, unused entries last
    auto sorted_sources = [&](int p, int n_src, int (&pos)[kNeighbours]) __attribute__((always_inline)) {
#pragma unroll
      for (int k = 0; k < kNeighbours; ++k) pos[k] = k < n_src ? (int)sources[p * kNeighbours + k] : 0x7FFFFFFF;
#pragma unroll
      for (int pass = 0; pass < kNeighbours; ++pass)
#pragma unroll
        for (int k = pass & 1; k + 1 < kNeighbours; k += 2) {
          const int lo = min(pos[k], pos[k + 1]), hi = max(pos[k], pos[k + 1]);
          pos[k] = lo; pos[k + 1] = hi;
        }
    };
    // The destination and its first two sources, which is all that most have, are fetched for four
    // destinations at a time; further sources follow when the destination's turn has come.
    constexpr int kFlight = 4, kEarly = 2;
    for (int at0 = tid / L::kPerPair; at0 < n_dst; at0 += kFlight * L::kPairs) {
      int pos[kFlight], n_src[kFlight];
      float wt[kFlight][kEarly + 1];
      uint4 rows[kFlight][kEarly + 1];
#pragma unroll
      for (int u = 0; u < kFlight; ++u) {
        const int at = at0 + u * L::kPairs;
        pos[u] = 0; n_src[u] = 0;
#pragma unroll
        for (int k = 0; k <= kEarly; ++k) { wt[u][k] = 0.f; rows[u][k] = make_uint4(0u, 0u, 0u, 0u); }
        if (at < n_dst) {
          const int p = dests[at];
          int from[kNeighbours];
          pos[u] = p;
          n_src[u] = (int)((l.cnt[p >> 2] >> (8 * (p & 3))) & 0xFFu);
          if (__all(n_src[u] <= kEarly)) {               // (what most have)
            const int one = sources[p * kNeighbours], other = sources[p * kNeighbours + 1];
            from[0] = n_src[u] == 2 ? min(one, other) : one;
            from[1] = max(one, other);
          } else {
            sorted_sources(p, n_src[u], from);
          }
          rows[u][0] = row_at(p);
          wt[u][0] = weight_at(p);
#pragma unroll
          for (int k = 0; k < kEarly; ++k)
            if (k < n_src[u]) { rows[u][k + 1] = row_at(from[k]); wt[u][k + 1] = weight_at(from[k]); }
        }
      }
#pragma unroll
      for (int u = 0; u < kFlight; ++u) {
        const int at = at0 + u * L::kPairs;
        if (at >= n_dst) continue;
        const int p = pos[u];
        float sum_w = wt[u][0];
        float acc[8];
        {
          const unsigned w[4] = {rows[u][0].x, rows[u][0].y, rows[u][0].z, rows[u][0].w};
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            acc[2 * k] = wt[u][0] * bf16_lo(w[k]);
            acc[2 * k + 1] = wt[u][0] * bf16_hi(w[k]);
          }
        }
        auto add = [&](const uint4& row, float wgt) __attribute__((always_inline)) {
          sum_w += wgt;
          const unsigned w[4] = {row.x, row.y, row.z, row.w};
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            acc[2 * k] = __builtin_fmaf(wgt, bf16_lo(w[k]), acc[2 * k]);
            acc[2 * k + 1] = __builtin_fmaf(wgt, bf16_hi(w[k]), acc[2 * k + 1]);
          }
        };
#pragma unroll
        for (int k = 0; k < kEarly; ++k)
          if (k < n_src[u]) add(rows[u][k + 1], wt[u][k + 1]);
        if (n_src[u] > kEarly) {
          int from[kNeighbours];
          sorted_sources(p, n_src[u], from);
          uint4 late[kNeighbours - kEarly];
          float late_w[kNeighbours - kEarly];
#pragma unroll
          for (int k = kEarly; k < kNeighbours; ++k) {
            late[k - kEarly] = make_uint4(0u, 0u, 0u, 0u);
            late_w[k - kEarly] = 0.f;
            if (k < n_src[u]) { late[k - kEarly] = row_at(from[k]); late_w[k - kEarly] = weight_at(from[k]); }
          }
#pragma unroll
          for (int k = kEarly; k < kNeighbours; ++k)
            if (k < n_src[u]) add(late[k - kEarly], late_w[k - kEarly]);
        }
        const float inv = 1.f / sum_w;                 // (eight divisions by the same weight: one, and a correction each)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = divided(acc[e], sum_w, inv);
        uint4 res;
        res.x = pack_bf16(acc[0], acc[1]);
        res.y = pack_bf16(acc[2], acc[3]);
        res.z = pack_bf16(acc[4], acc[5]);
        res.w = pack_bf16(acc[6], acc[7]);
        if (p < c) {
          *reinterpret_cast<uint4*>(cache + (size_t)p * D) = res;
          if (sub == 0) weight[p] = sum_w;
        } else {
          *reinterpret_cast<uint4*>(staged + (size_t)at * D) = res;
          if (sub == 0) staged_w[at] = sum_w;
        }
      }
    }
    __syncthreads();                                   // sources have been read, staging rows written
  }

  // ---- kept block rows into the free slots, eight per group of lanes in flight
  {
    constexpr int kFlight = 8;
    for (int i0 = tid / L::kPerPair; i0 < (int)total_new; i0 += kFlight * L::kPairs) {
      uint4 row[kFlight];
      float wt[kFlight];
      int pos[kFlight];
#pragma unroll
      for (int u = 0; u < kFlight; ++u) {
        const int i = i0 + u * L::kPairs;
        row[u] = make_uint4(0u, 0u, 0u, 0u);
        wt[u] = 1.f;
        pos[u] = 0;
        if (i < (int)total_new) {
          const int p = moved[i];
          const bool merged = a.merge && ((l.cnt[p >> 2] >> (8 * (p & 3))) & 0xFFu) != 0u;
          const int at = merged ? (int)key_words[2 * p + 1] : 0;
          pos[u] = p;
          row[u] = *reinterpret_cast<const uint4*>(merged ? staged + (size_t)at * D : fresh + (size_t)(p - c) * fresh_stride);
          if (merged) wt[u] = staged_w[at];
        }
      }
#pragma unroll
      for (int u = 0; u < kFlight; ++u) {
        const int i = i0 + u * L::kPairs;
        if (i < (int)total_new) {
          const int slot = l.free_slot[i];
          *reinterpret_cast<uint4*>(cache + (size_t)slot * D) = row[u];
          if (sub == 0) {
            token_idx[slot] = a.t0 + (pos[u] - c);
            weight[slot] = wt[u];
          }
        }
      }
    }
  }
}

template <int D>
hipError_t launch_head_dim(const SelectArgs& a, int n_kv_heads, hipStream_t s) {
  const size_t lds = select_lds_bytes(a);
  const dim3 grid(n_kv_heads, a.g.n_layers);
  // (built for one and two candidates per thread: what a loop over four of them skips is a fifth of the instructions there;
  // with the 512 bins and one reciprocal per merged row 4 heads of d 64, 192 candidates 9.8 -> 9.2 us, 4 heads of d 128, 768
  // candidates 8.0 -> 7.6 us; with the arguments in registers 8.7 and 7.4.
  // Of 1024 threads for two, three and four, against four alone: a whole prefix of 4 heads of d 64, 1444 candidates, 24 layers
  // 7719 -> 7689 us, of 4 heads of d 128, 1536 candidates, 16 layers, scored by the prompt 4697 -> 4687 us, of 8 heads of d 128,
  // 3072 candidates, 32 layers 33908 -> 33850 us; runs of one side differ by 0.1 %)
  if (a.items > 4) hipLaunchKernelGGL((compact_kernel<D, kMaxItemsAny, 1024>), grid, dim3(1024), lds, s, a);
  else if (a.threads == 1024 && a.items == 4) hipLaunchKernelGGL((compact_kernel<D, 4, 1024>), grid, dim3(1024), lds, s, a);
  else if (a.threads == 1024 && a.items == 3) hipLaunchKernelGGL((compact_kernel<D, 3, 1024>), grid, dim3(1024), lds, s, a);
  else if (a.threads == 1024) hipLaunchKernelGGL((compact_kernel<D, 2, 1024>), grid, dim3(1024), lds, s, a);
  else if (a.items > 2) {
    // (512 threads and more than 1024 candidates: scored by the keys, of which they hold 2048 at d 64 only)
    if constexpr (D == 64) hipLaunchKernelGGL((compact_kernel<D, 4, 512>), grid, dim3(512), lds, s, a);
    else return hipErrorInvalidValue;
  } else if (a.items == 2) hipLaunchKernelGGL((compact_kernel<D, 2, 512>), grid, dim3(512), lds, s, a);
  else hipLaunchKernelGGL((compact_kernel<D, 1, 512>), grid, dim3(512), lds, s, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_select(const SelectArgs& a, int n_kv_heads, hipStream_t s) {
  return a.head_dim == 128 ? launch_head_dim<128>(a, n_kv_heads, s) : launch_head_dim<64>(a, n_kv_heads, s);
}

// Allows the kernels the dynamic LDS of the largest head they can be given (the attribute
// belongs to the function on the current device: called at cache creation).
hipError_t prepare_select() {
  for (const void* fn : {reinterpret_cast<const void*>(compact_kernel<64, 1, 512>), reinterpret_cast<const void*>(compact_kernel<128, 1, 512>),
                         reinterpret_cast<const void*>(compact_kernel<64, 2, 512>), reinterpret_cast<const void*>(compact_kernel<128, 2, 512>),
                         reinterpret_cast<const void*>(compact_kernel<64, 4, 512>),
                         reinterpret_cast<const void*>(compact_kernel<64, 2, 1024>), reinterpret_cast<const void*>(compact_kernel<128, 2, 1024>),
                         reinterpret_cast<const void*>(compact_kernel<64, 3, 1024>), reinterpret_cast<const void*>(compact_kernel<128, 3, 1024>),
                         reinterpret_cast<const void*>(compact_kernel<64, 4, 1024>), reinterpret_cast<const void*>(compact_kernel<128, 4, 1024>),
                         reinterpret_cast<const void*>(compact_kernel<64, kMaxItemsAny, 1024>),
                         reinterpret_cast<const void*>(compact_kernel<128, kMaxItemsAny, 1024>)}) {
    const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kSelectLdsLimit);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace kvp
