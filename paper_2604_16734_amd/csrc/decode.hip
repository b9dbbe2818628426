// One decode step of one layer (Eq. 1 with a single query row per head, Sec. 2.1):
// the current token's queries attend over the layer's cache entries and over the
// keys and values of the tokens generated so far, the current one included (the
// "tail", which the caller keeps).
//
// Bound by latency long before HBM: 2049 keys of eight KV heads are 8.4 MB, a microsecond and a half of
// memory bandwidth, and a launch costs more than that.  So a thread has all its loads in flight
// together (one trip to memory), everything that crosses lanes goes over the DPP network or the
// lane-swap instructions instead of through LDS (butterflies by shuffle were half of the 11 us a step
// used to take), and waves meet once or twice.
//
// A thread holds one 8-channel piece of some K rows and of the same V rows, with coalesced 16-byte loads.
//   scores   it dots its pieces with the query; the pieces of a row sit in neighbouring lanes and are
//            added on the DPP network, so that every lane of a row knows its logit;
//   weights  every lane then has the exponentials of its own rows, against a maximum of the wave or the
//            workgroup;
//   values   with few rows per thread, or few query heads per KV head, it scales its V pieces, and the sums over the rows of a
//            wave are taken pairwise by lane swaps (a swap and an addition halve two values at once); else the products of weights and
//            values, sums over the wave included, are matrix instructions (weigh_rows).  Those over the waves go through LDS.
// Two ways to spread the work:
//   few keys (up to 640 at head dimension 128): one workgroup of 1024 threads per QUERY head takes all of
//            them and writes the result, one launch.  (A CU takes 64 bytes a clock from L2: beyond
//            about 700 keys that costs more than the second launch below.)  The kernel is built for each
//            number of rows a thread may hold, one to ten: rows past the end are loaded again at full price,
//            so a step takes the fewest that cover its keys.  4.3 us per layer at 32/32 heads, 265 keys, 5.4 at 28/4 heads, 553
//            keys;
//   else     a workgroup of 256 threads takes 64 keys of one KV head at a time for all G query heads of
//            the group and leaves (unnormalised output, maximum, sum) per query head; a second kernel
//            folds the workgroups' partials in a fixed order and rounds once to bfloat16.
#include <mutex>

#include "kvp_internal.h"
#include "lane_tools.h"
#include "mfma_tools.h"

// Scratch of kvp_decode_step_static (the entry point for callers that cannot allocate): the
// partial results of the step, KVP_STATIC_SCRATCH_BYTES per GPU, held until the process ends.
static __device__ __align__(256) float scratch[KVP_STATIC_SCRATCH_BYTES / sizeof(float)];

namespace kvp {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int kHeadThreads = 1024;   // of the one-workgroup-per-query-head kernel
constexpr int kTile = kDecodeTile;   // keys per workgroup step
constexpr int kGroupLimit = kDecodeGroupLimit;   // query heads per KV head

// a piece of key or value j of a KV head's list: cache slot j for j < c, then the tail rows
template <int D, class Offset>
struct Rows {
  const u16* cached;
  const u16* tail;
  unsigned tail_bytes;
  int c;
  __device__ __forceinline__ Rows(const u16* cache, const u16* tail_rows, const DecodeArgs& a, int hk, int piece)
      : cached(cache + (size_t)hk * a.budget * D + 8 * piece), tail(tail_rows + (size_t)hk * D + 8 * piece),
        tail_bytes(2u * (unsigned)(a.n_kv_heads * D)), c(a.c) {}
  __device__ __forceinline__ uint4 load(int j) const {
    return *reinterpret_cast<const uint4*>(row_of_two<Offset>(cached, 2u * D, tail, tail_bytes, j, c));
  }
};

__device__ __forceinline__ u16 round_bf16(float r) {
  unsigned u = __float_as_uint(r);               // round to nearest even
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (u16)(u >> 16);
}

// (pairs of bf16 products into an fp32 sum: both are bf16 in memory, the products exact, and the sum of a pair is rounded once;
// denormal keys and queries count in full)
__device__ __forceinline__ float dot8(const uint4 k, const uint4 q) {
  float s = dot2(k.x, q.x, 0.f);
  s = dot2(k.y, q.y, s);
  s = dot2(k.z, q.z, s);
  return dot2(k.w, q.w, s);
}

// The products of weights with value rows, on the matrix cores without a move between lanes.  A lane has 8 channels of one row with each
// of its loads, the lanes of a row 16-byte pieces side by side, and all of them the row's weight.  Matrix instruction e takes channel e of
// every piece: its B operand (contraction index: load and row of the wave, column: the lane's place among sixteen) is an 8 x 8 transposition inside the
// lane, half an instruction per value where conversion and multiplication were two.  The weights keep their 24 bits: each is cut into three
// bf16 numbers that add up to it, exactly, and those are three rows of the A operand, which a lane makes from its own weight: lane
// p of kEvery neighbouring ones part p.  (Of other lanes come rows of the result that nobody reads.)
template <int kEvery>
struct WeightPart {
  unsigned second, third;                        // what to take off first, by lane
  __device__ __forceinline__ explicit WeightPart(int lane)
      : second(lane % kEvery >= 1 ? 0xFFFF0000u : 0u), third(lane % kEvery >= 2 ? 0xFFFF0000u : 0u) {}
  __device__ __forceinline__ unsigned of(float p) const {    // in the upper half
    p -= __uint_as_float(__float_as_uint(p) & second);
    return __float_as_uint(p - __uint_as_float(__float_as_uint(p) & third));
  }
};
// The lower (e even) or upper halves of two dwords
__device__ __forceinline__ unsigned halves(unsigned lo, unsigned hi, int e) {
  return __builtin_amdgcn_perm(hi, lo, e % 2 ? 0x07060302u : 0x05040100u);
}
__device__ __forceinline__ unsigned dword(const uint4& x, int k) { return k == 0 ? x.x : k == 1 ? x.y : k == 2 ? x.z : x.w; }
// d[e] += weights times channel e of the pieces, kLoads rows per lane: parts[i] of row i's weight
template <int kLoads>
__device__ __forceinline__ void weigh_rows(const unsigned (&parts)[kLoads], const uint4 (&rows)[kLoads], f32x4 (&d)[8]) {
#pragma unroll
  for (int first = 0; first < kLoads; first += 8) {
    const bool wide = kLoads - first > 4;        // eight rows per lane to an instruction, or four
    unsigned a[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int i = first + 2 * k;
      a[k] = i < kLoads ? halves(parts[i], i + 1 < kLoads ? parts[i + 1 < kLoads ? i + 1 : i] : 0u, 1) : 0u;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      unsigned b[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int i = first + 2 * k;
        b[k] = i < kLoads ? halves(dword(rows[i < kLoads ? i : 0], e / 2), i + 1 < kLoads ? dword(rows[i + 1 < kLoads ? i + 1 : 0], e / 2) : 0u, e) : 0u;
      }
      if (wide)
        d[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, u32x4{a[0], a[1], a[2], a[3]}),
                                                       __builtin_bit_cast(bf16x8, u32x4{b[0], b[1], b[2], b[3]}), d[e], 0, 0, 0);
      else
        d[e] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(i16x4, u32x2{a[0], a[1]}), __builtin_bit_cast(i16x4, u32x2{b[0], b[1]}),
                                                         d[e], 0, 0, 0);
    }
  }
}
// The three parts' rows together.  (Where a value is infinite a part that is 0 makes NaN of it; the first part is 0 only where the weight is.)
__device__ __forceinline__ float of_parts(const f32x4& d) {
  return __builtin_fabsf(d[0]) <= __FLT_MAX__ ? d[0] + (d[1] + d[2]) : d[0];
}

// ---- one workgroup per query head, all keys, no partial results; kLoads rows per thread.  From six rows on the values go through the matrix
// cores, and a wave takes its weights against its own maximum, so that it begins with them when its own rows are there and not
// when everybody's are (each without the other gains nothing).  With fewer rows what the waves' maxima cost at the end is more than that.
// 16 launches, vector instructions against this: 28/4 heads of d 128, 509 keys 85.3 -> 79.0 us, 629 98.8 -> 92.4; 32/32 heads of d 64, 709
// keys 82.6 -> 76.4, 8/2, 1269 100.6 -> 92.5; with five rows 32/32 heads of d 128, 265 keys 69.8 -> 68.0, 28/4, 309 61.5 -> 62.8; one row, 29 keys
// 39.6 -> 45.8.  What bounds it then is the path into the CU: 283 KB of 28/4 heads and 553 keys are 4400 of its clocks.
constexpr float kDownscale = 0x1p-32f;           // far enough for the rows of a wave
template <int D, int kLoads>
__global__ void __launch_bounds__(kHeadThreads)
decode_head_kernel(const DecodeArgs a) {
  constexpr int kPieces = D / 8, kRows = kHeadThreads / kPieces, kHeadWaves = kHeadThreads / 64;
  constexpr bool kMatrix = kLoads > 5;
  constexpr int kSlots = kMatrix && D == 64 ? 2 * kHeadWaves : kHeadWaves;
  __shared__ float s_m[kHeadWaves], s_l[kHeadWaves];
  __shared__ __align__(16) float s_o[kSlots][D];
  have_arguments(a.q, a.k_tail, a.v_tail, a.out, a.k_cache, a.v_cache, a.c, a.n_tail, a.n_kv_heads, a.budget, a.group, a.scale_log2);
  // grid (KV heads, query heads of one): neighbouring workgroups take different KV heads, and a KV head's query heads share
  // the L2 of one or two dies
  const int hk = blockIdx.x, h = hk * a.group + blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int piece = tid % kPieces, sub = tid / kPieces;
  const int n_keys = a.c + a.n_tail;
  uint4 kw[kLoads], vw[kLoads];
  const uint4 qw = *reinterpret_cast<const uint4*>(a.q + (size_t)h * D + 8 * piece);
  const Rows<D, unsigned> k_rows(a.k_cache, a.k_tail, a, hk, piece), v_rows(a.v_cache, a.v_tail, a, hk, piece);
#pragma unroll
  for (int i = 0; i < kLoads; ++i) kw[i] = k_rows.load(min(kRows * i + sub, n_keys - 1));
#pragma unroll
  for (int i = 0; i < kLoads; ++i) vw[i] = v_rows.load(min(kRows * i + sub, n_keys - 1));
  __builtin_amdgcn_sched_barrier(0);             // all loads on their way before the first is waited for
  float s[kLoads], mx = -INFINITY;
#pragma unroll
  for (int i = 0; i < kLoads; ++i) {
    s[i] = row_sum<kPieces>(dot8(kw[i], qw));
    s[i] = kRows * i + sub < n_keys ? s[i] : -INFINITY;
    mx = fmaxf(mx, s[i]);
  }
  mx = over_rows(mx, FloatMax{}, kPieces == 8);
  if (lane == 0) s_m[wave] = mx;
  float ref = mx;                                // that the wave's weights are taken against
  if constexpr (kMatrix) {
    ref = mx == -INFINITY ? 0.f : mx;            // its own maximum, or all of its keys lie past the end
  } else {
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kHeadWaves; ++w) ref = fmaxf(ref, s_m[w]);     // finite: there is at least one key
  }
  float l = 0.f;
  if constexpr (kMatrix) {
    const WeightPart<kPieces> part(lane);
    unsigned parts[kLoads];
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      const float p = __builtin_amdgcn_exp2f((s[i] - ref) * a.scale_log2);   // 0 for a key past the end
      l += p;
      parts[i] = part.of(p);
    }
    f32x4 d[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) d[e] = f32x4{0.f, 0.f, 0.f, 0.f};
    weigh_rows<kLoads>(parts, vw, d);
    // Register r of lane l is row 4 (l / 16) + r of the result, column l % 16.  At d 64 the odd rows of the wave lie in lanes 8 .. 15 of
    // sixteen: their parts are rows 8 .. 10, their columns 8 .. 15.
    const int slot = D == 64 && lane >= 32 ? kHeadWaves + wave : wave;
    const bool leaves = D == 128 ? lane < 16 : lane < 8 || (lane >= 40 && lane < 48);
    float o[8];
    auto have_sums = [&]() __attribute__((always_inline)) {      // are all of them finite?
      bool finite = true;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        o[e] = of_parts(d[e]);
        finite = finite && __builtin_fabsf(o[e]) <= __FLT_MAX__;
      }
      return finite || !leaves;
    };
    // Values near the largest number there is may be too much for sums against the wave's own maximum, where the row's is far above that:
    // then the weights are taken against a reference further up.
    if (!__all(have_sums()) && mx != -INFINITY) {
#pragma unroll
      for (int i = 0; i < kLoads; ++i) parts[i] = __float_as_uint(__uint_as_float(parts[i]) * kDownscale);
      l *= kDownscale;
      if (lane == 0) s_m[wave] = ref - __builtin_log2f(kDownscale) / a.scale_log2;
#pragma unroll
      for (int e = 0; e < 8; ++e) d[e] = f32x4{0.f, 0.f, 0.f, 0.f};
      weigh_rows<kLoads>(parts, vw, d);
      have_sums();
    }
    if (leaves) {
#pragma unroll
      for (int e = 0; e < 8; e += 4) *reinterpret_cast<float4*>(&s_o[slot][8 * piece + e]) = make_float4(o[e], o[e + 1], o[e + 2], o[e + 3]);
    }
  } else {
    float o[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = 0.f;
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      const float p = __builtin_amdgcn_exp2f((s[i] - ref) * a.scale_log2);   // 0 for a key past the end
      l += p;
      float vx[8];
      unpack8(vw[i], vx);
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = __builtin_fmaf(p, vx[e], o[e]);
    }
    sum_rows<kPieces, 8>(o);                     // lanes 16 r ..: channels 2 r, 2 r + 1 of the piece
    if (lane % 16 < kPieces) *reinterpret_cast<float2*>(&s_o[wave][8 * piece + 2 * (lane / 16)]) = make_float2(o[0], o[1]);
  }
  l = over_rows(l, FloatSum{}, kPieces == 8);
  if (lane == 0) s_l[wave] = l;
  __syncthreads();
  if (tid < D) {
    float num = 0.f, den = 0.f;
    if constexpr (kMatrix) {
      float m[kHeadWaves], all = -INFINITY;
#pragma unroll
      for (int w = 0; w < kHeadWaves; ++w) { m[w] = s_m[w]; all = fmaxf(all, m[w]); }    // finite: there is at least one key
#pragma unroll
      for (int w = 0; w < kHeadWaves; ++w) {
        const float f = __builtin_amdgcn_exp2f((m[w] - all) * a.scale_log2);
        num = __builtin_fmaf(D == 64 ? s_o[w][tid] + s_o[kSlots - kHeadWaves + w][tid] : s_o[w][tid], f, num);
        den = __builtin_fmaf(s_l[w], f, den);
      }
    } else {
#pragma unroll
      for (int w = 0; w < kHeadWaves; ++w) { num += s_o[w][tid]; den += s_l[w]; }
    }
    a.out[(size_t)h * D + tid] = round_bf16(num / den);
  }
}

// The waves' results, with what leaves the workgroup: per query head of the KV head the unnormalised output, maximum and sum.
template <int D, int GM>
__device__ __forceinline__ void leave_partials(const DecodeArgs& a, const float (&s_o)[kWaves][GM][D], const float (&s_m)[kWaves][GM],
                                               const float (&s_l)[kWaves][GM], int G, int hk, int split) {
  for (int i = threadIdx.x; i < G * D; i += kThreads) {
    const int g = i / D, ch = i % D;
    float mm = s_m[0][g];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) mm = fmaxf(mm, s_m[w][g]);          // finite: a tile holds at least one key
    float num = 0.f, den = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const float f = __builtin_amdgcn_exp2f((s_m[w][g] - mm) * a.scale_log2);
      num = __builtin_fmaf(s_o[w][g][ch], f, num);
      den = __builtin_fmaf(s_l[w][g], f, den);
    }
    float* part = a.partial + (((size_t)hk * G + g) * a.n_splits + split) * (D + 2);
    part[ch] = num;
    if (ch == 0) { part[D] = mm; part[D + 1] = den; }
  }
}

// ---- grid (n_splits, Hkv).  G = query heads per KV head, at most GM (the compiled bound, which
// sizes the register arrays; queries beyond G read as zero and their results are dropped).  kGroup: G where the kernel is
// built for that number alone, 0 for any: without the questions whether a query head is there, the heads' chains of
// cross-lane additions run among one another.
template <int D, int GM, int kGroup>
__global__ void __launch_bounds__(kThreads)
decode_kernel(const DecodeArgs a) {
  constexpr int kPieces = D / 8;                 // 16-byte pieces per row
  constexpr int kRowsPerLoad = kThreads / kPieces;
  constexpr int kLoads = kTile / kRowsPerLoad;   // rows of a tile a thread holds a piece of
  __shared__ float s_m[kWaves][GM], s_l[kWaves][GM];
  __shared__ __align__(16) float s_o[kWaves][GM][D];
  have_arguments(a.q, a.k_tail, a.v_tail, a.partial, a.k_cache, a.v_cache, a.c, a.n_tail, a.n_kv_heads, a.budget, a.group, a.n_splits,
                 a.scale_log2);
  const int split = blockIdx.x, hk = blockIdx.y;
  const int G = kGroup ? kGroup : a.group;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int piece = tid % kPieces, sub = tid / kPieces;
  const int n_keys = a.c + a.n_tail;
  const int n_tiles = (n_keys + kTile - 1) / kTile;

  const Rows<D, unsigned long long> k_rows(a.k_cache, a.k_tail, a, hk, piece), v_rows(a.v_cache, a.v_tail, a, hk, piece);
  float o[8 * GM], m[GM], l[GM];                 // of this wave's rows; l of this lane's
#pragma unroll
  for (int g = 0; g < GM; ++g) {
    m[g] = -INFINITY;
    l[g] = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[8 * g + e] = 0.f;
  }
  for (int tile = split; tile < n_tiles; tile += a.n_splits) {
    // every K and V piece of the tile, all loads in flight together
    uint4 kw[kLoads], vw[kLoads];
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      kw[i] = k_rows.load(min(tile * kTile + kRowsPerLoad * i + sub, n_keys - 1));
    }
    uint4 qw[GM];
#pragma unroll
    for (int g = 0; g < GM; ++g) {
      qw[g] = make_uint4(0u, 0u, 0u, 0u);
      if (g < G) qw[g] = *reinterpret_cast<const uint4*>(a.q + ((size_t)hk * G + g) * D + 8 * piece);
    }
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      vw[i] = v_rows.load(min(tile * kTile + kRowsPerLoad * i + sub, n_keys - 1));
    }
    // all loads on their way before the first is waited for (with up to four query heads: 32/8 heads of d 128, 2176 keys, 32 layers 308 -> 302 us,
    // where the constant number of heads alone gave 311; 32/32 heads, 2068 keys, 16 layers 187 -> 182; 28/4 heads, 1100 keys 134.1 -> 136.3)
    if constexpr (GM == 4) __builtin_amdgcn_sched_barrier(0);
    float p[GM][kLoads];
#pragma unroll
    for (int g = 0; g < GM; ++g) {
      if (g >= G) continue;
      float mx = m[g];
#pragma unroll
      for (int i = 0; i < kLoads; ++i) {
        p[g][i] = row_sum<kPieces>(dot8(kw[i], qw[g]));
        p[g][i] = tile * kTile + kRowsPerLoad * i + sub < n_keys ? p[g][i] : -INFINITY;
        mx = fmaxf(mx, p[g][i]);
      }
      mx = over_rows(mx, FloatMax{}, kPieces == 8);
      const float m_use = mx == -INFINITY ? 0.f : mx;      // all of this wave's keys so far lie past the end
      const float f = __builtin_amdgcn_exp2f((m[g] - m_use) * a.scale_log2);    // 0 on the first tile
      l[g] *= f;
#pragma unroll
      for (int e = 0; e < 8; ++e) o[8 * g + e] *= f;
#pragma unroll
      for (int i = 0; i < kLoads; ++i) {
        p[g][i] = __builtin_amdgcn_exp2f((p[g][i] - m_use) * a.scale_log2);     // 0 for a key past the end
        l[g] += p[g][i];
      }
      m[g] = mx;
    }
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      float vx[8];
      unpack8(vw[i], vx);
#pragma unroll
      for (int g = 0; g < GM; ++g) {
        if (g >= G) continue;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[8 * g + e] = __builtin_fmaf(p[g][i], vx[e], o[8 * g + e]);
      }
    }
  }
  // ---- rows of a wave, then the waves
#pragma unroll
  for (int g = 0; g < GM; ++g) {
    if (g >= G) continue;
    l[g] = over_rows(l[g], FloatSum{}, kPieces == 8);
    if (lane == 0) { s_m[wave][g] = m[g]; s_l[wave][g] = l[g]; }
  }
  sum_rows<kPieces, 8 * GM>(o);                  // lanes 16 r ..: query heads r GM / 4 .. (r + 1) GM / 4 - 1
  if (lane % 16 < kPieces) {
#pragma unroll
    for (int k = 0; k < GM / 4; ++k)
#pragma unroll
      for (int e = 0; e < 8; e += 4)
        *reinterpret_cast<float4*>(&s_o[wave][(lane / 16) * (GM / 4) + k][8 * piece + e]) =
            make_float4(o[8 * k + e], o[8 * k + e + 1], o[8 * k + e + 2], o[8 * k + e + 3]);
  }
  __syncthreads();
  leave_partials<D, GM>(a, s_o, s_m, s_l, G, hk, split);
}

// ---- The same grid, d 128 and GM / 4 sets of four query heads, with the products of weights and values on the matrix cores: of the sixteen lanes
// of a row four each take one head of a set from its logits on (one exponential per lane and row instead of one per head), the parts of
// that head's weights are four neighbouring rows of a product's result (the fourth is not read), and a group of sixteen lanes has one head's
// output, over all rows of the wave.
template <int GM, int kGroup>
__global__ void __launch_bounds__(kThreads)
decode_group_kernel(const DecodeArgs a) {
  constexpr int D = 128, kPieces = D / 8, kRowsPerLoad = kThreads / kPieces, kLoads = kTile / kRowsPerLoad, kSets = GM / 4;
  __shared__ float s_m[kWaves][GM], s_l[kWaves][GM];
  __shared__ __align__(16) float s_o[kWaves][GM][D];
  have_arguments(a.q, a.k_tail, a.v_tail, a.partial, a.k_cache, a.v_cache, a.c, a.n_tail, a.n_kv_heads, a.budget, a.group, a.n_splits,
                 a.scale_log2);
  const int split = blockIdx.x, hk = blockIdx.y;
  const int G = kGroup ? kGroup : a.group;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int piece = tid % kPieces, sub = tid / kPieces;
  const int n_keys = a.c + a.n_tail;
  const int n_tiles = (n_keys + kTile - 1) / kTile;
  const int head = lane % kPieces / 4;           // of a set, this lane's

  const Rows<D, unsigned long long> k_rows(a.k_cache, a.k_tail, a, hk, piece), v_rows(a.v_cache, a.v_tail, a, hk, piece);
  const WeightPart<4> part(lane);
  f32x4 d[kSets][8];
  float m[kSets], l[kSets];                      // of this wave's rows; l of this lane's
#pragma unroll
  for (int set = 0; set < kSets; ++set) {
    m[set] = -INFINITY;
    l[set] = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) d[set][e] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  for (int tile = split; tile < n_tiles; tile += a.n_splits) {
    // every K and V piece of the tile, all loads in flight together
    uint4 kw[kLoads], vw[kLoads], qw[GM];
#pragma unroll
    for (int i = 0; i < kLoads; ++i) kw[i] = k_rows.load(min(tile * kTile + kRowsPerLoad * i + sub, n_keys - 1));
#pragma unroll
    for (int g = 0; g < GM; ++g) {
      qw[g] = make_uint4(0u, 0u, 0u, 0u);
      if (g < G) qw[g] = *reinterpret_cast<const uint4*>(a.q + ((size_t)hk * G + g) * D + 8 * piece);
    }
#pragma unroll
    for (int i = 0; i < kLoads; ++i) vw[i] = v_rows.load(min(tile * kTile + kRowsPerLoad * i + sub, n_keys - 1));
    if constexpr (GM == 4) __builtin_amdgcn_sched_barrier(0);    // (as in decode_kernel)
    float s[GM][kLoads];
#pragma unroll
    for (int g = 0; g < GM; ++g)
#pragma unroll
      for (int i = 0; i < kLoads; ++i) {
        s[g][i] = 0.f;
        if (g < G) s[g][i] = row_sum<kPieces>(dot8(kw[i], qw[g]));
      }
#pragma unroll
    for (int set = 0; set < kSets; ++set) {
      if (4 * set >= G) continue;
      float x[kLoads], mx = m[set];
#pragma unroll
      for (int i = 0; i < kLoads; ++i) {
        x[i] = s[4 * set][i];
#pragma unroll
        for (int k = 1; k < 4; ++k) x[i] = head == k ? s[4 * set + k][i] : x[i];
        x[i] = tile * kTile + kRowsPerLoad * i + sub < n_keys ? x[i] : -INFINITY;
        mx = fmaxf(mx, x[i]);
      }
      mx = over_rows(mx, FloatMax{}, false);
      const float m_use = mx == -INFINITY ? 0.f : mx;      // all of this wave's keys so far lie past the end
      if (tile != split) {                                 // onto the new reference: the lane's own head, and that of its group's output
        const float f = __builtin_amdgcn_exp2f((m[set] - m_use) * a.scale_log2);
        l[set] *= f;
        const float of_group = __uint_as_float((unsigned)__builtin_amdgcn_ds_bpermute(16 * (lane / 16), (int)__float_as_uint(f)));
#pragma unroll
        for (int e = 0; e < 8; ++e) d[set][e] *= of_group;
      }
      unsigned parts[kLoads];
#pragma unroll
      for (int i = 0; i < kLoads; ++i) {
        const float p = __builtin_amdgcn_exp2f((x[i] - m_use) * a.scale_log2);     // 0 for a key past the end
        l[set] += p;
        parts[i] = part.of(p);
      }
      m[set] = mx;
      weigh_rows<kLoads>(parts, vw, d[set]);
    }
  }
#pragma unroll
  for (int set = 0; set < kSets; ++set) {
    l[set] = over_rows(l[set], FloatSum{}, false);
    if (lane < kPieces && lane % 4 == 0) { s_m[wave][4 * set + head] = m[set]; s_l[wave][4 * set + head] = l[set]; }
#pragma unroll
    for (int e = 0; e < 8; e += 4)
      *reinterpret_cast<float4*>(&s_o[wave][4 * set + lane / 16][8 * piece + e]) =
          make_float4(of_parts(d[set][e]), of_parts(d[set][e + 1]), of_parts(d[set][e + 2]), of_parts(d[set][e + 3]));
  }
  __syncthreads();
  leave_partials<D, GM>(a, s_o, s_m, s_l, G, hk, split);
}

// ---- grid (Hq); kFoldLanes threads per channel, each folding every kFoldLanes-th partial.  The outputs, maxima and
// sums of a batch of them are in flight together: one trip to memory up to 48 partials.
constexpr int kFoldLanes = 4, kFoldBatch = 12;
template <int D>
__global__ void __launch_bounds__(kFoldLanes * D)
decode_fold_kernel(const DecodeArgs a) {
  __shared__ float s_o[kFoldLanes][D], s_m[kFoldLanes], s_l[kFoldLanes];
  have_arguments(a.out, a.partial, a.n_splits, a.scale_log2);
  const int h = blockIdx.x, tid = threadIdx.x;
  const int ch = tid % D, grp = tid / D;
  const float* const part = a.partial + (size_t)h * a.n_splits * (D + 2);
  float m = -INFINITY, o = 0.f, l = 0.f;
  for (int first = grp; first < a.n_splits; first += kFoldLanes * kFoldBatch) {
    float po[kFoldBatch], pm[kFoldBatch], pl[kFoldBatch];
#pragma unroll
    for (int u = 0; u < kFoldBatch; ++u) {
      const int s = first + kFoldLanes * u;
      // (past the end: the last one again, with weight 0; a load under a condition would be waited for on the spot)
      const float* const from = part + (size_t)min(s, a.n_splits - 1) * (D + 2);
      po[u] = from[ch]; pm[u] = from[D]; pl[u] = from[D + 1];
    }
#pragma unroll
    for (int u = 0; u < kFoldBatch; ++u)
      if (first + kFoldLanes * u >= a.n_splits) pm[u] = -INFINITY;
    float mx = m;
#pragma unroll
    for (int u = 0; u < kFoldBatch; ++u) mx = fmaxf(mx, pm[u]);
    const float f0 = __builtin_amdgcn_exp2f((m - mx) * a.scale_log2);    // 0 on the first batch
    o *= f0;
    l *= f0;
#pragma unroll
    for (int u = 0; u < kFoldBatch; ++u) {
      const float f = __builtin_amdgcn_exp2f((pm[u] - mx) * a.scale_log2);
      o = __builtin_fmaf(po[u], f, o);
      l = __builtin_fmaf(pl[u], f, l);
    }
    m = mx;
  }
  s_o[grp][ch] = o;
  if (ch == 0) { s_m[grp] = m; s_l[grp] = l; }
  __syncthreads();
  if (grp == 0) {
    float mm = s_m[0];
#pragma unroll
    for (int k = 1; k < kFoldLanes; ++k) mm = fmaxf(mm, s_m[k]);
    float num = 0.f, den = 0.f;
#pragma unroll
    for (int k = 0; k < kFoldLanes; ++k) {
      const float f = __builtin_amdgcn_exp2f((s_m[k] - mm) * a.scale_log2);    // 0 for a group without partials
      num = __builtin_fmaf(s_o[k][ch], f, num);
      den = __builtin_fmaf(s_l[k], f, den);
    }
    a.out[(size_t)h * D + ch] = round_bf16(num / den);
  }
}

// few keys: one launch, as many rows per thread as the keys need
constexpr int kHeadLoads = 10;
template <int D> constexpr int kHeadRows = kHeadThreads / (D / 8);
template <int D, int kLoads = 1>
hipError_t launch_head(const DecodeArgs& a, hipStream_t s) {
  if constexpr (kLoads < kHeadLoads)
    if (a.c + a.n_tail > kLoads * kHeadRows<D>) return launch_head<D, kLoads + 1>(a, s);
  hipLaunchKernelGGL((decode_head_kernel<D, kLoads>), dim3(a.n_kv_heads, a.group), dim3(kHeadThreads), 0, s, a);
  return hipGetLastError();
}

template <int D, int GM, int kGroup>
void launch_split(const DecodeArgs& a, hipStream_t s) {
  // At d 128 with three query heads or more the values go through the matrix cores.  16 layers, vector instructions against that:
  // 24/8 heads, 2009 keys 119.8 -> 117.7 us; 32/8, 2185 144.0 -> 130.7; 40/8, 2009 139.1 -> 128.7; 12/2, 3009 128.0 -> 117.5; 28/4, 5009
  // 199.0 -> 171.7; 32/4, 2009 144.0 -> 129.9; 32/2, 3009 301.6 -> 272.9; two heads, 16/8, 3009 126.3 -> 126.2; one, 32/32, 2009 176 -> 190 (twice the
  // registers).  At d 64 a product would serve half as many heads: 28/4, 3009 keys 116.5 -> 122.8, 32/2 170 -> 300.
  if constexpr (D == 128 && kGroup != 1 && kGroup != 2)
    hipLaunchKernelGGL((decode_group_kernel<GM, kGroup>), dim3(a.n_splits, a.n_kv_heads), dim3(kThreads), 0, s, a);
  else
    hipLaunchKernelGGL((decode_kernel<D, GM, kGroup>), dim3(a.n_splits, a.n_kv_heads), dim3(kThreads), 0, s, a);
}

template <int D>
hipError_t launch_for(const DecodeArgs& a, hipStream_t s) {
  // (a row's offset in 32 bits: lists of few keys, KV heads of less than 4 GiB together)
  if ((long long)a.c + a.n_tail <= kHeadLoads * kHeadRows<D> && a.n_kv_heads <= 8192) return launch_head<D>(a, s);
  // Built for the number of query heads up to eight (whole passes of 16 to 32 layers, any number against this one: 28/4 heads of d 128,
  // 1100 keys 147.6 -> 134.4 us, 5000 keys 423 -> 414; 24/4 heads, 2099 keys 228 -> 209; 10/2, 3000 keys 288 -> 264; 32/4, 803 keys 149 -> 139;
  // 12/2 of d 64, 3000 keys 273 -> 262; 16/4 of d 64, 4099 keys 199.4 -> 193.7; 32/8 and 32/32 with the fence behind the loads).
  switch (a.group) {
    case 1: launch_split<D, 4, 1>(a, s); break;
    case 2: launch_split<D, 4, 2>(a, s); break;
    case 3: launch_split<D, 4, 3>(a, s); break;
    case 4: launch_split<D, 4, 4>(a, s); break;
    case 5: launch_split<D, 8, 5>(a, s); break;
    case 6: launch_split<D, 8, 6>(a, s); break;
    case 7: launch_split<D, 8, 7>(a, s); break;
    case 8: launch_split<D, 8, 8>(a, s); break;
    default: launch_split<D, 16, 0>(a, s);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(decode_fold_kernel<D>, dim3(a.n_q_heads), dim3(kFoldLanes * D), 0, s, a);
  return hipGetLastError();
}

// ---- kvp_decode_step_static: the partial results live in a file-scope device array instead of
// the cache's scratch set.  Every GPU the library runs on holds its own copy of the array, at its
// own address, until the process ends; host code never uses the array's name as an address, only
// the pointer hipGetSymbolAddress gave for the device in question.
constexpr size_t kStaticScratchFloats = sizeof(scratch) / sizeof(float);
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
float* g_scratch_ptr[kMaxDevices] = {};

}  // namespace

// Looks the array's address up for the CURRENT device (once per device) and returns it.
hipError_t decode_static_scratch(float** ptr, size_t* n_floats) {
  *ptr = nullptr;
  *n_floats = kStaticScratchFloats;
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    float* p = nullptr;
    e = hipGetSymbolAddress(reinterpret_cast<void**>(&p), HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = p;
  }
  *ptr = g_scratch_ptr[dev];
  return hipSuccess;
}

hipError_t launch_decode(const DecodeArgs& a, int head_dim, hipStream_t s) {
  if (a.n_q_heads / a.n_kv_heads > kGroupLimit || a.n_splits < 1 || a.c + a.n_tail < 1) return hipErrorInvalidValue;
  return head_dim == 128 ? launch_for<128>(a, s) : launch_for<64>(a, s);
}

}  // namespace kvp
