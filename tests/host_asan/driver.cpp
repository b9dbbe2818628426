// Drives the C ABI of the host-only sanitized build through the dry-run cases of the Python host
// tests: configuration and segment validation, sizes, the per-layer state machine over all five
// workloads and all three ways of scoring, kvp_prefill_block in groups, the decode entry points
// and their limits; and, with the launches recorded, kvp_prefill_block over layers that depend on each other, and
// the divisions by multiplication of launches of few and of many heads, and where blocks are scored by the keys alone.  Exits 0 when every check holds; the sanitizers abort on any invalid access.
#include <cstdio>
#include <cstdlib>
#include <string>
#include <vector>

#include "kvp.h"
#include "stubs.h"

#define CHECK(cond)                                                            \
  do {                                                                         \
    if (!(cond)) {                                                             \
      std::fprintf(stderr, "%s:%d: check failed: %s\n", __FILE__, __LINE__, #cond); \
      std::exit(1);                                                            \
    }                                                                          \
  } while (0)

struct Shape {
  const char* name;
  int layers, hq, hkv, d, chunk, budget, gh, gw, planes, temporal, n_text;
};
static const Shape kShapes[] = {
    {"tiny", 1, 4, 4, 64, 64, 128, 24, 24, 1, 0, 32},
    {"single_image", 4, 32, 32, 128, 128, 256, 24, 24, 1, 0, 64},
    {"tiled_image", 8, 28, 4, 128, 256, 512, 24, 24, 5, 0, 128},
    {"video", 16, 28, 4, 128, 512, 1024, 14, 14, 32, 1, 128},
    {"long_video", 32, 32, 8, 128, 1024, 2048, 16, 16, 64, 1, 256},
    {"limit", 2, 16, 1, 64, 2048, 6144, 16, 16, 47, 1, 256},        // 8192 candidates, 16 heads per KV head
};

static kvp_config config_of(const Shape& s, int sets) {
  kvp_config c{};
  c.n_layers = s.layers; c.n_q_heads = s.hq; c.n_kv_heads = s.hkv; c.head_dim = s.d;
  c.budget = s.budget; c.chunk_max = s.chunk; c.merge = 1; c.scratch_sets = sets;
  c.flags = KVP_FLAG_DRY_RUN; c.softmax_scale = 0.f;
  return c;
}

static std::vector<kvp_segment> segments_of(const Shape& s) {
  const int nvis = s.gh * s.gw * s.planes;
  return {kvp_segment{0, nvis, KVP_VISUAL, s.gh, s.gw, s.planes, s.temporal},
          kvp_segment{nvis, s.n_text, KVP_TEXT, 0, 0, 0, 0}};
}

// kvp_prefill_block on a cache that is no dry run, every launch recorded: layers whose tensors are independent share
// launches, layers that depend on each other go in their order.  The addresses are never looked at.
static void check_dependent_layers() {
  const Shape s{"block", 8, 8, 2, 64, 32, 64, 4, 4, 40, 1, 32};
  const std::vector<kvp_segment> segs = segments_of(s);
  kvp_config cfg = config_of(s, s.layers);
  cfg.flags = 0;
  const size_t q_bytes = (size_t)s.chunk * s.hq * s.d * 2, kv_bytes = (size_t)s.chunk * s.hkv * s.d * 2;
  auto at = [](size_t bytes) { return reinterpret_cast<void*>((size_t)0x100000000 + bytes); };
  auto launches = [&](int scoring, auto&& change) {
    std::vector<Launch> seen;
    recorded = &seen;
    kvp_cache* c = nullptr;
    CHECK(kvp_init_cache(&cfg, segs.data(), 2, at(0), (size_t)1 << 40, nullptr, &c) == KVP_OK && c);
    for (int l = 0; l < s.layers; ++l) CHECK(kvp_set_state(c, l, s.budget, s.budget) == KVP_OK);       // the block evicts
    std::vector<const void*> q(s.layers), k(s.layers), v(s.layers), obs(s.layers);
    std::vector<void*> out(s.layers);
    for (int l = 0; l < s.layers; ++l) {               // neighbours in memory, without a byte in common
      const size_t base = (size_t)(l + 1) << 30;
      q[l] = at(base); k[l] = at(base + q_bytes); v[l] = at(base + q_bytes + kv_bytes);
      out[l] = at(base + q_bytes + 2 * kv_bytes); obs[l] = at(base + 2 * q_bytes + 2 * kv_bytes);
    }
    change(q, k, v, out, obs);
    CHECK(kvp_prefill_block(c, s.budget, s.chunk, q.data(), k.data(), v.data(), out.data(), scoring, obs.data(), s.chunk,
                            nullptr, nullptr) == KVP_OK);
    for (int l = 0; l < s.layers; ++l) {
      kvp_view vw{};
      CHECK(kvp_decode_ready(c, l, &vw) == KVP_OK && vw.next_token == s.budget + s.chunk);
    }
    kvp_free_cache(c);
    recorded = nullptr;
    std::string all;
    for (const Launch& x : seen) all += std::string(x.kernel) + std::to_string(x.layers) + " ";
    return all;
  };
  auto times = [](int n, const std::string& what) {
    std::string all;
    for (int i = 0; i < n; ++i) all += what;
    return all;
  };
#define EXPECT(got, want)                                                                                       \
  do {                                                                                                          \
    const std::string g = (got), w = (want);                                                                    \
    if (g != w) {                                                                                               \
      std::fprintf(stderr, "%s:%d: launches\n  %s\nexpected\n  %s\n", __FILE__, __LINE__, g.c_str(), w.c_str()); \
      std::exit(1);                                                                                             \
    }                                                                                                           \
  } while (0)
  const int own = KVP_SCORE_OWN;
  EXPECT(launches(own, [](auto&, auto&, auto&, auto&, auto&) {}), "attention8 select8 ");
  // one out for all layers; two in turn
  EXPECT(launches(own, [](auto&, auto&, auto&, auto& out, auto&) { for (void*& o : out) o = out[0]; }), times(8, "attention1 ") + "select8 ");
  EXPECT(launches(own, [](auto&, auto&, auto&, auto& out, auto&) { for (int l = 2; l < 8; ++l) out[l] = out[l % 2]; }),
         times(4, "attention2 ") + "select8 ");
  // a layer's out is the next one's q, or the last byte of its k
  EXPECT(launches(own, [](auto& q, auto&, auto&, auto& out, auto&) { for (int l = 1; l < 8; ++l) q[l] = out[l - 1]; }),
         times(8, "attention1 ") + "select8 ");
  EXPECT(launches(own, [&](auto&, auto& k, auto&, auto& out, auto&) { k[3] = static_cast<char*>(out[2]) - kv_bytes + 1; }),
         "attention3 attention5 select8 ");
  // a layer's out overwrites what an earlier layer's attention has read
  EXPECT(launches(own, [](auto& q, auto&, auto&, auto& out, auto&) { out[5] = const_cast<void*>(q[1]); }), "attention5 attention3 select8 ");
  // ... or what its compaction has yet to read
  EXPECT(launches(own, [](auto&, auto& k, auto&, auto& out, auto&) { out[5] = const_cast<void*>(k[1]); }),
         "attention5 select5 attention3 select3 ");
  EXPECT(launches(own, [&](auto&, auto&, auto& v, auto& out, auto&) {
           for (int l = 1; l < 8; ++l) out[l] = static_cast<char*>(const_cast<void*>(v[l - 1])) + kv_bytes - 1;
         }), times(8, "attention1 select1 "));
  // ... or its scoring pass
  EXPECT(launches(KVP_SCORE_PROXY, [](auto&, auto&, auto&, auto&, auto&) {}), "attention8 rowstat8 colsum8 select8 ");
  EXPECT(launches(KVP_SCORE_PROXY, [](auto&, auto&, auto&, auto& out, auto& obs) { out[4] = const_cast<void*>(obs[1]); }),
         times(2, "attention4 rowstat4 colsum4 select4 "));
  EXPECT(launches(own, [](auto&, auto&, auto&, auto& out, auto& obs) { out[4] = const_cast<void*>(obs[1]); }), "attention8 select8 ");
  // an error in a later group: the layers before it have gone through
  {
    std::vector<Launch> seen;
    recorded = &seen;
    kvp_cache* c = nullptr;
    CHECK(kvp_init_cache(&cfg, segs.data(), 2, at(0), (size_t)1 << 40, nullptr, &c) == KVP_OK && c);
    for (int l = 0; l < s.layers; ++l) CHECK(kvp_set_state(c, l, 0, 0) == KVP_OK);
    std::vector<const void*> in(s.layers, at(0));
    std::vector<void*> out(s.layers);
    for (int l = 0; l < s.layers; ++l) out[l] = at((size_t)(l + 1) << 30);
    out[3] = at(0);
    in[6] = nullptr;
    CHECK(kvp_prefill_block(c, 0, s.chunk, in.data(), in.data(), in.data(), out.data(), own, nullptr, 0, nullptr, nullptr) == KVP_EINVAL);
    for (int l = 0; l < s.layers; ++l) {
      kvp_view vw{};
      CHECK(kvp_decode_ready(c, l, &vw) == KVP_OK && vw.next_token == (l < 6 ? s.chunk : 0));
    }
    for (int n_tokens : {0, -5, s.chunk + 1})
      CHECK(kvp_prefill_block(c, s.chunk, n_tokens, in.data(), in.data(), in.data(), out.data(), own, nullptr, 0, nullptr, nullptr) == KVP_EINVAL);
    kvp_free_cache(c);
    recorded = nullptr;
  }
}

// Blocks of few and of very many heads, every way of scoring and both ways of summing, every launch recorded: the stub
// launchers check the divisions by multiplication that the kernels would make of their work items.
static void check_divisions() {
  struct Heads { int hq, hkv; };
  for (const Heads& heads : {Heads{46410, 1}, Heads{65900, 2}, Heads{100000, 1}, Heads{3000, 3000}, Heads{190, 1}, Heads{182, 2},
                             Heads{64, 64}, Heads{28, 4}, Heads{32, 8}, Heads{4, 4}, Heads{1, 1}})
    for (int chunk : {1, 33, 128, 300, 1024}) {
      if ((long long)heads.hq * chunk > 20000000) continue;
      Shape s{"heads", 2, heads.hq, heads.hkv, 64, chunk, 320, 4, 4, 400, 1, 32};
      const std::vector<kvp_segment> segs = segments_of(s);
      kvp_config cfg = config_of(s, 2);
      cfg.flags = 0;
      std::vector<Launch> seen;
      recorded = &seen;
      void* const at = reinterpret_cast<void*>((size_t)1 << 32);
      kvp_cache* c = nullptr;
      CHECK(kvp_init_cache(&cfg, segs.data(), 2, at, (size_t)1 << 50, nullptr, &c) == KVP_OK && c);
      for (int fused : {1, 0})
        for (int mode = 0; mode < 3; ++mode) {
          CHECK(kvp_set_score_sweep(c, fused) == KVP_OK);
          for (int l = 0; l < 2; ++l) {
            CHECK(kvp_set_state(c, l, s.budget, s.budget) == KVP_OK);
            const int rc = mode == 0 ? kvp_prefill_chunk(c, l, s.budget, chunk, at, at, at, at, nullptr)
                         : mode == 1 ? kvp_prefill_chunk_proxy(c, l, s.budget, chunk, at, at, at, at, at, (chunk + 1) / 2, nullptr)
                                     : kvp_prefill_chunk_keydiff(c, l, s.budget, chunk, at, at, at, at, nullptr);
            CHECK(rc == KVP_OK);
          }
          CHECK(kvp_compact_layers(c, 0, 2, nullptr) == KVP_OK);
        }
      kvp_free_cache(c);
      recorded = nullptr;
    }
}

// Scored by the keys alone: beside the attention, in the compaction or by kernels of its own, once and only once.
static void check_key_scoring() {
  auto launches = [&](int layers, int hq, int hkv, int d, int n, int budget, int shape) {
    Shape s{"keys", layers, hq, hkv, d, n, budget, 4, 4, 400, 1, 32};
    const std::vector<kvp_segment> segs = segments_of(s);
    kvp_config cfg = config_of(s, layers);
    cfg.flags = 0;
    std::vector<Launch> seen;
    recorded = &seen;
    kvp_cache* c = nullptr;
    void* const at = reinterpret_cast<void*>((size_t)1 << 32);
    CHECK(kvp_init_cache(&cfg, segs.data(), 2, at, (size_t)1 << 50, nullptr, &c) == KVP_OK && c);
    CHECK(kvp_set_attention_shape(c, shape) == KVP_OK);
    std::vector<const void*> in(layers, at);
    std::vector<void*> out(layers);
    for (int l = 0; l < layers; ++l) {
      CHECK(kvp_set_state(c, l, budget, budget) == KVP_OK);
      out[l] = reinterpret_cast<void*>((size_t)(l + 2) << 32);
    }
    CHECK(kvp_prefill_block(c, budget, n, in.data(), in.data(), in.data(), out.data(), KVP_SCORE_KEYDIFF, nullptr, 0, nullptr, nullptr) == KVP_OK);
    kvp_free_cache(c);
    recorded = nullptr;
    std::string all;
    for (const Launch& x : seen) all += std::string(x.kernel) + std::to_string(x.layers) + " ";
    return all;
  };
  // 32-row workgroups, one round of 256 with the scoring ones: 224 + 8, 248 + 8, 256 + 8, 240 + 16, 256 + 32
  EXPECT(launches(1, 28, 4, 128, 256, 512, -1), "attention+keys1 select1 ");
  EXPECT(launches(1, 31, 1, 128, 256, 512, -1), "attention+keys1 select1 ");
  EXPECT(launches(1, 32, 8, 128, 256, 512, -1), "attention1 keys+select1 ");
  EXPECT(launches(1, 60, 10, 128, 128, 512, -1), "attention+keys1 select1 ");
  EXPECT(launches(1, 32, 32, 128, 256, 512, -1), "attention1 keys+select1 ");
  EXPECT(launches(8, 28, 4, 128, 256, 512, -1), "attention+keys8 select8 ");
  // 64-row workgroups, one round or more
  EXPECT(launches(1, 28, 4, 128, 512, 512, -1), "attention+keys1 select1 ");
  EXPECT(launches(1, 40, 8, 128, 512, 512, -1), "attention+keys1 select1 ");
  EXPECT(launches(8, 40, 8, 128, 512, 512, -1), "attention+keys8 select8 ");
  // d 64: 768 workgroups in all layers of the launch (4 x 184, 5 x 184; 2 x 328, 3 x 328)
  EXPECT(launches(4, 16, 4, 64, 333, 1111, -1), "attention+keys4 select4 ");
  EXPECT(launches(5, 16, 4, 64, 333, 1111, -1), "attention5 keys+select5 ");
  EXPECT(launches(2, 40, 8, 64, 512, 1024, -1), "attention+keys2 select2 ");
  EXPECT(launches(3, 40, 8, 64, 512, 1024, -1), "attention3 keys+select3 ");
  // 128-row workgroups, and one more key than a workgroup holds
  EXPECT(launches(2, 32, 8, 128, 1000, 24, -1), "attention2 keys+select2 ");
  EXPECT(launches(2, 28, 4, 128, 256, 512, 2), "attention2 keys+select2 ");
  EXPECT(launches(2, 28, 4, 128, 256, 768, 2), "attention2 keys+select2 ");
  EXPECT(launches(2, 4, 4, 64, 256, 1792, 2), "attention2 keys+select2 ");
  EXPECT(launches(2, 28, 4, 128, 256, 769, -1), "attention2 keydiff2 select2 ");
  EXPECT(launches(2, 4, 4, 64, 256, 1793, -1), "attention2 keydiff2 select2 ");
}

int main() {
  check_key_scoring();
  check_dependent_layers();
  check_divisions();
  CHECK(kvp_strerror(KVP_OK) && kvp_strerror(-77));
  for (const Shape& s : kShapes) {
    const std::vector<kvp_segment> segs = segments_of(s);
    const int n_tokens = segs[0].n_tokens + segs[1].n_tokens;
    for (int sets : {1, 2, s.layers}) {
      if (sets > s.layers) continue;
      kvp_config cfg = config_of(s, sets);
      CHECK(kvp_cache_bytes(&cfg) > kvp_persistent_bytes(&cfg));
      CHECK(kvp_persistent_bytes(&cfg) >= (size_t)2 * s.layers * s.hkv * s.d * 2 * s.budget);
      kvp_cache* c = nullptr;
      CHECK(kvp_init_cache(&cfg, segs.data(), 2, nullptr, 0, nullptr, &c) == KVP_OK && c);
      // per-layer calls, every way of scoring in turn
      int count = 0, block = 0;
      for (int t0 = 0; t0 < n_tokens; t0 += s.chunk, ++block) {
        const int n = t0 + s.chunk <= n_tokens ? s.chunk : n_tokens - t0;
        for (int l = 0; l < s.layers; ++l) {
          int rc;
          if (block % 3 == 0) rc = kvp_prefill_chunk(c, l, t0, n, nullptr, nullptr, nullptr, nullptr, nullptr);
          else if (block % 3 == 1) rc = kvp_prefill_chunk_keydiff(c, l, t0, n, nullptr, nullptr, nullptr, nullptr, nullptr);
          else rc = kvp_prefill_chunk_proxy(c, l, t0, n, nullptr, nullptr, nullptr, nullptr, nullptr, 1 + block % s.chunk, nullptr);
          CHECK(rc == KVP_OK);
          CHECK(kvp_prefill_chunk(c, l, t0 + n, 1, nullptr, nullptr, nullptr, nullptr, nullptr) == KVP_ESTATE);
          kvp_view vw{};
          CHECK(kvp_decode_ready(c, l, &vw) == KVP_ESTATE);
          CHECK(kvp_compact(c, l, nullptr, nullptr) == KVP_OK);
          CHECK(kvp_compact(c, l, nullptr, nullptr) == KVP_ESTATE);
          CHECK(kvp_decode_ready(c, l, &vw) == KVP_OK);
          const int want = count + n < s.budget ? count + n : s.budget;
          CHECK(vw.count == want && vw.next_token == t0 + n && vw.budget == s.budget);
          if (s.hq / s.hkv <= 16) {
            CHECK(kvp_decode_step(c, l, nullptr, nullptr, nullptr, 1 + block, nullptr, nullptr) == KVP_OK);
            const int rcs = kvp_decode_step_static(c, l, nullptr, nullptr, nullptr, 1 + block, nullptr, nullptr);
            CHECK(rcs == KVP_OK || rcs == KVP_ENOMEM);
          }
        }
        count = count + n < s.budget ? count + n : s.budget;
      }
      CHECK(kvp_prefill_chunk(c, 0, n_tokens, 1, nullptr, nullptr, nullptr, nullptr, nullptr) == KVP_EINVAL);
      // the whole prefix again through kvp_prefill_block (groups of layers), after a restore
      for (int l = 0; l < s.layers; ++l) CHECK(kvp_set_state(c, l, 0, 0) == KVP_OK);
      std::vector<const void*> in(s.layers, nullptr);
      std::vector<void*> out(s.layers, nullptr);
      int blk = 0;
      for (int t0 = 0; t0 < n_tokens; t0 += s.chunk, ++blk) {
        const int n = t0 + s.chunk <= n_tokens ? s.chunk : n_tokens - t0;
        // the three ways of scoring in turn: the proxy and key-only passes go out for a group of layers
        const int scoring = blk % 3 == 0 ? KVP_SCORE_OWN : blk % 3 == 1 ? KVP_SCORE_PROXY : KVP_SCORE_KEYDIFF;
        CHECK(kvp_prefill_block(c, t0, n, in.data(), in.data(), in.data(), out.data(), scoring,
                                scoring == KVP_SCORE_PROXY ? in.data() : nullptr, 1 + blk % s.chunk,
                                nullptr, nullptr) == KVP_OK);
      }
      CHECK(kvp_prefill_join(c, nullptr, nullptr) == KVP_OK);
      // and once more layer by layer with one kvp_compact_layers per block, as far as the scratch
      // sets allow layers to be pending together
      for (int l = 0; l < s.layers; ++l) CHECK(kvp_set_state(c, l, 0, 0) == KVP_OK);
      CHECK(kvp_compact_layers(c, 0, s.layers + 1, nullptr) == KVP_EINVAL);
      CHECK(kvp_compact_layers(c, 0, 1, nullptr) == KVP_ESTATE);
      for (int t0 = 0; t0 < n_tokens; t0 += s.chunk) {
        const int n = t0 + s.chunk <= n_tokens ? s.chunk : n_tokens - t0;
        const int together = sets < s.layers ? sets : s.layers;
        for (int first = 0; first < s.layers; first += together) {
          const int count = first + together <= s.layers ? together : s.layers - first;
          for (int l = first; l < first + count; ++l)
            CHECK(kvp_prefill_chunk(c, l, t0, n, nullptr, nullptr, nullptr, nullptr, nullptr) == KVP_OK);
          CHECK(kvp_compact_layers(c, first, count, nullptr) == KVP_OK);
        }
      }
      for (int l = 0; l < s.layers; ++l) {
        kvp_view vw{};
        CHECK(kvp_decode_ready(c, l, &vw) == KVP_OK && vw.next_token == n_tokens);
      }
      CHECK(kvp_set_attention_shape(c, 3) == KVP_EINVAL && kvp_set_attention_shape(c, 1) == KVP_OK);
      CHECK(kvp_set_score_sweep(c, 2) == KVP_EINVAL && kvp_set_score_sweep(c, 0) == KVP_OK);
      const uint64_t* totals = reinterpret_cast<const uint64_t*>(1);
      CHECK(kvp_debug_totals(c, &totals) == KVP_OK && totals == nullptr);
      kvp_kernel_stat stats[KVP_K_COUNT];
      CHECK(kvp_profile_enable(c, 1) == KVP_OK && kvp_profile_read(c, stats) == KVP_OK);
      kvp_free_cache(c);
    }
  }
  // refused configurations and layouts
  {
    kvp_config bad = config_of(kShapes[0], 1);
    bad.head_dim = 96;
    CHECK(kvp_cache_bytes(&bad) == 0);
    kvp_config big = config_of(kShapes[0], 1);
    big.budget = 8190;
    CHECK(kvp_cache_bytes(&big) == 0);
    kvp_config ok = config_of(kShapes[0], 1);
    kvp_cache* c = nullptr;
    kvp_segment gap[2] = {{0, 10, KVP_VISUAL, 2, 5, 1, 0}, {11, 5, KVP_TEXT, 0, 0, 0, 0}};
    CHECK(kvp_init_cache(&ok, gap, 2, nullptr, 0, nullptr, &c) == KVP_EINVAL && !c);
    CHECK(kvp_init_cache(&ok, gap, 0, nullptr, 0, nullptr, &c) == KVP_EINVAL);
    CHECK(kvp_init_cache(&ok, nullptr, 1, nullptr, 0, nullptr, &c) == KVP_EINVAL);
    CHECK(kvp_compact(nullptr, 0, nullptr, nullptr) == KVP_EINVAL);
    kvp_free_cache(nullptr);
  }
  std::puts("host state machine under the sanitizers: ok");
  return 0;
}
