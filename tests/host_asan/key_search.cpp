// The search for the budget-th largest selection key (key_range.h), run as the selection runs it -- count the keys by
// bin, enter the bin with the wanted key, divide it while it holds more than 64 -- against a sort.
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <random>
#include <string>
#include <vector>

#include "key_range.h"

#ifndef KEY_SEARCH_BITS                    // of the histogram: one of the selection's two sizes
#define KEY_SEARCH_BITS kvp::kSelectBinBits
#endif
constexpr int kBits = KEY_SEARCH_BITS, kBins = 1 << kBits;
using KeyRange = kvp::KeyRangeOf<kBits>;
typedef unsigned long long Key;

static unsigned order_bits(float x) {
  if (x == 0.f) x = 0.f;
  unsigned u;
  std::memcpy(&u, &x, 4);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
static Key key_of(float score, unsigned token) { return ((Key)order_bits(score) << 32) | (Key)~token; }

// the number of keys that reach the threshold, and whether it is the budget-th largest key
static bool right(const std::vector<Key>& keys, unsigned budget, const std::string& what) {
  unsigned lo = ~0u, hi = 0;
  for (Key k : keys) {
    lo = std::min(lo, (unsigned)(k >> 32));
    hi = std::max(hi, (unsigned)(k >> 32));
  }
  KeyRange range = KeyRange::over(lo, hi);
  unsigned want = budget, in_bin = 0;
  std::vector<unsigned> hist;
  for (int pass = 0;; ++pass) {
    if (pass > 6) {                        // 64 bits, nine or eleven at a time, less what the first range leaves out
      std::printf("%s: no end after %d passes\n", what.c_str(), pass);
      return false;
    }
    hist.assign(kBins, 0u);
    for (Key k : keys)
      if (unsigned bin; range.holds(k, bin)) ++hist[bin];
    unsigned above = 0;
    int digit = kBins - 1;
    for (; digit >= 0 && above + hist[digit] < want; --digit) above += hist[digit];
    if (digit < 0) {
      std::printf("%s: fewer keys in the range than wanted\n", what.c_str());
      return false;
    }
    want -= above;
    in_bin = hist[digit];
    range.enter((unsigned)digit);
    if (in_bin <= 64u || range.shift == 0) break;
    range.divide();
  }
  if (in_bin > 64u) {                      // equal keys, as only a cache written from outside has them
    std::vector<Key> sorted = keys;
    std::sort(sorted.rbegin(), sorted.rend());
    if (range.lo == sorted[budget - 1]) return true;
    std::printf("%s: another key\n", what.c_str());
    return false;
  }
  std::vector<Key> members;
  for (Key k : keys)
    if (unsigned bin; range.holds(k, bin)) members.push_back(k);
  if (members.size() != in_bin) {
    std::printf("%s: %zu keys in a bin of %u\n", what.c_str(), members.size(), in_bin);
    return false;
  }
  std::sort(members.rbegin(), members.rend());
  const Key threshold = members[want - 1];
  std::vector<Key> sorted = keys;
  std::sort(sorted.rbegin(), sorted.rend());
  if (threshold == sorted[budget - 1]) return true;
  std::printf("%s: keeps %zu of %zu, wanted %u\n", what.c_str(),
              (size_t)std::count_if(keys.begin(), keys.end(), [&](Key k) { return k >= threshold; }), keys.size(), budget);
  return false;
}

int main() {
  std::mt19937 rng(1);
  int bad = 0, cases = 0;
  auto check = [&](const std::vector<Key>& keys, unsigned budget, const std::string& what) {
    ++cases;
    bad += !right(keys, budget, what);
  };
  struct Size { unsigned n, budget, token0; };
  const Size sizes[] = {{3072, 2048, 0}, {2048, 1536, 0}, {768, 512, 700}, {8192, 6144, 0}, {130, 65, 1000}, {2, 1, 0},
                        {1500, 900, 1020}, {4096, 1, 2047}, {4096, 4095, 16777216 - 4096}};
  for (const Size& s : sizes) {
    std::vector<unsigned> token(s.n);
    for (unsigned i = 0; i < s.n; ++i) token[i] = s.token0 + i;
    std::shuffle(token.begin(), token.end(), rng);
    auto keys = [&](auto score) {
      std::vector<Key> k(s.n);
      for (unsigned i = 0; i < s.n; ++i) k[i] = key_of(score(i), token[i]);
      return k;
    };
    const std::string at = std::to_string(s.n) + " keys, budget " + std::to_string(s.budget);
    check(keys([](unsigned) { return 0.75f; }), s.budget, at + ", all equal");
    check(keys([](unsigned) { return 0.f; }), s.budget, at + ", all zero");
    std::uniform_real_distribution<float> uniform(0.f, 4.f);
    for (unsigned some : {s.n / 2, s.n / 3, s.n - 1, 1u})
      check(keys([&](unsigned i) { return i < some ? uniform(rng) : 0.f; }), s.budget, at + ", zeros beside ordinary scores");
    for (int levels : {2, 3, 5, 9, 40, 1000})
      check(keys([&](unsigned) { return (float)(1 + rng() % (unsigned)levels) / 7.f; }), s.budget, at + ", " + std::to_string(levels) + " levels");
    check(keys([&](unsigned) { return -uniform(rng); }), s.budget, at + ", negative");
    check(keys([&](unsigned i) { return i % 3 ? -0.f : 0.f; }), s.budget, at + ", both zeros");
    // token indices that repeat: in pairs, in forties, by the hundred, all the same
    for (unsigned copies : {2u, 40u, 100u, s.n})
      for (int levels : {1, 3}) {
        std::vector<Key> k(s.n);
        for (unsigned i = 0; i < s.n; ++i) k[i] = key_of((float)(1 + rng() % (unsigned)levels), s.token0 + i / copies);
        check(k, s.budget, at + ", tokens " + std::to_string(copies) + " times");
      }
    // scores that span 2^j steps of the float scale: the first shift is 21 + j, every one from 21 to 53 - with the
    // threshold among equal scores at the bottom, in the middle and at the top
    for (int j = 0; j <= 32; ++j)
      for (int where = 0; where < 3; ++where) {
        const unsigned span = j == 32 ? 0xFFFFFFFFu : (1u << j) - 1u;
        const unsigned base = j >= 31 ? 0u : 0x80000000u >> (j == 0 ? 0 : 1);
        std::vector<Key> k(s.n);
        for (unsigned i = 0; i < s.n; ++i) {
          const unsigned of = i == 0 ? 0u : i == 1 ? span : where == 0 ? 0u : where == 1 ? span / 2 : span;
          k[i] = ((Key)(base + of) << 32) | (Key)~token[i];
        }
        check(k, s.budget, at + ", span 2^" + std::to_string(j));
      }
  }
  std::printf("%d of %d cases wrong\n", bad, cases);
  return bad != 0;
}
