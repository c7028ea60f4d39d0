// The host layout planner (relabel, dense prefix, capacities, regions, the
// sampler's units and light batches; the all-host reference behind
// lda_describe_layout) under AddressSanitizer and
// UndefinedBehaviorSanitizer, CPU only: seeded corpora of many shapes, with
// the layout invariants checked.  Exit status 0 = every check held.
#include <algorithm>
#include <cstdio>
#include <numeric>
#include <random>
#include <vector>

#include "lda_internal.h"

#define CHECK(c)                                                      \
  do {                                                                \
    if (!(c)) {                                                       \
      std::fprintf(stderr, "check failed at line %d: %s\n", __LINE__, #c); \
      return 1;                                                       \
    }                                                                 \
  } while (0)

// The sampler's units and light batches of a region table: every token of every
// region belongs to exactly one, or topic slots would be drawn twice or left stale.
static int units_and_batches(std::mt19937 &g, const std::vector<uint32_t> &region, int64_t light_begin, int K) {
  const int64_t n = int64_t(region.size() / 3);
  uint64_t tokens = 0;
  for (size_t r = 0; r < region.size(); r += 3) tokens += region[r + 2] - region[r + 1];
  const int threads = 256 << (g() % 3);
  const int64_t workgroups = 1 + int64_t(g() % 3000);
  const std::vector<uint32_t> u = lda::sampler_units(region, light_begin, int64_t(tokens), K, workgroups, threads);
  size_t at = 0;
  for (int64_t r = 0; r < light_begin; ++r) {
    const uint32_t v = region[3 * size_t(r)], b = region[3 * size_t(r) + 1], e = region[3 * size_t(r) + 2];
    for (uint32_t pos = b; pos < e;) {
      CHECK(at + 3 <= u.size());
      CHECK(u[at] == (pos == b ? v : v | lda::kUnitContinues));  // one unit of a region starts it
      CHECK(u[at + 1] == pos && u[at + 2] > pos && u[at + 2] <= e);
      // no cut below the tokens that give every wave a batch, nor below K (half the least unit, by rounding)
      CHECK(e - b <= uint32_t(std::max(threads, 2 * K)) || u[at + 2] - pos >= uint32_t(std::max(threads, 2 * K)) / 2);
      pos = u[at + 2];
      at += 3;
    }
  }
  CHECK(at == u.size());
  const std::vector<uint32_t> c = lda::light_batches(region, light_begin, 1 + int64_t(g() % 5000));
  CHECK(!c.empty() && c.front() == 0 && c.back() == uint32_t(n - light_begin));
  for (size_t q = 0; q + 1 < c.size(); ++q) {
    CHECK(c[q + 1] > c[q] && c[q + 1] - c[q] <= 64);  // a lane per word
    const size_t first = 3 * size_t(light_begin + c[q]), last = 3 * size_t(light_begin + c[q + 1] - 1);
    CHECK(region[last + 2] - region[first + 1] <= lda::kLightTokens);  // a lane per token
    for (size_t r = first; r < last; r += 3) CHECK(region[r + 2] == region[r + 4]);  // consecutive tokens
  }
  return 0;
}

// Where the regions of at most kLightTokens tokens that end the table begin.
static int64_t light_suffix(const std::vector<uint32_t> &region) {
  int64_t r = int64_t(region.size() / 3);
  while (r > 0 && region[3 * size_t(r - 1) + 2] - region[3 * size_t(r - 1) + 1] <= lda::kLightTokens) --r;
  return r;
}

static int one(std::mt19937 &g, int trial) {
  const int V = 1 + int(g() % 60), K = 2 + int(g() % 300), R = 1 + int(g() % 50);
  const int M = 1 + int(g() % 40), n = 1 + int(g() % 3000);
  const int cutoff = int(g() % 4) == 0 ? -1 : int(g() % 3) == 0 ? int(g() % 20) : 0;
  std::vector<int32_t> word(static_cast<size_t>(n)), doc(static_cast<size_t>(n));
  for (int i = 0; i < n; ++i) {
    word[size_t(i)] = int32_t(g() % uint32_t(V));
    doc[size_t(i)] = int32_t(g() % uint32_t(M));
  }
  if (trial % 2) std::sort(doc.begin(), doc.end());
  lda::Layout L;
  std::string msg;
  CHECK(lda::build_layout(word.data(), doc.data(), n, V, K, R, cutoff, L, msg) == LDA_OK);
  CHECK(L.word_off.size() == size_t(L.n_present) + 1 && L.word_off.back() == uint32_t(n));
  std::vector<int> seen(static_cast<size_t>(n), 0);
  for (uint32_t k : L.wt_key) seen[k]++;
  for (int s : seen) CHECK(s == 1);
  std::vector<int> covered(static_cast<size_t>(n), 0);
  for (size_t r = 0; r < L.region.size(); r += 3) {
    const uint32_t v = L.region[r], b = L.region[r + 1], e = L.region[r + 2];
    CHECK(int32_t(v) < L.n_present && b < e && L.word_off[v] <= b && e <= L.word_off[v + 1]);
    CHECK(e - b <= uint32_t(R) || int32_t(v) >= L.n_dense);
    for (uint32_t q = b; q < e; ++q) covered[q]++;
  }
  for (int c : covered) CHECK(c == 1);
  for (int32_t d = 0; d < L.M; ++d) CHECK(L.d_cap[size_t(d) + 1] > L.d_cap[size_t(d)]);
  // regions of a word-offset table with empty words, as an out-of-core chunk plans them
  std::vector<uint32_t> woff(static_cast<size_t>(V) + 1, 0);
  for (int v = 0; v < V; ++v) woff[size_t(v) + 1] = woff[size_t(v)] + (g() % 3 == 0 ? 0u : uint32_t(g() % 40));
  std::vector<uint8_t> split;
  std::vector<uint32_t> region;
  int64_t ndr = 0;
  lda::make_regions(woff, V, R, split, region, ndr);
  uint64_t tokens = 0;
  for (size_t r = 0; r < region.size(); r += 3) tokens += region[r + 2] - region[r + 1];
  CHECK(tokens == woff.back() && ndr == int64_t(region.size() / 3));
  for (const std::vector<uint32_t> &r : {L.region, region}) {
    if (units_and_batches(g, r, light_suffix(r), K)) return 1;
    if (units_and_batches(g, r, int64_t(r.size() / 3), K)) return 1;  // no light region
  }
  return 0;
}

// Words of given token counts (in order), cut with R: counts at multiples of the least unit and around them, one
// region, light regions only, split words among the light suffix (R = 1, 7).
static int edges(std::mt19937 &g) {
  const std::vector<std::vector<uint32_t>> shapes = {
      {1}, {64}, {65}, {255, 256, 257, 511, 512, 513, 1024, 65536, 1, 64, 64, 1, 1}, {100000, 3, 2, 1},
      std::vector<uint32_t>(300, 1), std::vector<uint32_t>(70, 64), {20, 20, 20, 20, 20, 20}};
  for (const auto &s : shapes)
    for (int R : {1, 7, 63, 64, 65, 10000})
      for (int nd : {0, 1, int(s.size())}) {
        std::vector<uint32_t> woff(1, 0);
        for (uint32_t c : s) woff.push_back(woff.back() + c);
        std::vector<uint8_t> split;
        std::vector<uint32_t> region;
        int64_t ndr = 0;
        lda::make_regions(woff, std::min(nd, int(s.size())), R, split, region, ndr);
        for (int K : {2, 100, 128, 1000})
          if (units_and_batches(g, region, light_suffix(region), K)) return 1;
      }
  return 0;
}

int main() {
  std::mt19937 g(20240);
  if (edges(g)) return 1;
  for (int trial = 0; trial < 300; ++trial)
    if (one(g, trial)) {
      std::fprintf(stderr, "trial %d\n", trial);
      return 1;
    }
  std::printf("layout checks passed\n");
  return 0;
}
