// Cuts random ranges and batches into sieve segments as a search does, walks
// them as the sieve's workgroups do, and turns word indices back into integers.
// Prints "ok" and the number of integers looked at, or the first that is wrong.
#include <cstdio>
#include <cstdlib>
#include <random>

#include "bx_segments.h"

using bx::Query;

static uint64_t check(std::vector<Query> q, uint64_t wgs, uint32_t longest, bool one_range, std::mt19937_64& rng) {
  uint64_t n = 0;
  for (Query& e : q) {
    e.top = e.b;
    n += e.b - e.a;
  }
  const std::vector<Query> whole = q;
  const uint32_t seg_len = bx::cut_search(&q, n, wgs, longest, one_range);
  std::vector<uint64_t> prefix(1, 0);
  for (const Query& e : q) prefix.push_back(prefix.back() + (e.b - e.a + e.seg_len - 1) / e.seg_len);
  const uint64_t n_segs = prefix.back();
  const uint32_t W = static_cast<uint32_t>(std::min<uint64_t>(n_segs, wgs));
  auto bad = [&](const char* what, uint64_t x) {
    std::printf("%s: x=%llu of [%llu, %llu), %llu workgroups, longest %u, step %u\n", what,
                static_cast<unsigned long long>(x), static_cast<unsigned long long>(whole[0].a),
                static_cast<unsigned long long>(whole[0].b), static_cast<unsigned long long>(wgs), longest, seg_len);
    std::exit(1);
  };
  // The parts make up the range.
  for (size_t i = 0; i + 1 < q.size() && one_range; ++i)
    if (q[i].b != q[i + 1].a) bad("gap", q[i].b);
  if (q[0].a != whole[0].a || q.back().b != whole.back().b) bad("ends", q[0].a);
  for (const Query& e : q)
    if (e.seg_len == 0 || e.seg_len > longest) bad("segment length", e.seg_len);
  const uint32_t li_bits = bx::index_bits(n_segs, W, seg_len);
  const bx::WordSource S{q.data(), prefix.data(), static_cast<uint32_t>(q.size()), seg_len, W, li_bits, !one_range};
  uint64_t seen = 0;
  std::vector<uint32_t> ws = {0, W - 1, static_cast<uint32_t>(rng() % W)};
  for (uint32_t w : ws) {
    uint64_t li0 = 0, rounds = (n_segs - w + W - 1) / W;
    const uint64_t skip = rounds > 64 ? rounds / 64 : 1;  // of long walks, some segments
    for (uint64_t s = w, r = 0; s < n_segs; s += W, li0 += seg_len, ++r) {
      if (r % skip && s + W < n_segs) continue;
      size_t i = 0;
      while (prefix[i + 1] <= s) ++i;
      const uint64_t start = q[i].a + (s - prefix[i]) * q[i].seg_len;
      const uint64_t len = std::min<uint64_t>(q[i].seg_len, q[i].b - start);
      for (uint64_t off : {uint64_t(0), len - 1, len / 2, rng() % len, rng() % len}) {
        const uint64_t li = li0 + off;
        if (li >= (1ull << li_bits) - 1) bad("index bits", start + off);
        uint32_t grp;
        if (bx::word_integer(S, w, li, &grp) != start + off) bad("integer", start + off);
        if (grp != (one_range ? 0u : i)) bad("query", start + off);
        ++seen;
      }
    }
  }
  return seen;
}

int main() {
  std::mt19937_64 rng(20260101);
  auto log_uniform = [&](double lo, double hi) {
    return static_cast<uint64_t>(std::exp2(std::uniform_real_distribution<double>(lo, hi)(rng)));
  };
  uint64_t seen = 0;
  for (int t = 0; t < 20000; ++t) {
    const uint64_t wgs = t % 3 ? 256 : 1 + rng() % 304;
    const uint32_t longest = t % 2 ? 1u << 18 : static_cast<uint32_t>(8192 * (1 + rng() % 64));
    uint64_t a = t % 4 ? 1 : log_uniform(0, 41), n = log_uniform(1, 37);
    if (t % 5 < 3) {  // just past full rounds of all workgroups
      n = wgs * longest * log_uniform(0, 8);
      n += rng() % (32 * static_cast<uint64_t>(std::sqrt(static_cast<double>(n))) + 2);
    }
    const uint64_t b = std::min<uint64_t>(a + n, (1ull << 42) - 1);
    if (b < a + 2) continue;
    seen += check({Query{a, b}}, wgs, longest, true, rng);
  }
  for (int t = 0; t < 500; ++t) {
    std::vector<Query> q;
    for (uint64_t k = 1 + rng() % 60; k; --k) {
      const uint64_t a = log_uniform(0, 40);
      q.push_back(Query{a, a + log_uniform(1, 26)});
    }
    seen += check(q, 256, 1u << 18, false, rng);
  }
  std::printf("ok %llu\n", static_cast<unsigned long long>(seen));
  return 0;
}
