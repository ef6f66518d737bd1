// How ranges are cut into sieve segments, and the index that a first-level
// word holds for an integer.  Used by the host, the kernels and a CPU test.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <vector>

namespace bx {

// A range to sieve: a query, or one of the parts of a single query.
struct Query {
  uint64_t a, b;     // x in [a, b); radicals over [a, b]
  uint64_t top;      // the query's end (the bound of the member test)
  uint32_t seg_len;  // of its segments
  uint32_t pad;
};

inline uint64_t round_up(uint64_t v, uint64_t m) { return (v + m - 1) / m * m; }

// Segment length for n integers over `wgs` workgroups: as many equal rounds of
// all workgroups as segments of at most `longest` need, in multiples of `unit`.
// (Not monotonic in n: where a round is added, the length drops.)
// Segments of 2^18 left the chip idle on short ranges (2^20 integers at 2^40 on
// 4 of 256 CUs: sieve 81 us) and ran a last round for a few of them; a short
// segment repeats the hit list's look at every large power (about 9 us at 2^40),
// so those of a range run side by side.
inline uint32_t fit_seg_len(uint64_t n, uint64_t wgs, uint32_t longest, uint32_t unit) {
  const uint64_t rounds = std::max<uint64_t>(1, (n + wgs * longest - 1) / (wgs * longest));
  const uint64_t len = round_up(std::max<uint64_t>(1, (n + wgs * rounds - 1) / (wgs * rounds)), unit);
  return static_cast<uint32_t>(std::min<uint64_t>(len, longest));
}

constexpr uint32_t kKeySegUnit = 4096;  // four subtiles: a wave per SIMD at work at least
constexpr uint32_t kLowSegUnit = 256;   // where all integers may be kept

// Segment lengths for searches of the queries `q`, of n segmented integers in
// all; returns the longest, by which the sieve counts a workgroup's integers.
//
// The search of one range (one_range) that reaches below 32 sqrt(b) is sieved
// in two parts, that low zone in shorter segments, so that it spreads over the
// chip: there most integers are looked at or kept (one in nine above), and a
// wave with 1024 kept integers takes ten times its time (3e6 integers: 70000
// cycles beside 7000).  Sieve of 3e6 integers 41 -> 29 us, of 2^32 5.02 -> 4.91
// ms.  A batch's segments are all alike: its queries fill the chip together.
inline uint32_t cut_search(std::vector<Query>* q, uint64_t n, uint64_t wgs, uint32_t longest, bool one_range) {
  const uint32_t whole = fit_seg_len(n, wgs, longest, kKeySegUnit);
  for (Query& e : *q) e.seg_len = whole;
  if (!one_range) return whole;
  Query low = (*q)[0];
  const uint64_t zl = static_cast<uint64_t>(32.0 * std::sqrt(static_cast<double>(low.top))) + 1;
  if (low.a >= zl || zl >= low.b) return whole;
  low.b = zl;
  low.seg_len = std::min(whole, fit_seg_len(zl - low.a, wgs, longest, kLowSegUnit));
  Query& rest = (*q)[0];
  rest.a = zl;
  rest.seg_len = fit_seg_len(rest.b - zl, wgs, longest, kKeySegUnit);
  // (The rest may need a round less than the whole: its segments are longer then.)
  const uint32_t longer = std::max(low.seg_len, rest.seg_len);
  q->insert(q->begin(), low);
  return longer;
}

// Bits of a word's index: indices run up to segments per workgroup * seg_len - 1,
// and the bit length of that product keeps the all-ones index free.
inline uint32_t bits_of(uint64_t v) {  // the least b with v < 2^b
  uint32_t b = 0;
  while (b < 64 && (v >> b)) ++b;
  return b;
}
inline uint32_t index_bits(uint64_t n_segs, uint64_t wgs, uint32_t seg_len) {
  return std::max(1u, bits_of((n_segs + wgs - 1) / wgs * seg_len));
}

// Where the first level's words came from: enough to turn a word's index back
// into its integer.
struct WordSource {
  const Query* queries;
  const uint64_t* seg_prefix;
  uint32_t n_queries;
  uint32_t seg_len, W;  // the longest segment; sieve workgroups
  uint32_t li_bits;
  int batch;
};

// The integer with index li of sieve workgroup w, and its query (0 unless
// batched).  Workgroup w sieves the segments w, w + W, ..., each at the next
// multiple of seg_len of its indices.
__host__ __device__ inline uint64_t word_integer(const WordSource& S, uint32_t w, uint64_t li, uint32_t* grp) {
  const uint64_t s = w + (li / S.seg_len) * S.W;
  uint32_t lo = 0, hi = S.n_queries;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (S.seg_prefix[mid] <= s)
      lo = mid;
    else
      hi = mid;
  }
  *grp = S.batch ? lo : 0u;
  return S.queries[lo].a + (s - S.seg_prefix[lo]) * S.queries[lo].seg_len + li % S.seg_len;
}

}  // namespace bx
