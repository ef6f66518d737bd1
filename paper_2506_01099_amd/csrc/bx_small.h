// The small-query size class: a range [a, b) of at most T integers (one LDS
// tile) handled from start to end by one workgroup, with no word written to
// HBM and no partition or join launch.  The workgroup sieves rad(x) for x in
// [a, b] (Algorithm 1 on one tile: the powers q <= T from a static slot per
// multiple, every other power q <= b at its one possible multiple), applies the
// member test, takes the fingerprint of every kept set {rad(x), rad(x+1)} (of
// the query too, in batched calls) and joins them in an LDS hash table as the
// partition join does (Algorithm 3's insert step: every earlier equal
// fingerprint on the probe chain is a candidate).  Candidates go to the same
// verification as those of the passes.
//
// What bounds it is the look at every power up to b (8.4e4 at 2^40) by one
// workgroup (PowerTables).  The join's table lies over the tile once the
// fingerprints are in registers, which leaves room for two workgroups per CU:
// 300 queries of up to 8192 integers in one round of them.  Their
// fingerprints take one kept integer per lane (300 queries 28 -> 19 us, one of
// 4096 integers 12 -> 8).
#pragma once
#include "bx_kernels.h"

namespace bx {

struct SmallParams {
  const Query* queries;
  const uint32_t* list;  // indices of the small queries, one per workgroup
  int batch;
  uint32_t prune;
  PowerTables powers;
  uint32_t n_dense;        // powers.pw[0, n_dense) have slots (q <= T)
  const MidSlot* slots;    // their multiples in T + 1 integers
  uint32_t n_slots;
  uint64_t fp_mask;
  Cand* cand;
  uint32_t cand_cap;
  uint32_t* flags;
  unsigned long long* acc;  // acc[kAccEntries], acc[kAccJoined]
};

// T: the largest query length served (2048 or 8192, the tiles with slots);
// BLOCK threads per workgroup.
template <int T, int BLOCK>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(BLOCK / 128 > 4 ? 8 : 4))) void k_small(SmallParams P) {
  constexpr int ITER = T / BLOCK;
  static_assert(ITER <= 32 && (ITER % 2 == 0), "kept bits; two parts");
  constexpr int SLOTS = (dense_slot_cap(T) + BLOCK - 1) / BLOCK;
  constexpr uint32_t kPart = T / 2;  // kept integers joined at once (table of T slots, load <= 0.5)
  constexpr uint32_t kEmpty = 0xFFFFFFFFu;
  constexpr uint32_t kIdxMask = (1u << kJoinIdxBits) - 1;
  static_assert(T % BLOCK == 0 && kPart < (1u << kJoinIdxBits), "tile and index field");
  __shared__ union {
    uint64_t tile[T + 1];  // rad(a + i)
    struct {
      uint64_t fp[kPart];  // fingerprints of the kept integers, in order
      uint32_t table[T];
    } join;
  } sh;
  __shared__ uint16_t where[kPart];  // their i
  __shared__ uint32_t wsum[BLOCK / 64];
  const int tid = threadIdx.x;
  note_time(P.flags, K_SMALL);
  const uint32_t qi = P.list[blockIdx.x];
  const uint64_t qa = P.queries[qi].a, qb = P.queries[qi].b;
  const uint32_t L = static_cast<uint32_t>(qb - qa);  // 2 <= L <= T (checked by the host)
  const uint32_t grp = P.batch ? qi : 0u;
  const double S = static_cast<double>(qa), Ld = static_cast<double>(L);
  MidSlot slot[SLOTS];
#pragma unroll
  for (int k = 0; k < SLOTS; ++k) {
    const uint32_t t = tid + k * BLOCK;
    slot[k] = P.slots[t < P.n_slots ? t : 0u];
    if (t >= P.n_slots) slot[k].jq = T + 1;  // (past any query)
  }
  // Start values: a + i with the factor 2 reduced, for i in [0, L].
  for (uint32_t i = tid; i <= L; i += BLOCK) sh.tile[i] = strip_two(qa + i);
  __syncthreads();
#pragma unroll
  for (int k = 0; k < SLOTS; ++k) {
    const uint32_t pos = static_cast<uint32_t>(first_multiple(S, slot[k].q, slot[k].invq)) + slot[k].jq;
    if (pos <= L) lds_div(&sh.tile[pos], slot[k].p, inv32(slot[k].p));
  }
  // The other powers (q > T >= L): at most one multiple in [a, b] each.
  sparse_hits<BLOCK, 8>(P.powers, P.n_dense, S, Ld, tid, [&](uint32_t j, uint32_t p) { lds_div(&sh.tile[j], p, inv32(p)); });
  __syncthreads();
  // Member test; the kept integers are numbered over the workgroup and their
  // fingerprints made one per lane (made where they are found, eight rounds of
  // which few lanes take part, they took a third of the kernel).
  uint32_t keep = 0, mine = 0;  // bit it: integer it * BLOCK + tid
#pragma unroll
  for (int it = 0; it < ITER; ++it) {
    const uint32_t i = it * BLOCK + tid;
    if (i < L && (!P.prune || may_pair(qa + i, sh.tile[i], sh.tile[i + 1], qb))) {
      keep |= 1u << it;
      ++mine;
    }
  }
  uint32_t n;
  const uint32_t first = block_exclusive_scan<BLOCK>(mine, wsum, &n);
  constexpr int OWN = (T + BLOCK - 1) / BLOCK;  // kept integers tid + k * BLOCK
  uint64_t fp[OWN];
  uint32_t at[OWN];
#pragma unroll
  for (int part = 0; part < 2; ++part) {
    if (part * kPart >= n) break;  // uniform
    uint32_t idx = first - part * kPart;
    for (uint32_t m = keep; m; m &= m - 1, ++idx)
      if (idx < kPart) where[idx] = static_cast<uint16_t>(__builtin_ctz(m) * BLOCK + tid);
    __syncthreads();
#pragma unroll
    for (int k = part * OWN / 2; k < (part + 1) * OWN / 2; ++k) {
      const uint32_t e = k * BLOCK + tid;
      if (e < n) {
        const uint32_t i = where[e - part * kPart];
        const uint64_t r0 = sh.tile[i], r1 = sh.tile[i + 1];
        at[k] = i;
        fp[k] = (key64(r0 < r1 ? r0 : r1, r0 < r1 ? r1 : r0, grp) >> 11) & P.fp_mask;
      }
    }
    __syncthreads();
  }
  if (tid == 0 && n) {
    atomicAdd(&P.acc[kAccEntries], static_cast<unsigned long long>(n));
    atomicAdd(&P.acc[kAccJoined], static_cast<unsigned long long>(n));
  }
  const uint64_t qbits = static_cast<uint64_t>(qi) << kGrpShift;
  auto found = [&](uint32_t i, uint32_t o, uint64_t f) {
    const uint32_t k = atomicAdd(&P.flags[kFlagCand], 1u);
    if (k < P.cand_cap) {
      Cand c;
      c.a = make_entry(P.batch ? (i | qbits) : qa + i, f);
      c.b = make_entry(P.batch ? (o | qbits) : qa + o, f);
      P.cand[k] = c;
    }
  };
  // Inserts: each walks its probe chain to the first empty slot and compares
  // with every occupied slot whose tag matches.  Equal fingerprints walk the
  // same chain, so the one that claims the later slot reports the pair (once).
  // More than kPart kept integers (low ranges, the member test off) are joined
  // part by part: those after a part probe it.
#pragma unroll
  for (int part = 0; part < 2; ++part) {
    const uint32_t p0 = part * kPart;
    if (p0 >= n) break;  // uniform
    uint32_t slots = 256;
    while (slots < 2 * min(n - p0, kPart) && slots < static_cast<uint32_t>(T)) slots <<= 1;
    for (uint32_t s = tid; s < slots; s += BLOCK) sh.join.table[s] = kEmpty;
#pragma unroll
    for (int k = part * OWN / 2; k < (part + 1) * OWN / 2; ++k) {
      const uint32_t e = k * BLOCK + tid;
      if (e >= n) continue;
      sh.join.fp[e - p0] = fp[k];
      where[e - p0] = static_cast<uint16_t>(at[k]);
    }
    __syncthreads();
#pragma unroll
    for (int k = part * OWN / 2; k < (part + 1) * OWN / 2; ++k) {
      const uint32_t e = k * BLOCK + tid;
      if (e >= n) continue;
      const uint32_t h = static_cast<uint32_t>(fp[k]);
      const uint32_t word = (h & ~kIdxMask) | (e - p0);
      for (uint32_t s = h & (slots - 1);; s = (s + 1) & (slots - 1)) {
        const uint32_t v = atomicCAS(&sh.join.table[s], kEmpty, word);
        if (v == kEmpty) break;
        const uint32_t o = v & kIdxMask;
        if (((v ^ word) & ~kIdxMask) == 0 && sh.join.fp[o] == fp[k]) found(at[k], where[o], fp[k]);
      }
    }
    __syncthreads();
    if (part == 1 || n <= kPart) break;
#pragma unroll
    for (int k = OWN / 2; k < OWN; ++k) {
      const uint32_t e = k * BLOCK + tid;
      if (e >= n) continue;
      const uint32_t h = static_cast<uint32_t>(fp[k]);
      uint32_t s = h & (slots - 1);
      for (uint32_t v = sh.join.table[s]; v != kEmpty; s = (s + 1) & (slots - 1), v = sh.join.table[s]) {
        const uint32_t o = v & kIdxMask;
        if (((v ^ h) & ~kIdxMask) == 0 && sh.join.fp[o] == fp[k]) found(at[k], where[o], fp[k]);
      }
    }
    __syncthreads();
  }
}

}  // namespace bx
