// The key sieve of the searches: Algorithm 1 as far as the join needs it.
//
// The join takes only the integers x that pass the member test, almost all of
// them with x and x + 1 non-squarefree (10.7%), so rad(x) is needed for few x.
// k_sieve_keys therefore keeps, per integer, one bit (x is a multiple of the
// square of a prime) and the product of the larger prime powers' factors (the
// cell E), finds the kept x from the bits, and computes rad(x) and rad(x + 1)
// by one division each for those alone:
//
//   e(x) = x / rad(x) = 2^(a-1) * s(x) * E(x)
//     2^(a-1)  from the trailing zeros of x,
//     s(x)     one factor 3, 5, 7 for 9, 25, 49 | x, from x's residues,
//     E(x)     one factor p for every other odd power p^k | x, k >= 2.
//
// A wave sieves a subtile of 1024 integers on its own: its cells, bits and
// kept list are private to it, so no barrier falls inside a subtile (LDS
// accesses of one wave execute in order).  The words of the kept x leave
// through per-bucket queues in LDS, from which any wave writes out a run as
// soon as the run is claimed, without a barrier too (put_words).  The workgroup
// meets only to list the hits of the powers above 361: per chunk of 2^18
// integers those of the powers above 2^16, per block of 2^17 all of them.
#pragma once
#include "bx_kernels.h"

namespace bx {

constexpr int kSub = 1024;               // integers of a subtile
constexpr int kPerLane = kSub / 64;      // consecutive integers of a lane
static_assert(kKeySegUnit == 4 * kSub && kLowSegUnit == kSub / 4, "segments in subtiles");
constexpr int kKeyBlock = 1024;          // threads of a workgroup
constexpr int kKeyWaves = kKeyBlock / 64;
constexpr uint32_t kRow = kSub * kKeyWaves;  // integers of a row of subtiles
constexpr uint32_t kKeyChunk = 1u << 18;
constexpr uint32_t kKeyLen = 1u << 17;
constexpr uint32_t kKeySubs = kKeyLen / kSub;
constexpr uint32_t kMidMax = 1u << 16;    // powers up to here are hit through static slots
constexpr int kMidPer = 2;                // of them per thread (1974 slots at kKeyLen)
constexpr uint32_t kHitMax = 2304;        // hits of a block held in LDS (about 2030 at 2^42)
constexpr uint32_t kSparseMax = 512;      // hits of a chunk by powers above kMidMax (about 200)
constexpr uint32_t kKeySpill = 1u << 15;  // per workgroup in device memory: hits past kSparseMax, then past kHitMax
constexpr uint32_t kRecMax = 128;         // kept integers a wave turns into words at once
constexpr int kCellPitch = kSub + 4;      // cells 0 .. kSub of a subtile
constexpr int kBitPitch = kSub / 32 + 2;  // bits 0 .. kSub
constexpr uint32_t kQueueSlots = 8192;    // words in the bucket queues, together

// The powers with a static slot per multiple in a subtile (73 slots, in two
// rounds); 27 stands for 27, 81, 243 and 729 (lut3).  Every odd power up to
// kFixedQMax, and 729, has its slot here or is in s(x).
constexpr uint32_t kFixedQMax = 361;
constexpr int kFixed = 7, kFixedSlots = 73, kFixedPer = 2;
__device__ constexpr uint16_t kFixedQ[kFixed] = {27, 125, 343, 121, 169, 289, 361};
__device__ constexpr uint8_t kFixedP[kFixed] = {3, 5, 7, 11, 13, 17, 19};

// Tables by residues, made on the host and copied into LDS (made there they
// took 3 of the 19 us of a short range).  By x mod 729, for 27 | x: 3^(v-2),
// v = min(v_3(x), 6).  By x mod 225 and x mod 49: the bits of small_f.  (Long
// enough to need no reduction.)
struct KeyLuts {
  double2 small_f[64];  // s(x), s(x + 1) by 9 | x, 9 | x + 1, 25 | x, ...
  uint8_t lut3[729 + kSub + 3], lut225[225 + kSub + 3], lut49[49 + kSub + 3];
};

struct KeyParams {
  const Query* queries;
  const uint64_t* seg_prefix;  // n_queries + 1: first segment of each query
  uint32_t n_queries;
  uint64_t n_segs;
  uint32_t seg_len;  // the longest segment
  const KeyLuts* luts;
  const MidSlot* mid;
  PowerTables powers;
  uint32_t sparse_first;  // powers above kMidMax in powers.pw
  uint64_t* spill;       // kKeySpill words per workgroup
  uint32_t* flags;
  int batch;
  uint32_t ph_lo, ph_len;  // FILTER: keep x only when pass_hash(key) is in [ph_lo, ph_lo + ph_len)
  uint32_t b1bits;   // first-level bucket = low b1bits bits of key64
  uint32_t li_bits;  // of a word (l1_word)
  uint64_t kl_mask;
  uint32_t W;      // workgroups
  uint64_t* l1;    // region (w, b) of bucket b written by workgroup w: l1 + (w * B1 + b) * cap1
  uint32_t cap1;   // words per region (a multiple of 64; B1 * cap1 < 2^29)
  uint32_t* cnt1;  // W x B1 fill counts, written at the end of the kernel
  unsigned long long* entries;  // += words written
};

// A queue writes out runs of 2^run_log words: half its slots, at most 64.
__host__ __device__ constexpr uint32_t run_log(uint32_t b1bits) { return b1bits > 6 ? 12 - b1bits : 6; }

// LDS of the workgroup.  The queues: bucket b has the 2^(13 - b1bits) slots
// from b << (13 - b1bits); an empty slot holds kNoWord.
struct KeySh {
  __align__(16) uint32_t cell[kKeyWaves * kCellPitch];
  uint64_t queue[kQueueSlots];
  __align__(16) KeyLuts lut;
  uint64_t sparse[kSparseMax];        // position in the chunk | p << 19
  uint32_t bits[kKeyWaves * kBitPitch], cbits[kKeyWaves * kBitPitch];
  uint32_t hits[kHitMax];             // position in the subtile | p << 11, by subtile
  uint32_t hcnt[kKeySubs + 1];        // hits per subtile, then their first index
  uint32_t cur[kB1Max];               // words claimed per bucket
  uint32_t sparse_n, spill_n;
  uint16_t rec[kKeyWaves * kRecMax];  // kept integers of each wave's subtile
};
static_assert(sizeof(KeySh) <= 160 * 1024, "LDS of a CU");

// first_multiple for a small q.
__device__ __forceinline__ uint32_t first_multiple_small(double S, uint32_t q) {
  const double qd = static_cast<double>(q);
  return static_cast<uint32_t>(first_multiple(S, qd, (1.0 / qd) * (1.0 - 0x1p-46)));
}

// This thread's index, not to be hoisted: addresses made from it are made where
// they are used, so that they take no registers in the rows.
__device__ __forceinline__ uint32_t thread_here() {
  uint32_t t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

__device__ __forceinline__ void set_priority(uint32_t p) {  // uniform
  if (p == 0)
    __builtin_amdgcn_s_setprio(0);
  else if (p == 1)
    __builtin_amdgcn_s_setprio(1);
  else if (p == 2)
    __builtin_amdgcn_s_setprio(2);
  else
    __builtin_amdgcn_s_setprio(3);
}

// Waits until this wave's loads and stores are done (vmcnt 0).
__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// a * b, or 0 (which stays 0) once the product passes 32 bits.
__device__ __forceinline__ uint32_t mul_or_zero(uint32_t a, uint32_t b) { return __umulhi(a, b) ? 0u : a * b; }

// Multiplies cells of this wave: cell[pos[u]] by v[u] where on[u].  Two lanes
// may hit one cell at once: each exchange leaves the product of the cell and
// of the values in the lanes' hands unchanged, and a lane is done when it got
// 1 back.  v[u] becomes the value left: the last to finish on a cell leaves the
// whole product.
template <int N>
__device__ __forceinline__ void mul_cells(uint32_t* cell, const uint32_t (&pos)[N], uint32_t (&v)[N], const bool (&on)[N]) {
  uint32_t old[N];
#pragma unroll
  for (int u = 0; u < N; ++u) old[u] = on[u] ? atomicExch(&cell[pos[u]], v[u]) : 1u;
#pragma unroll
  for (int u = 0; u < N; ++u) {
    while (old[u] != 1u) {
      v[u] = mul_or_zero(old[u], atomicExch(&cell[pos[u]], 1u));
      old[u] = atomicExch(&cell[pos[u]], v[u]);
    }
  }
}

// The rare x whose cell passed 32 bits: then rad(x) < 2^10 * 2 * 105, every
// prime of E(x) is at most x / E(x) < 2^10, and dividing out the primes below
// 2^10 leaves 1 or a product of primes dividing x once.
__device__ __attribute__((noinline)) uint64_t rad_by_division(uint64_t x) {
  uint64_t r = 1;
  if ((x & 1) == 0) {
    r = 2;
    x >>= __builtin_ctzll(x);
  }
  for (uint32_t d = 3; d < 1024; d += 2) {
    if (x % d) continue;
    r *= d;
    while (x % d == 0) x /= d;
  }
  return r * x;
}

__device__ __forceinline__ bool any_lane(bool p) { return __builtin_amdgcn_ballot_w64(p) != 0; }

// Lanes below this one that are in m.
__device__ __forceinline__ uint32_t rank_in(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(m >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0u));
}

// Hands the words of this wave's lanes (those with `keep`) to their buckets.
//
// A word claims the next place `pos` of its bucket, which is its index in this
// workgroup's region as well, and goes into the queue's slot pos mod slots.
// Whoever claims the last place of a run (half a queue, at most 64 words)
// writes the run out: one lane per slot takes the slot's word and stores it,
// so the stores of a run are consecutive and, runs being aligned, full lines
// or halves of them.  A slot passes from word to word by compare-and-swap
// (empty -> word) and exchange (word -> empty).  A lane that finds its slot
// still taken, or not yet filled, tries again; each round of the loop tries
// all of them, and the oldest run's words never wait for anything, so the loop
// ends.  (A word may be taken with a neighbouring run of its bucket: the
// region is an unordered list.)  Two words per lane at once were no faster
// (2^36: 96 against 92 ms): twice as many runs end in a round.
__device__ __forceinline__ void put_words(KeySh& sh, const KeyParams& P, bool keep, uint32_t bk, uint64_t word) {
  const uint32_t lane = lane_id();
  const uint32_t slog = 13 - P.b1bits, smask = (1u << slog) - 1u;
  const uint32_t hlog = run_log(P.b1bits), hmask = (1u << hlog) - 1u, most = 64u >> hlog;
  unsigned long long* const queue = reinterpret_cast<unsigned long long*>(sh.queue);
  uint32_t pos = 0;
  if (P.b1bits == 0) {  // one bucket: claimed for the wave at once
    const uint64_t m = __builtin_amdgcn_ballot_w64(keep);
    uint32_t base = 0;
    if (lane == 0) base = atomicAdd(&sh.cur[0], static_cast<uint32_t>(__popcll(m)));
    pos = __builtin_amdgcn_readfirstlane(base) + rank_in(m);
  } else if (keep) {
    pos = atomicAdd(&sh.cur[bk], 1u);
  }
  unsigned long long* const slot = queue + ((bk << slog) + (pos & smask));
  uint64_t runs = __builtin_amdgcn_ballot_w64(keep && (pos & hmask) == hmask);  // lanes with a run to write out
  bool put = keep, take = false;
  unsigned long long* from = queue;
  uint32_t to = ~0u;
  uint64_t* const mine = P.l1 + blockIdx.x * (static_cast<uint64_t>(P.cap1) << P.b1bits);
  for (;;) {
    if (put) put = atomicCAS(slot, kNoWord, word) != kNoWord;
    if (runs && !any_lane(take)) {
      // The next 64 >> hlog runs, one lane per word: lane k gets the k-th
      // run's bucket and place, then the run's lanes do.  (Lanes without a run
      // push to lane 63, which is not read from: a run has two words or more.)
      const uint32_t rank = rank_in(runs);
      const bool has = (runs >> lane) & 1ull, give = has && rank < most;
      const int pushed = __builtin_amdgcn_ds_permute(give ? static_cast<int>(rank * 4) : 63 * 4,
                                                     static_cast<int>(((pos >> hlog) << 10) | bk));
      const uint32_t run = static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(static_cast<int>(lane >> hlog) * 4, pushed));
      const uint32_t rb = run & 1023u, rp = ((run >> 10) << hlog) + (lane & hmask);
      take = (lane >> hlog) < static_cast<uint32_t>(__popcll(runs));
      runs = __builtin_amdgcn_ballot_w64(has && !give);
      from = queue + (take ? (rb << slog) + (rp & smask) : 0u);
      to = rp < P.cap1 ? rb * P.cap1 + rp : ~0u;
    }
    if (take) {
      const unsigned long long w = atomicExch(from, kNoWord);
      take = w == kNoWord;
      if (!take && to != ~0u) mine[to] = w;  // (a region that overflows is reported at the end)
    }
    if (!any_lane(put || take) && !runs) break;
  }
}

// One workgroup per CU walks its segments (s mod W).
//
// Bound by instruction issue: 30 VALU lane-operations per integer, issued in
// 75% of the cycles.  (A tile of 64-bit radicals divided in place by
// compare-and-swap took 42 and 45%, with three barriers per 8192 integers.)
// Of a workgroup's cycles at 2^40, 74% are rows of subtiles, 14% the look at
// the large powers (in single precision first: in double it took twice that),
// 4% the hit lists and 7% waits at their barriers; the waves take turns at
// high priority so that they reach these at nearly one time.  A subtile of 512
// took 70% longer (latency); a sorted stage with coalesced flushes instead of
// the queues 40%.
// 2^36 integers 158 -> 76.7 ms, 2^32 9.55 -> 4.8 ms, 2^28 at 2^40 0.71 -> 0.29.
//
// FILTER: one of several passes.  Every record's radicals are made, and those of
// the pass wait in lanes until 64 are together, so that the key and the queues
// are paid for the pass's own records alone.
//
// ALL: the member test is off and every integer is kept: no bits, and no list
// (which took 1024 records in eight parts; 2^32 29.6 -> 20.2 ms, and with FILTER
// 2^36 in five passes 2278 -> 1203 ms).  Else x that cannot be a member of any
// pair (may_pair) are dropped.
template <bool FILTER, bool ALL>
__global__ __launch_bounds__(kKeyBlock) void k_sieve_keys(KeyParams P) {
  __shared__ KeySh sh;
  note_time(P.flags, K_SIEVE);
  const uint32_t lane = lane_id();
  const uint32_t wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint32_t* cell = sh.cell + wid * kCellPitch;
  uint32_t* bits = sh.bits + wid * kBitPitch;
  uint32_t* cbits = sh.cbits + wid * kBitPitch;
  uint16_t* rec = sh.rec + wid * kRecMax;
  {
    const uint32_t tid = threadIdx.x;
    for (uint32_t i = tid; i < kKeyWaves * kCellPitch; i += kKeyBlock) sh.cell[i] = 1u;
    for (uint32_t i = tid; i < kQueueSlots; i += kKeyBlock) sh.queue[i] = kNoWord;
    for (uint32_t i = tid; i < kKeyWaves * kBitPitch; i += kKeyBlock) sh.bits[i] = sh.cbits[i] = 0u;
    static_assert(sizeof(KeyLuts) % 4 == 0, "copied in words");
    for (uint32_t i = tid; i < sizeof(KeyLuts) / 4; i += kKeyBlock)
      reinterpret_cast<uint32_t*>(&sh.lut)[i] = reinterpret_cast<const uint32_t*>(P.luts)[i];
    for (uint32_t b = tid; b < kB1Max; b += kKeyBlock) sh.cur[b] = 0;
  }
  // This lane's static slots: a power's multiple slot_jq past its first one in
  // the subtile.
  uint32_t slot_q[kFixedPer], slot_jq[kFixedPer], slot_p[kFixedPer], slot_adv[kFixedPer];
#pragma unroll
  for (int u = 0; u < kFixedPer; ++u) {
    slot_q[u] = slot_jq[u] = slot_adv[u] = 0;
    slot_p[u] = 1;
    uint32_t first = 0;
    const uint32_t t = lane + 64 * u;
#pragma unroll
    for (int k = 0; k < kFixed; ++k) {
      const uint32_t q = kFixedQ[k], n = kSub / q + 1;
      if (t >= first && t < first + n) {
        slot_q[u] = q;
        slot_jq[u] = (t - first) * q;
        slot_p[u] = kFixedP[k];
        slot_adv[u] = kRow % q;
      }
      first += n;
    }
  }
  constexpr uint32_t kFree = 64 * kFixedPer - kFixedSlots;  // lanes of the last round left for listed hits
  uint64_t* spill = P.spill + static_cast<uint64_t>(blockIdx.x) * kKeySpill;
  constexpr uint32_t kSpillHalf = kKeySpill / 2;

  uint64_t li0 = 0;  // index of the segment's first integer in this workgroup's sequence
  for (uint64_t s = blockIdx.x; s < P.n_segs; s += P.W, li0 += P.seg_len) {
    // Segment s -> its query: the prefix is searched 64 entries at a time.
    uint32_t qlo = 0, qn = P.n_queries;
    while (qn > 1) {
      const uint32_t step = (qn + 63) / 64;
      const uint32_t at = lane * step;
      const uint64_t m = __ballot(at < qn && P.seg_prefix[qlo + (at < qn ? at : 0u)] <= s);
      const uint32_t k = static_cast<uint32_t>(__popcll(m)) - 1;  // lane 0 always holds
      qlo += k * step;
      qn = min(step, qn - k * step);
    }
    const uint32_t qi = __builtin_amdgcn_readfirstlane(qlo);
    const uint64_t qb = P.queries[qi].top;
    const uint64_t seg0 = P.queries[qi].a + (s - P.seg_prefix[qi]) * static_cast<uint64_t>(P.queries[qi].seg_len);
    const uint64_t seg1 = min(seg0 + P.queries[qi].seg_len, P.queries[qi].b);
    const uint32_t grp = P.batch ? qi : 0u;

    for (uint64_t start = seg0; start < seg1; start += kKeyLen) {
      const uint32_t tid = thread_here();
      const uint32_t len = static_cast<uint32_t>(min(static_cast<uint64_t>(kKeyLen), seg1 - start));
      const uint32_t nsub = (len + kSub - 1) / kSub;
      const double S = static_cast<double>(start);
      // 1. Every second block begins a chunk: the hits of the powers above
      // kMidMax on its positions 0 .. chunk length.
      const uint32_t c0 = static_cast<uint32_t>((start - seg0) % kKeyChunk);  // the block's place in the chunk
      MidSlot m[kMidPer];
#pragma unroll
      for (int u = 0; u < kMidPer; ++u) m[u] = P.mid[tid + u * kKeyBlock];
      if (tid < kKeySubs) sh.hcnt[tid] = 0;
      if (c0 == 0) {
        if (tid == 0) sh.sparse_n = 0;
        __syncthreads();
        const double Lc = static_cast<double>(min(static_cast<uint64_t>(kKeyChunk), seg1 - start));
        sparse_hits<kKeyBlock, 8>(P.powers, P.sparse_first, S, Lc, tid, [&](uint32_t j, uint32_t p) {
          const uint64_t e = j | (static_cast<uint64_t>(p) << 19);
          const uint32_t k = atomicAdd(&sh.sparse_n, 1u);
          if (k < kSparseMax)
            sh.sparse[k] = e;
          else if (k - kSparseMax < kSpillHalf)
            spill[k - kSparseMax] = e;
          else
            atomicOr(&P.flags[kFlagSpillOverflow], 1u);
        });
      }
      if (tid == 0) sh.spill_n = 0;
      __syncthreads();
      // 2. The block's hits by subtile: positions 0 .. len of the multiples of
      // the powers above kFixedQMax (but 729), counted, then placed.  A hit on
      // the first integer of a subtile also belongs to the subtile before (as
      // its last value, x + 1 of its last x).
      const uint32_t nsp = min(sh.sparse_n, kSparseMax + kSpillHalf);
      auto sparse_at = [&](uint32_t k, uint32_t* pos, uint32_t* p) {  // whether hit k falls in the block
        const uint64_t e = k < kSparseMax ? sh.sparse[k] : spill[k - kSparseMax];
        *pos = (static_cast<uint32_t>(e) & 0x7FFFFu) - c0;
        *p = static_cast<uint32_t>(e >> 19);
        return *pos <= len;  // (a hit before the block wraps around)
      };
      constexpr int kOwn = kMidPer + 1;  // this thread's slots, and one listed hit
      uint32_t hpos[kOwn], hp[kOwn], hrank[kOwn], hdup[kOwn];
#pragma unroll
      for (int u = 0; u < kMidPer; ++u) {
        const uint32_t pos = static_cast<uint32_t>(first_multiple(S, m[u].q, m[u].invq)) + m[u].jq;
        hpos[u] = pos <= len ? pos : ~0u;
        hp[u] = m[u].p;
      }
      hpos[kMidPer] = ~0u;
      if (tid < nsp && !sparse_at(tid, &hpos[kMidPer], &hp[kMidPer])) hpos[kMidPer] = ~0u;
      auto count = [&](uint32_t pos, uint32_t* rank, uint32_t* dup) {
        const uint32_t sub = pos / kSub;
        if (sub < nsub) *rank = atomicAdd(&sh.hcnt[sub], 1u);
        if (pos % kSub == 0 && pos) *dup = atomicAdd(&sh.hcnt[sub - 1], 1u);
      };
#pragma unroll
      for (int u = 0; u < kOwn; ++u)
        if (hpos[u] != ~0u) count(hpos[u], &hrank[u], &hdup[u]);
      __syncthreads();
      if (wid == 0) {
        static_assert(kKeySubs == 128, "two counts per lane");
        const uint32_t n0 = sh.hcnt[2 * lane], n1 = sh.hcnt[2 * lane + 1];
        const uint32_t end = wave_inclusive_scan(n0 + n1);
        sh.hcnt[2 * lane] = end - n0 - n1;
        sh.hcnt[2 * lane + 1] = end - n1;
        if (lane == 63) sh.hcnt[kKeySubs] = end;
      }
      __syncthreads();
      // Hits past kHitMax go to the second half of the spill, which every
      // subtile then reads: position in the subtile | subtile << 11 | p << 21.
      auto put_spill = [&](uint32_t sub, uint32_t at, uint32_t p) {
        const uint32_t o = atomicAdd(&sh.spill_n, 1u);
        if (o < kSpillHalf)
          spill[kSpillHalf + o] = at | (sub << 11) | (static_cast<uint64_t>(p) << 21);
        else
          atomicOr(&P.flags[kFlagSpillOverflow], 1u);
      };
      auto place = [&](uint32_t pos, uint32_t p, uint32_t rank, uint32_t dup) {
        auto put = [&](uint32_t sub, uint32_t at, uint32_t o) {
          if (o < kHitMax)
            sh.hits[o] = at | (p << 11);
          else
            put_spill(sub, at, p);
        };
        const uint32_t sub = pos / kSub;
        if (sub < nsub) put(sub, pos % kSub, sh.hcnt[sub] + rank);
        if (pos % kSub == 0 && pos) put(sub - 1, kSub, sh.hcnt[sub - 1] + dup);
      };
#pragma unroll
      for (int u = 0; u < kOwn; ++u)
        if (hpos[u] != ~0u) place(hpos[u], hp[u], hrank[u], hdup[u]);
      for (uint32_t k = tid + kKeyBlock; k < nsp; k += kKeyBlock) {  // a chunk with more hits than threads
        uint32_t pos, p;
        if (!sparse_at(k, &pos, &p)) continue;
        if (pos / kSub < nsub) put_spill(pos / kSub, pos % kSub, p);
        if (pos % kSub == 0 && pos) put_spill(pos / kSub - 1, kSub, p);
      }
      __syncthreads();
      const uint32_t nspill = min(sh.spill_n, kSpillHalf);
      // Nothing the rows need is in flight: said here, so that no wait for
      // memory (for the stores of words, then) falls inside the rows.
      wait_loads();

      // 3. The wave's residues at its first subtile, then advanced by a row.
      const double Sw = S + static_cast<double>(wid * kSub);
      uint32_t f[kFixedPer];
#pragma unroll
      for (int u = 0; u < kFixedPer; ++u) f[u] = slot_q[u] ? first_multiple_small(Sw, slot_q[u]) : 0u;
      const double Sl = Sw + static_cast<double>(kPerLane * lane);
      uint32_t r9 = first_multiple_small(Sl, 9), r25 = first_multiple_small(Sl, 25), r49 = first_multiple_small(Sl, 49);
      auto residue = [&](uint32_t q) {
        return __builtin_amdgcn_readfirstlane((q - first_multiple_small(Sw, q)) % q);
      };
      uint32_t o729 = residue(729), o225 = residue(225), o49 = residue(49);
      const uint32_t c4 = 0x11111u << ((4u - (static_cast<uint32_t>(start) & 3u)) & 3u);
      for (uint32_t sub = wid; sub < nsub; sub += kKeyWaves) {
        // The SIMD's four waves (wid / 4) take the highest priority in turn:
        // by age alone the oldest runs ahead, and the block's end waits for
        // the youngest, which then has the SIMD to itself.
        set_priority((sub / kKeyWaves + wid / 4) & 3u);
        const uint64_t x0 = start + static_cast<uint64_t>(sub) * kSub;
        const double x0d = S + static_cast<double>(sub * kSub);
        const uint32_t cntv = min(static_cast<uint32_t>(kSub), len - sub * kSub);
        const bool lower = !ALL && (x0 <= 3 || x0 <= (qb >> 1));
        // Below b / 2 a squarefree y of {x, x + 1} with y * M <= b is kept
        // too, M = max(2, rad(z) - 1) of its neighbour z: then e(z) >= ethr.
        // With ethr small every x with a non-squarefree neighbour is looked
        // at (68% of them); else those next to a z with 105 * 2^(a-1) * E(z) >=
        // ethr, marked in cbits (from ethr = 1024 on at most a quarter).
        float ethr = 0.f;
        uint32_t look = 0;  // 0: the bits decide, 1: any, 2: one non-squarefree, 3: marked
        if (lower) {
          const double bd = static_cast<double>(qb);
          ethr = static_cast<float>(0.99 * x0d / (bd / x0d + 1.0));
          look = x0d * x0d <= bd + 8 ? 1 : ethr < 1024.f ? 2 : 3;
        }
        auto mark = [&](uint32_t pos, uint32_t e) {
          if constexpr (ALL) return;
          atomicOr(&bits[pos >> 5], 1u << (pos & 31u));
          if (look == 3) {
            const uint64_t z = x0 + pos;
            const int a1 = (z & 1) ? 0 : __builtin_ctzll(z) - 1;
            if (e == 0 || static_cast<float>(e) * 105.f * __builtin_ldexpf(1.f, a1) >= ethr)
              atomicOr(&cbits[pos >> 5], 1u << (pos & 31u));
          }
        };
        {
          const uint32_t h0 = min(sh.hcnt[sub], kHitMax), h1 = min(sh.hcnt[sub + 1], kHitMax);
          // Two rounds: the static slots, then the listed hits in the lanes
          // that have none.
          uint32_t pos[kFixedPer], v[kFixedPer];
          bool on[kFixedPer];
#pragma unroll
          for (int u = 0; u < kFixedPer; ++u) {
            pos[u] = f[u] + slot_jq[u];
            v[u] = slot_p[u];
            on[u] = pos[u] <= kSub;
            if (slot_p[u] == 3) v[u] = sh.lut.lut3[min(pos[u] + o729, 728u + kSub)];
          }
          {
            constexpr int u = kFixedPer - 1;
            if (lane >= 64 - kFree) {
              const uint32_t hi = h0 + lane - (64 - kFree);
              on[u] = hi < h1;
              const uint32_t e = sh.hits[on[u] ? hi : 0u];
              pos[u] = e & 2047u;
              v[u] = e >> 11;
            }
          }
          mul_cells(cell, pos, v, on);
#pragma unroll
          for (int u = 0; u < kFixedPer; ++u)
            if (on[u]) mark(pos[u], v[u]);
          auto hit = [&](uint32_t at, uint32_t p) {
            const uint32_t one_pos[1] = {at};
            uint32_t one_v[1] = {p};
            const bool one_on[1] = {true};
            mul_cells(cell, one_pos, one_v, one_on);
            mark(at, one_v[0]);
          };
          for (uint32_t h = h0 + kFree + lane; __any(h < h1); h += 64) {
            if (h < h1) {
              const uint32_t e = sh.hits[h];
              hit(e & 2047u, e >> 11);
            }
          }
          if (nspill) {
            for (uint32_t h = lane; h < nspill; h += 64) {
              const uint64_t e = spill[kSpillHalf + h];
              if ((static_cast<uint32_t>(e >> 11) & 0x3FFu) == sub)
                hit(static_cast<uint32_t>(e) & 0x7FFu, static_cast<uint32_t>(e >> 21));
            }
            wait_loads();
          }
        }
        wave_sync();
        // Kept bits of this lane's integers X .. X + kPerLane - 1.
        constexpr uint32_t kLaneMask = (1u << kPerLane) - 1u;
        const uint16_t* bb = reinterpret_cast<const uint16_t*>(bits);
        static_assert(kPerLane == 16, "one halfword of bits per lane");
        const uint32_t ns = bb[lane] | (static_cast<uint32_t>(bb[lane + 1]) << 16) | c4 | (0x201u << r9) | (1u << r25) |
                            (1u << min(r49, 31u));
        uint32_t K = ns & (ns >> 1);
        if (look) {  // uniform
          if (look == 1) {
            K = kLaneMask;
          } else if (look == 2) {
            K = ns | (ns >> 1);
          } else {
            const uint16_t* cb = reinterpret_cast<const uint16_t*>(cbits);
            uint32_t C = cb[lane] | (static_cast<uint32_t>(cb[lane + 1]) << 16);
            // Powers of two alone: z = 0 mod 8 with 105 * 2^(a-1) >= ethr.
            const uint64_t X = x0 + kPerLane * lane;
            for (uint32_t k = static_cast<uint32_t>(-static_cast<int64_t>(X)) & 7u; k <= kPerLane; k += 8)
              if (105.f * __builtin_ldexpf(1.f, __builtin_ctzll(X + k) - 1) >= ethr) C |= 1u << k;
            K |= C | (C >> 1);
          }
        }
        K &= kLaneMask;
        if (cntv < static_cast<uint32_t>(kSub)) {  // uniform
          const uint32_t left = cntv > kPerLane * lane ? cntv - kPerLane * lane : 0u;
          if (left < kPerLane) K &= (1u << left) - 1u;
        }
        const uint32_t pc = __popc(K);
        const uint32_t inc = wave_inclusive_scan(pc);
        const uint32_t total = ALL ? cntv : __builtin_amdgcn_readlane(inc, 63);
        const uint64_t li = li0 + (x0 - seg0);
        const uint32_t x0odd = static_cast<uint32_t>(x0) & 1u;
        const bool wraps = static_cast<uint32_t>(x0) - 1u > 0xFFFFFFFFu - kSub - 1u;  // a multiple of 2^32 near the subtile
        auto put = [&](uint64_t klo, uint64_t khi, uint32_t i, bool keep) {
          const uint64_t h = key64(klo, khi, grp);
          put_words(sh, P, keep, static_cast<uint32_t>(h) & ((1u << P.b1bits) - 1u), l1_word(h, P.kl_mask, P.li_bits, li + i));
        };
        uint32_t held = 0, h0 = 0, h1 = 0, h2 = 0;  // FILTER: records waiting, one in each of the first lanes
        for (uint32_t rb = 0; rb < total; rb += kRecMax) {
          if constexpr (!ALL) {
            uint32_t kt = K, slot = inc - pc - rb;
            if (total <= kRecMax) {
              while (kt) {
                rec[slot++] = static_cast<uint16_t>(kPerLane * lane + __builtin_ctz(kt));
                kt &= kt - 1;
              }
            } else {
              for (; kt; ++slot, kt &= kt - 1)
                if (slot < kRecMax) rec[slot] = static_cast<uint16_t>(kPerLane * lane + __builtin_ctz(kt));
            }
            wave_sync();
          }
          const uint32_t nrec = min(total - rb, kRecMax);
          for (uint32_t q0 = 0; q0 < nrec; q0 += 64) {
            bool keep = q0 + lane < nrec;
            const uint32_t i = ALL ? (keep ? rb + q0 + lane : 0u) : rec[keep ? q0 + lane : 0u];
            const uint32_t E0 = cell[i], E1 = cell[i + 1];
            const double2 sf = sh.lut.small_f[sh.lut.lut225[i + o225] | sh.lut.lut49[i + o49]];
            const uint64_t x = x0 + i;
            const double xd = x0d + static_cast<double>(i);
            // The even one of x, x + 1 has the factor 2^(a-1), half its lowest
            // set bit (in the low word, but for multiples of 2^32).
            const uint32_t odd = (i & 1u) ^ x0odd, ev = static_cast<uint32_t>(x) + odd;
            double low = static_cast<double>(ev & (0u - ev));
            if (wraps && ev == 0) low = 0x1p32 * static_cast<double>((x + odd) >> 32 & (0 - ((x + odd) >> 32)));
            low *= 0.5;
            const double d0 = static_cast<double>(E0) * sf.x * (odd ? 1.0 : low);
            const double d1 = static_cast<double>(E1) * sf.y * (odd ? low : 1.0);
            // rad = x / e, an integer below 2^42: one Newton step on the
            // hardware's reciprocal of both e's product, rounded to the integer
            // by adding 2^52.  The e's are exact (each divides its integer); the
            // instruction is specified to 2^29 ulp (2^-23 relative), so the step
            // leaves 2^-46 and the four roundings 2^-51: rad is off by less than
            // 1/8 before it is rounded.
            const double dd = d0 * d1;
            double ri = __builtin_amdgcn_rcp(dd);
            ri = __builtin_fma(ri, __builtin_fma(-dd, ri, 1.0), ri);
            double q0d = __builtin_fma(xd, ri * d1, 0x1p52), q1d = __builtin_fma(xd + 1.0, ri * d0, 0x1p52);
            if (keep && (E0 == 0 || E1 == 0)) {
              q0d = 0x1p52 + static_cast<double>(E0 ? static_cast<uint64_t>(xd / d0) : rad_by_division(x));
              q1d = 0x1p52 + static_cast<double>(E1 ? static_cast<uint64_t>((xd + 1.0) / d1) : rad_by_division(x + 1));
            }
            constexpr uint64_t kMant = (1ull << 52) - 1;
            const uint64_t klo = __builtin_bit_cast(uint64_t, __builtin_fmin(q0d, q1d)) & kMant;
            const uint64_t khi = __builtin_bit_cast(uint64_t, __builtin_fmax(q0d, q1d)) & kMant;
            if (lower)
              keep = keep && may_pair(x, __builtin_bit_cast(uint64_t, q0d) & kMant, __builtin_bit_cast(uint64_t, q1d) & kMant, qb);
            if constexpr (FILTER) {
              keep = keep && pass_hash(klo, khi, grp) - P.ph_lo < P.ph_len;
              // The pass's records go behind those that wait (the others to the
              // remaining lanes): two radicals below 2^42 and a place below 2^10.
              const uint64_t m = __builtin_amdgcn_ballot_w64(keep);
              const uint32_t rank = rank_in(m), have = held + static_cast<uint32_t>(__popcll(m));
              const int to = static_cast<int>(((keep ? held + rank : have + lane - rank) & 63u) * 4u);
              const uint32_t w0 = __builtin_amdgcn_ds_permute(to, static_cast<int>(klo));
              const uint32_t w1 = __builtin_amdgcn_ds_permute(to, static_cast<int>(khi));
              const uint32_t w2 = __builtin_amdgcn_ds_permute(
                  to, static_cast<int>(static_cast<uint32_t>(klo >> 32) | static_cast<uint32_t>(khi >> 32) << 10 | i << 20));
              if (lane >= held) {
                h0 = w0;
                h1 = w1;
                h2 = w2;
              }
              held = have;
              const bool last = rb + q0 + 64 >= total;
              while (held >= 64 || (last && held)) {
                put(h0 | static_cast<uint64_t>(h2 & 1023u) << 32, h1 | static_cast<uint64_t>(h2 >> 10 & 1023u) << 32, h2 >> 20,
                    lane < held);
                h0 = w0;  // (those past the 64th, in the first lanes)
                h1 = w1;
                h2 = w2;
                held = held > 64 ? held - 64 : 0;
              }
            } else {
              put(klo, khi, i, keep);
            }
          }
          wave_sync();
        }
        // The cells and bits for the next subtile, the residues a row on.
        static_assert(kCellPitch == 4 * 256 + 4, "four stores per lane and one");
#pragma unroll
        for (uint32_t c = 0; c < 4; ++c) reinterpret_cast<uint4*>(cell)[64 * c + lane] = make_uint4(1u, 1u, 1u, 1u);
        if (lane == 0) reinterpret_cast<uint4*>(cell)[256] = make_uint4(1u, 1u, 1u, 1u);
        if (lane < kBitPitch) bits[lane] = 0u;
        if (look == 3 && lane < kBitPitch) cbits[lane] = 0u;
        wave_sync();
        auto step = [](uint32_t r, uint32_t c, uint32_t q) {
          const uint32_t t = r - c;
          return min(t, t + q);
        };
#pragma unroll
        for (int u = 0; u < kFixedPer; ++u) f[u] = step(f[u], slot_adv[u], slot_q[u]);
        r9 = step(r9, kRow % 9u, 9u);
        r25 = step(r25, kRow % 25u, 25u);
        r49 = step(r49, kRow % 49u, 49u);
        auto sstep = [](uint32_t r, uint32_t c, uint32_t q) { return r + c >= q ? r + c - q : r + c; };
        o729 = sstep(o729, kRow % 729u, 729u);
        o225 = sstep(o225, kRow % 225u, 225u);
        o49 = sstep(o49, kRow % 49u, 49u);
      }
      __builtin_amdgcn_s_setprio(0);
      __syncthreads();
    }
  }
  __syncthreads();
  // What the queues still hold: each bucket's last, unfinished run.
  const uint32_t slog = 13 - P.b1bits, smask = (1u << slog) - 1u, hmask = (1u << run_log(P.b1bits)) - 1u;
  uint64_t* const mine = P.l1 + blockIdx.x * (static_cast<uint64_t>(P.cap1) << P.b1bits);
  for (uint32_t i = threadIdx.x; i < kQueueSlots; i += kKeyBlock) {
    const uint32_t b = i >> slog, n = sh.cur[b];
    const uint32_t first = n & ~hmask;  // places of the run: [first, n)
    const uint32_t k = first + ((i - first) & smask);
    if (k < n && k < P.cap1) mine[b * P.cap1 + k] = sh.queue[i];
  }
  if (threadIdx.x == 0) sh.sparse_n = 0;
  __syncthreads();
  static_assert(kB1Max == kKeyBlock, "one bucket per thread");
  if (const uint32_t b = threadIdx.x; b < (1u << P.b1bits)) {
    const uint32_t n = sh.cur[b];
    P.cnt1[(static_cast<uint64_t>(blockIdx.x) << P.b1bits) + b] = n;
    if (n > P.cap1) atomicOr(&P.flags[kFlagL1Overflow], 1u);
    if (n) atomicAdd(&sh.sparse_n, n);
  }
  __syncthreads();
  if (threadIdx.x == 0 && sh.sparse_n) atomicAdd(P.entries, static_cast<unsigned long long>(sh.sparse_n));
}

}  // namespace bx
