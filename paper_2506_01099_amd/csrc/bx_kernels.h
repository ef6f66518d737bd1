// HIP kernels of the Benelux-pair search for gfx950.
//
//   k_sieve             Algorithm 1 on LDS tiles, radicals written to HBM (the
//                       searches' sieve is k_sieve_keys, bx_keysieve.h).
//   k_partition         second partition scatter (fan-out B2), XCD-aware.
//   k_join              LDS hash join of one partition: inserts that detect
//                       every earlier equal fingerprint on their probe chain,
//                       as the insert step of Algorithm 3 does, so each pair
//                       of a group of equal sets is reported exactly once.
//   k_verify            every candidate pair recomputed by trial division with
//                       the resident primes (equal fingerprints of different
//                       sets are dropped here), classified (first kind when
//                       rad(m) = rad(n), Algorithm 2) and filtered by kind.
//   k_fill_u32          fills a word array.
//   k_begin             starts a call: clears its counters and writes its query
//                       tables.
#pragma once
#include <type_traits>

#include "bx_device.h"

namespace bx {

// Sparse hits held in LDS per segment of the radical sieve: the 8192 tile has
// about 850 per 2^18 values; of the 2050 of the 2048 tile the excess goes to a
// list in device memory.
constexpr uint32_t kHitCap = 1024;
constexpr int kB1Max = 1024;       // first partition fan-out
constexpr int kB2Max = 2048;       // second partition fan-out
constexpr int kPartChunk = 8192;   // entries per workgroup in k_partition
constexpr uint32_t kKindThird = 4; // kinds bit: also test rad(m + 2) = rad(n + 2)
constexpr int kJoinCap = 8192;     // entries of one LDS join chunk (held in registers)
constexpr int kJoinSlots = 16384;  // LDS hash-table slots (load <= 0.5)
constexpr int kJoinIdxBits = 14;   // slot = tag (18 bits) << 14 | entry index

struct SieveParams {
  const Query* queries;
  const uint64_t* seg_prefix;  // n_queries + 1: first segment of each query
  uint32_t n_queries;
  uint64_t n_segs;
  uint32_t seg_len;
  PowerTables powers;
  uint32_t n_dense;  // powers.pw[0, n_dense) are the dense ones (q <= tile)
  const DenseTab* dense;
  uint64_t* spill;  // per workgroup: spill + blockIdx.x * spill_cap
  uint32_t spill_cap;
  uint32_t* flags;
  uint64_t* rad_out;
  uint64_t rad_lo;  // the first radical's integer
};

template <int T, int BLOCK>
struct SieveSh {
  uint64_t tile[T];
  uint64_t hits[kHitCap];
  uint32_t dres[kDenseMax], doff[kDenseMax], dq[kDenseMax], dtq[kDenseMax];
  uint32_t hit_n;
};

// Counting sort of n staged entries (bucket of entry i in sb[i]) into runs per
// bucket: LDS histogram, one global reservation per non-empty bucket, then the
// runs are written with consecutive threads on consecutive entries (coalesced
// stores).  cnt/gofs hold NB words; perm holds n.  gcur[b] is the cursor of
// bucket b, shared by all workgroups (global, one atomic per non-empty bucket).
// dst(b, k) stores the k-th entry of the bucket (k < cap).
template <int BLOCK, int NB, int NMAX, typename Item, typename Bucket, typename Dst, typename Mid>
__device__ void scatter_runs(uint32_t n, uint32_t nb, const Item* ent, Bucket sb, uint16_t* perm,
                             uint32_t* cnt, uint32_t* gofs, uint32_t* wsum, uint32_t* gcur, uint64_t cap,
                             uint32_t* flag, Dst dst, Mid mid) {
  constexpr int BINS = (NB + BLOCK - 1) / BLOCK;
  // n <= NMAX: each thread takes the U entries tid + u * BLOCK, and every
  // step issues the LDS reads and atomics of all of them before it waits on
  // any (a thread past n reads entry 0 and leaves it alone).
  constexpr int U = (NMAX + BLOCK - 1) / BLOCK;
  const int tid = threadIdx.x;
  for (uint32_t b = tid; b < nb; b += BLOCK) cnt[b] = 0;
  __syncthreads();
  uint32_t bk[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint32_t i = tid + u * BLOCK;
    bk[u] = sb(i < n ? i : 0u);
  }
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (tid + u * BLOCK < n) atomicAdd(&cnt[bk[u]], 1u);
  __syncthreads();
  uint32_t loc[BINS];
  uint32_t sum = 0;
#pragma unroll
  for (int k = 0; k < BINS; ++k) {
    const uint32_t b = tid * BINS + k;
    loc[k] = b < nb ? cnt[b] : 0u;
    sum += loc[k];
  }
  uint32_t tot;
  uint32_t ex = block_exclusive_scan<BLOCK>(sum, wsum, &tot);
#pragma unroll
  for (int k = 0; k < BINS; ++k) {
    const uint32_t b = tid * BINS + k;
    if (b < nb) {
      const uint32_t g = loc[k] ? atomicAdd(&gcur[b], loc[k]) : 0u;
      gofs[b] = g - ex;  // slot j of the sorted order lands at run position g + (j - ex)
      cnt[b] = ex;       // becomes the LDS cursor of bucket b
    }
    ex += loc[k];
  }
  __syncthreads();
  mid();  // the global cursors are taken: work that may overlap the scatter
  uint32_t slot[U];
#pragma unroll
  for (int u = 0; u < U; ++u)
    slot[u] = tid + u * BLOCK < n ? atomicAdd(&cnt[bk[u]], 1u) : 0u;
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (tid + u * BLOCK < n) perm[slot[u]] = static_cast<uint16_t>(tid + u * BLOCK);
  __syncthreads();
  uint32_t pi[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint32_t j = tid + u * BLOCK;
    pi[u] = perm[j < n ? j : 0u];
  }
  uint32_t pb[U];
  Item pe[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    pb[u] = sb(pi[u]);
    pe[u] = ent[pi[u]];
  }
  uint32_t pk[U];
#pragma unroll
  for (int u = 0; u < U; ++u) pk[u] = gofs[pb[u]] + tid + u * BLOCK;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    if (tid + u * BLOCK < n) {
      if (pk[u] < cap)
        dst(pb[u], pk[u], pe[u]);
      else
        atomicOr(flag, 1u);
    }
  }
  __syncthreads();
}

// Orders the LDS accesses of one wave (its lanes read what others of it wrote).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Bound by its writes: 2e8 radicals (1.6 GB) take 0.18 ms without them, and a
// fill alone 0.24.  A thread reads its cells together, and goes on to the next
// tile without a barrier after its writes, which of a large output go past the
// caches (PAST).  With the large tile one workgroup of 1024 threads has a CU to
// itself: two would share it at 64 registers, but then 60 bytes a thread go to
// scratch, and the writes of 2e8 radicals at 2^40 take 0.354 ms instead of
// 0.317, those of 2^28 at 2^32 0.445 instead of 0.394.
// (Segments twice as long, for half the looks at the large powers, measured
// slower; 16-byte writes the same as 8-byte ones.)
template <int T, int BLOCK, bool PAST>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(T >= 8192 ? 4 : 8))) void k_sieve(SieveParams P) {
  static_assert(T % BLOCK == 0 && T <= 65536, "tile shape");
  constexpr int ITER = T / BLOCK;                                     // keys per thread per tile
  constexpr int SLOTS = (dense_slot_cap(T) + BLOCK - 1) / BLOCK;      // dense slots per thread
  static_assert(kDenseMax <= 64 && T / 9 < 1024, "dense slot packing (sdj below)");
  __shared__ SieveSh<T, BLOCK> sh;
  const int tid = threadIdx.x;
  const DenseTab* D = P.dense;
  const uint32_t nd = D->n, nslots = D->nslots;
  for (uint32_t i = tid; i < nd; i += BLOCK) {
    sh.dq[i] = D->q[i];
    sh.dtq[i] = static_cast<uint32_t>(T) % D->q[i];
  }
  // The dense schedule is the same for every tile: each thread keeps its
  // slots (power index, multiple index, q, p, p^-1) in registers.
  // sdj = d | j << 6 | p << 16 (d < kDenseMax = 64, j <= T / 9 < 1024,
  // p <= sqrt(T) < 2^16), packed to leave registers to the tile loop.
  uint32_t sdj[SLOTS], sq[SLOTS], spinv[SLOTS];
#pragma unroll
  for (int k = 0; k < SLOTS; ++k) {
    const uint32_t t = tid + k * BLOCK;
    if (t < nslots) {
      const uint32_t d = D->slot_d[t];
      sdj[k] = d | ((t - D->prefix[d]) << 6) | (D->p[d] << 16);
      sq[k] = D->q[d];
      spinv[k] = D->pinv[d];
    } else {
      sdj[k] = 1u << 16;
      sq[k] = 0;  // no slot
      spinv[k] = 1;
    }
  }
  __syncthreads();
  uint64_t* spill = P.spill + static_cast<uint64_t>(blockIdx.x) * P.spill_cap;

  for (uint64_t s = blockIdx.x; s < P.n_segs; s += gridDim.x) {
    // Segment s -> query q and its x-interval [start, start + len).
    uint32_t lo = 0, hi = P.n_queries;
    while (hi - lo > 1) {
      const uint32_t mid = (lo + hi) >> 1;
      if (P.seg_prefix[mid] <= s)
        lo = mid;
      else
        hi = mid;
    }
    const uint32_t qi = lo;
    const uint64_t qa = P.queries[qi].a, qb = P.queries[qi].b;
    const uint64_t start = qa + (s - P.seg_prefix[qi]) * static_cast<uint64_t>(P.seg_len);
    const uint32_t len = static_cast<uint32_t>(min(static_cast<uint64_t>(P.seg_len), qb - start));
    if (tid == 0) sh.hit_n = 0;
    if (static_cast<uint32_t>(tid) < nd) sh.dres[tid] = static_cast<uint32_t>(start % sh.dq[tid]);
    __syncthreads();

    // Sparse prime powers (q > tile): at most one multiple per tile.  Their
    // multiples in [start, V] are listed once per segment (Algorithm 1's
    // first-multiple offset, -start mod q).
    sparse_hits<BLOCK, 8>(P.powers, P.n_dense, static_cast<double>(start), static_cast<double>(len), tid,
                          [&](uint32_t j, uint32_t p) {
                            const uint32_t k = atomicAdd(&sh.hit_n, 1u);
                            const uint64_t e = (static_cast<uint64_t>(j) << 32) | p;
                            if (k < kHitCap)
                              sh.hits[k] = e;
                            else if (k - kHitCap < P.spill_cap)
                              spill[k - kHitCap] = e;
                            else
                              atomicOr(&P.flags[kFlagSpillOverflow], 1u);
                          });
    __syncthreads();
    const uint32_t nh = min(sh.hit_n, kHitCap + P.spill_cap);

    for (uint32_t base = 0; base < len; base += T) {
      const uint32_t cnt = min(static_cast<uint32_t>(T), len - base);
      const uint64_t x0 = start + base;
      // r[n] <- n with the prime 2 already reduced (count trailing zeros).
      // The whole tile is written (values past cnt are never used).
      if (const uint32_t x0lo = static_cast<uint32_t>(x0);
                 x0lo != 0u && x0lo <= 0xFFFFFFFFu - static_cast<uint32_t>(T)) {
        // Uniform: no x of the tile (x0 .. x0 + T) has a zero low word.
#pragma unroll
        for (int it = 0; it < ITER; ++it) sh.tile[it * BLOCK + tid] = strip_two_lo(x0 + it * BLOCK + tid);
      } else {
#pragma unroll
        for (int it = 0; it < ITER; ++it) sh.tile[it * BLOCK + tid] = strip_two(x0 + it * BLOCK + tid);
      }
      // dres[d] = x0 mod q_d, advanced by T mod q_d from tile to tile.
      if (static_cast<uint32_t>(tid) < nd) {
        const uint32_t qd = sh.dq[tid];
        uint32_t r = sh.dres[tid];
        if (base) {
          r += sh.dtq[tid];
          if (r >= qd) r -= qd;
          sh.dres[tid] = r;
        }
        sh.doff[tid] = r ? qd - r : 0u;
      }
      __syncthreads();
      // Dense odd prime powers: divide r by p at every multiple of q = p^k.
      // (All of a thread's offsets, then all of its cells, are read together.)
      uint32_t pos[SLOTS];
      uint64_t v[SLOTS];
#pragma unroll
      for (int k = 0; k < SLOTS; ++k) pos[k] = sh.doff[sdj[k] & 63u];
#pragma unroll
      for (int k = 0; k < SLOTS; ++k) {
        pos[k] = sq[k] ? pos[k] + ((sdj[k] >> 6) & 1023u) * sq[k] : cnt;
        v[k] = lds_read(&sh.tile[pos[k] < cnt ? pos[k] : 0u]);
      }
#pragma unroll
      for (int k = 0; k < SLOTS; ++k)
        if (pos[k] < cnt) lds_div(&sh.tile[pos[k]], v[k], sdj[k] >> 16, spinv[k]);
      // Sparse hits of this tile: the LDS list, then the rare spill.
      const uint32_t nh_lds = min(nh, kHitCap);
      for (uint32_t h = tid; h < nh_lds; h += BLOCK) {
        const uint64_t e = sh.hits[h];
        const uint32_t pos = static_cast<uint32_t>(e >> 32);
        if (pos - base < cnt) {
          const uint32_t p = static_cast<uint32_t>(e);
          lds_div(&sh.tile[pos - base], p, inv32(p));
        }
      }
      for (uint32_t h = kHitCap + tid; h < nh; h += BLOCK) {
        const uint64_t e = spill[h - kHitCap];
        const uint32_t pos = static_cast<uint32_t>(e >> 32);
        if (pos - base < cnt) {
          const uint32_t p = static_cast<uint32_t>(e);
          lds_div(&sh.tile[pos - base], p, inv32(p));
        }
      }
      __syncthreads();

      // (No barrier after this: a thread writes the same cells again next.)
      uint64_t* out = P.rad_out + (x0 - P.rad_lo) + tid;
      if (cnt == T) {
        uint64_t w[ITER];
#pragma unroll
        for (int it = 0; it < ITER; ++it) w[it] = sh.tile[it * BLOCK + tid];
        if constexpr (PAST) {
#pragma unroll
          for (int it = 0; it < ITER; ++it) __builtin_nontemporal_store(w[it], &out[it * BLOCK]);
        } else {
#pragma unroll
          for (int it = 0; it < ITER; ++it) out[it * BLOCK] = w[it];
        }
      } else {
        for (uint32_t i = tid; i < cnt; i += BLOCK) out[i - tid] = sh.tile[i];
      }
    }
  }
}

// pos43 of an Entry (bx_device.h).
__device__ __forceinline__ uint64_t word_pos43(const WordSource& S, uint32_t w, uint64_t li) {
  uint32_t grp;
  const uint64_t x = word_integer(S, w, li, &grp);
  return S.batch ? ((x - S.queries[grp].a) | (static_cast<uint64_t>(grp) << kGrpShift)) : x;
}

struct PartParams {
  const uint64_t* l1;
  uint64_t cap1;          // words per first-level region
  const uint32_t* cnt1;   // W x B1 region fill counts
  uint32_t W, B1;         // regions per bucket (sieve workgroups), buckets
  uint32_t first;  // first first-level bucket of this group
  uint32_t G;      // buckets in the group: 1, 2, 4 or 8
  uint32_t chunks_per_region;
  Entry* l2;       // group buffer: G x B2 sub-buckets of cap2 entries
  uint32_t cap2;
  uint32_t* cnt2;  // G x B2 cursors (zero on entry)
  uint32_t b2bits;  // second-level partition = top b2bits of the fingerprint
  uint64_t fp_mask;          // fingerprint bits kept (all 53 but in tests of the verification)
  uint32_t* flags;
  WordSource src;
  uint64_t kl_mask;  // fingerprint bits above a word's index
  // Compact second level: one 64-bit word per entry, fp_low << wl_bits |
  // w << li_bits | li: the first-level word's index with its region.  The top
  // of the fingerprint is the partition's own index.
  uint64_t* l2c;
  uint32_t wl_bits;
  uint64_t low_mask;  // fingerprint bits a compact word keeps
};

// Second scatter of one group of first-level buckets into the group buffer.
// Persistent: workgroup l runs on XCD l mod 8 (round-robin dispatch) and
// serves bucket (l mod 8) mod G, so with G = 8 a bucket never leaves its XCD
// and the partial lines of its sub-buckets are completed in that XCD's L2
// before they are written back.  The bucket's chunks are split into nbw
// contiguous ranges, one per workgroup; the next chunk is loaded into
// registers while the current one is scattered.  Bound by memory: 8 bytes read
// and 8 written per entry, at 3.2 to 3.6 TB/s (by the distance of the partitions
// in memory) of the 4.4 a large copy takes on this card (2^36: 36 to 42 ms, by
// process, -> 33 to 37 with 8-byte words read instead of 12-byte entries).
template <int BLOCK, bool COMPACT>
__global__ __launch_bounds__(BLOCK) void k_partition(PartParams P) {
  constexpr int EPT = kPartChunk / BLOCK;
  static_assert(kPartChunk % BLOCK == 0, "chunk shape");
  using Item = typename std::conditional<COMPACT, uint64_t, Entry>::type;  // what the chunk stages
  __shared__ Item ent[kPartChunk];
  __shared__ uint16_t sbk[kPartChunk], perm[kPartChunk];
  __shared__ uint32_t cnt[kB2Max], gofs[kB2Max];
  __shared__ uint32_t wsum[BLOCK / 64];
  note_time(P.flags, K_PART);
  const int tid = threadIdx.x;
  const uint32_t l = blockIdx.x;
  const uint32_t xcd = l & 7u, slot = l >> 3;
  const uint32_t per = 8u / P.G;
  const uint32_t gb = xcd % P.G;
  const uint32_t k = slot * per + xcd / P.G;  // index among the bucket's nbw workgroups
  const uint32_t nbw = (gridDim.x >> 3) * per;
  const uint32_t b1 = P.first + gb;
  const uint32_t B2 = 1u << P.b2bits;
  const uint32_t cpr = P.chunks_per_region;
  const uint64_t n_chunks = static_cast<uint64_t>(P.W) * cpr;
  const uint64_t c_begin = n_chunks * k / nbw, c_end = n_chunks * (k + 1) / nbw;
  Entry* out = P.l2 + static_cast<uint64_t>(gb) * B2 * P.cap2;
  uint64_t* outc = P.l2c + static_cast<uint64_t>(gb) * B2 * P.cap2;
  uint32_t* gcur = P.cnt2 + static_cast<uint64_t>(gb) * B2;
  const uint32_t cap2 = P.cap2;
  // The partition of an entry is the top of its fingerprint.
  auto bucket_of = [&](uint32_t i) -> uint32_t { return sbk[i]; };
  // Chunk ci of the bucket: entries [s0, s0 + n) of region ci / cpr.
  auto chunk = [&](uint64_t ci, const uint64_t** src) -> uint32_t {  // ci < n_chunks
    const uint64_t region = (ci / cpr) * P.B1 + b1;
    const uint64_t n1 = min(static_cast<uint64_t>(P.cnt1[region]), P.cap1);
    const uint64_t s0 = (ci % cpr) * static_cast<uint64_t>(kPartChunk);
    *src = P.l1 + region * P.cap1 + s0;
    return s0 >= n1 ? 0u : static_cast<uint32_t>(min(static_cast<uint64_t>(kPartChunk), n1 - s0));
  };
  uint64_t e[EPT];
  const uint64_t* src;
  uint32_t n = c_begin < c_end ? chunk(c_begin, &src) : 0u;
#pragma unroll
  for (int q = 0; q < EPT; ++q) {
    const uint32_t i = tid + q * BLOCK;
    if (i < n) e[q] = src[i];
  }
  for (uint64_t ci = c_begin; ci < c_end; ++ci) {
    const uint32_t w = static_cast<uint32_t>(ci / cpr);  // the chunk's region
    const uint64_t wl = static_cast<uint64_t>(w) << P.src.li_bits, li_mask = (1ull << P.src.li_bits) - 1;
#pragma unroll
    for (int q = 0; q < EPT; ++q) {
      const uint32_t i = tid + q * BLOCK;
      if (i < n) {
        const uint64_t x = e[q], li = x & li_mask, low = (x >> P.src.li_bits) & P.kl_mask;
        if constexpr (COMPACT)
          ent[i] = ((low & P.low_mask) << P.wl_bits) | wl | li;
        else
          ent[i] = make_entry(word_pos43(P.src, w, li), (((x >> 53) << 42) | low) & P.fp_mask);
        sbk[i] = static_cast<uint16_t>(x >> 53 >> (11 - P.b2bits));
      }
    }
    const uint32_t n_cur = n;
    n = ci + 1 < c_end ? chunk(ci + 1, &src) : 0u;
    // Issued after the global cursor atomics, whose returns would otherwise
    // wait for these loads as well.
    auto prefetch = [&] {
#pragma unroll
      for (int q = 0; q < EPT; ++q) {
        const uint32_t i = tid + q * BLOCK;
        if (i < n) e[q] = src[i];
      }
    };
    __syncthreads();
    if (n_cur)  // uniform over the workgroup
      scatter_runs<BLOCK, kB2Max, kPartChunk>(
          n_cur, B2, ent, bucket_of, perm, cnt, gofs, wsum, gcur, cap2, &P.flags[kFlagL2Overflow],
          [=](uint32_t b, uint32_t kk, const Item& x) {
            if constexpr (COMPACT)
              outc[static_cast<uint64_t>(b) * cap2 + kk] = x;
            else
              out[static_cast<uint64_t>(b) * cap2 + kk] = x;
          },
          prefetch);
    else
      prefetch();
  }
}

struct JoinParams {
  const Entry* l2;
  uint32_t cap2;
  uint32_t* cnt2;
  uint64_t n_sub;
  uint32_t gmask;
  Cand* cand;
  uint32_t cand_cap;
  uint32_t* flags;
  unsigned long long* joined;  // entries read, summed over partitions (64-bit: 2^36 searches pass 2^32)
  // Compact second level (k_join_c).
  const uint64_t* l2c;
  uint32_t wl_bits;
  uint64_t low_mask;
  WordSource src;
  // First-level buckets joined as they are (k_join_c<DIRECT>): the regions.
  const uint64_t* l1;
  uint64_t cap1;
  const uint32_t* cnt1;  // W x B1
  uint64_t kl_mask;
  const uint32_t* primes;  // 2, 3, 5, ...
  const PrimeInv* pinv;
  uint32_t n_primes;
  bool screen;  // k_join, k_join_sort: look at equal entries' integers first
};

__device__ __forceinline__ void emit_cand(const JoinParams& P, const Entry& a, const Entry& b) {
  const uint32_t k = atomicAdd(&P.flags[kFlagCand], 1u);
  if (k < P.cand_cap) {
    Cand c;
    c.a = a;
    c.b = b;
    P.cand[k] = c;
  }
}

// Whether S_x = S_y can hold, from the primes 3 .. 313, by one lane.  A prime
// that divides one of x, x + 1 has to divide the same one of y, y + 1 when x
// and y have the same parity (a pair of the first kind), and the other one else
// (the second kind; the prime 2 tells).  About one in 390 pairs of different
// sets passes.
__device__ __forceinline__ bool small_primes_agree(const JoinParams& P, uint64_t x, uint64_t y) {
  const bool cross = (x ^ y) & 1;
  const uint32_t n = min(P.n_primes, 65u);
  for (uint32_t i = 1; i < n; ++i) {
    const PrimeInv v = P.pinv[i];
    const bool a0 = x * v.inv <= v.lim, a1 = (x + 1) * v.inv <= v.lim;
    const bool b0 = y * v.inv <= v.lim, b1 = (y + 1) * v.inv <= v.lim;
    if (cross ? a0 != b1 || a1 != b0 : a0 != b0 || a1 != b1) return false;
  }
  return true;
}

// A candidate of k_join or k_join_sort.  The first level's words hold 35 of the
// fingerprint's 53 bits at 2^36, of which 1.5e6 pairs of different sets share
// all (the candidate buffer takes 2^20): with `screen` the divisibility of both
// integers by small primes has to agree as a pair's does.
__device__ __forceinline__ void emit_equal(const JoinParams& P, const Entry& a, const Entry& b) {
  if (P.screen) {
    const uint64_t off = P.src.batch ? P.src.queries[entry_grp(a, P.gmask)].a : 0ull;
    if (!small_primes_agree(P, entry_pos(a, P.src.batch) + off, entry_pos(b, P.src.batch) + off)) return;
  }
  emit_cand(P, a, b);
}

// LDS hash join of one second-level partition.  Each insert walks its probe
// chain to the first empty slot and compares the key with every occupied slot
// on the way (Algorithm 3's insert step).  Two equal keys follow the same
// chain, so the one that claims the later slot passes the other and reports
// the pair; every pair of a group is reported once.  A slot holds an 18-bit
// tag of the key hash and the entry's index; the entries themselves stay in
// registers (EPT per thread), and the rare tag match re-reads the other entry
// from the partition (L2-resident).  Partitions larger than one chunk are
// joined chunk by chunk: after chunk c is inserted, every later entry probes
// it, walking to an empty slot as the probe step does.
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(8))) void k_join(JoinParams P) {
  constexpr int EPT = kJoinCap / BLOCK;
  constexpr uint32_t kEmpty = 0xFFFFFFFFu;
  constexpr uint32_t kIdxMask = (1u << kJoinIdxBits) - 1;
  static_assert(kJoinCap < (1 << kJoinIdxBits), "index field must not reach the empty marker");
  __shared__ __align__(16) uint32_t table[kJoinSlots];
  const int tid = threadIdx.x;
  note_time(P.flags, K_JOIN);
  const uint64_t sbk = blockIdx.x;
  if (sbk >= P.n_sub) return;
  const uint32_t n = min(P.cnt2[sbk], P.cap2);
  __syncthreads();
  // This workgroup is the only reader of the cursor: clear it for the next group.
  if (tid == 0) {
    P.cnt2[sbk] = 0;
    if (n) atomicAdd(P.joined, static_cast<unsigned long long>(n));
  }
  if (n < 2) return;
  const Entry* src = P.l2 + sbk * P.cap2;
  for (uint32_t i0 = 0; i0 < n; i0 += kJoinCap) {
    const uint32_t m = min(static_cast<uint32_t>(kJoinCap), n - i0);
    // Table of at least twice the chunk's entries (load <= 0.5), power of two.
    uint32_t slots = 1024;
    while (slots < 2 * m && slots < static_cast<uint32_t>(kJoinSlots)) slots <<= 1;
    const uint32_t smask = slots - 1;
    // Every thread loads all its entries at once: lanes past the chunk load
    // entry 0 instead (m >= 2), so that no load waits behind a masked one.
    Entry e[EPT];
#pragma unroll
    for (int k = 0; k < EPT; ++k) {
      const uint32_t i = tid + k * BLOCK;
      e[k] = src[i0 + (i < m ? i : 0u)];
    }
    // Cleared four slots per store (slots is a multiple of 1024).
    for (uint32_t s = 4 * tid; s < slots; s += 4 * BLOCK)
      *reinterpret_cast<uint4*>(&table[s]) = make_uint4(kEmpty, kEmpty, kEmpty, kEmpty);
    __syncthreads();
    // Every entry first tries to claim its home slot; the EPT claims of a
    // thread are independent and issued together (at load <= 0.5 most
    // succeed).  A claim that finds the slot taken compares the tag and walks
    // on, claiming each next slot, until one is empty.
    // (In groups of four, to stay within the registers of 32 waves per CU.)
    constexpr int kClaim = EPT < 4 ? EPT : 4;
    static_assert(EPT % kClaim == 0, "claim groups");
#pragma unroll
    for (int k0 = 0; k0 < EPT; k0 += kClaim) {
      uint32_t got[kClaim];
#pragma unroll
      for (int u = 0; u < kClaim; ++u) {
        const uint32_t i = tid + (k0 + u) * BLOCK;
        const uint32_t h = static_cast<uint32_t>(entry_fp(e[k0 + u]));
        got[u] = i < m ? atomicCAS(&table[h & smask], kEmpty, (h & ~kIdxMask) | i) : kEmpty;
      }
#pragma unroll
      for (int u = 0; u < kClaim; ++u) {
        if (got[u] == kEmpty) continue;  // claimed (or no entry)
        const int k = k0 + u;
        const uint64_t fk = entry_fp(e[k]);
        const uint32_t gk = entry_grp(e[k], P.gmask);
        const uint32_t h = static_cast<uint32_t>(fk);
        const uint32_t mine = (h & ~kIdxMask) | (tid + k * BLOCK);
        uint32_t v = got[u], s = h & smask;
        for (;;) {
          if (((v ^ mine) & ~kIdxMask) == 0) {
            const Entry f = src[i0 + (v & kIdxMask)];
            if (entry_fp(f) == fk && entry_grp(f, P.gmask) == gk) emit_equal(P, e[k], f);
          }
          s = (s + 1) & smask;
          v = atomicCAS(&table[s], kEmpty, mine);
          if (v == kEmpty) break;
        }
      }
    }
    __syncthreads();
    for (uint32_t jj = i0 + m + tid; jj < n; jj += BLOCK) {
      const Entry g = src[jj];
      const uint64_t fk = entry_fp(g);
      const uint32_t gk = entry_grp(g, P.gmask);
      const uint32_t h = static_cast<uint32_t>(fk);
      uint32_t s = h & smask;
      for (;;) {
        const uint32_t v = table[s];
        if (v == kEmpty) break;
        if (((v ^ h) & ~kIdxMask) == 0) {
          const Entry f = src[i0 + (v & kIdxMask)];
          if (entry_fp(f) == fk && entry_grp(f, P.gmask) == gk) emit_equal(P, g, f);
        }
        s = (s + 1) & smask;
      }
    }
    __syncthreads();
  }
}

// Two compact words whose kept fingerprint bits met.
struct WordMatch {
  uint64_t a, b;
};
// Listed per chunk of a partition, in LDS.  Full partitions (7400 words) of one
// range expect 2 meetings at 2^36 and, with the 19 fingerprint bits left beside
// the index, 52 just below 2^42; fewer kept bits or larger partitions, which
// only options ask for, pass the list (k_join_c).
constexpr uint32_t kMatchMax = 128;

// The integers of a match; false if they belong to different queries.
struct MatchPair {
  uint64_t x, y;
  uint32_t grp;
};
__device__ __forceinline__ bool match_pair(const WordSource& S, uint32_t wl_bits, uint64_t a, uint64_t b, MatchPair* r) {
  const uint64_t wl_mask = (1ull << wl_bits) - 1, li_mask = (1ull << S.li_bits) - 1;
  uint32_t gb;
  r->x = word_integer(S, static_cast<uint32_t>((a & wl_mask) >> S.li_bits), a & li_mask, &r->grp);
  r->y = word_integer(S, static_cast<uint32_t>((b & wl_mask) >> S.li_bits), b & li_mask, &gb);
  return r->grp == gb;
}

__device__ __forceinline__ void emit_match(const JoinParams& P, uint64_t a, uint64_t b, const MatchPair& r) {
  const uint64_t off = P.src.batch ? P.src.queries[r.grp].a : 0ull, grp = static_cast<uint64_t>(r.grp) << kGrpShift;
  emit_cand(P, make_entry((r.x - off) | grp, a >> P.wl_bits), make_entry((r.y - off) | grp, b >> P.wl_bits));
}

// The same by one wave, from the primes 3 .. 2^11 and some more, one per lane.
// Different sets seldom pass the first 64.
__device__ __forceinline__ bool may_be_equal(const JoinParams& P, uint64_t x, uint64_t y) {
  const bool cross = (x ^ y) & 1;
  for (uint32_t i0 = 1; i0 < P.n_primes; i0 += 256) {
    PrimeInv v[4];  // four rounds read together
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const uint32_t i = i0 + 64 * u + lane_id();
      v[u] = P.pinv[i < P.n_primes ? i : P.n_primes - 1];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const bool a0 = x * v[u].inv <= v[u].lim, a1 = (x + 1) * v[u].inv <= v[u].lim;
      const bool b0 = y * v[u].inv <= v[u].lim, b1 = (y + 1) * v[u].inv <= v[u].lim;
      if (__any(cross ? a0 != b1 || a1 != b0 : a0 != b0 || a1 != b1)) return false;
    }
    if (P.primes[i0] >= (1u << 11)) break;
  }
  return true;
}

// k_join over compact words: the same inserts and probes, on the kept low
// fingerprint bits (the partition fixes the top ones).  Matches are listed, and
// at the end of a chunk each is looked at by one wave: its integers are taken
// from the words themselves, different queries and sets that a small prime
// tells apart are dropped, and the rest are candidates.  (The look takes a lane
// that found it 0.5 ms for an equal pair, a wave about a microsecond.)  A chunk
// with more matches than the list holds walks its chains once more instead, and
// the lane that finds a match looks at it, by fewer primes (small_primes_agree):
// 3e6 matches are more than the candidate buffer holds.
//
// DIRECT: of a short range the first level's buckets are the partitions, and
// the workgroup gathers its bucket's words from the regions into LDS (2^20
// integers: a partition launch of 15 us less).
//
// Bound by memory and LDS round trips: 58 GB of words at 3.0 to 3.2 TB/s at 2^36.
template <int BLOCK, bool DIRECT>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(DIRECT ? 4 : 8))) void k_join_c(JoinParams P) {
  constexpr int EPT = kJoinCap / BLOCK;
  constexpr uint32_t kEmpty = 0xFFFFFFFFu;
  constexpr uint32_t kIdxMask = (1u << kJoinIdxBits) - 1;
  static_assert(kJoinCap < (1 << kJoinIdxBits), "index field must not reach the empty marker");
  __shared__ __align__(16) uint32_t table[kJoinSlots];
  __shared__ uint32_t matches;  // words of this partition whose kept bits met
  __shared__ WordMatch match[kMatchMax];
  __shared__ uint64_t gathered[DIRECT ? kJoinCap : 1];
  __shared__ uint32_t wsum[BLOCK / 64];
  const int tid = threadIdx.x;
  note_time(P.flags, K_JOIN);
  const uint64_t sbk = blockIdx.x;
  if (sbk >= P.n_sub) return;
  uint32_t n;
  const uint64_t* src;
  if constexpr (DIRECT) {
    // Four threads per region, BLOCK / 4 regions at a time (n_sub = B1).
    n = 0;
    for (uint32_t w0 = 0; w0 < P.src.W; w0 += BLOCK / 4) {
      const uint32_t w = w0 + (static_cast<uint32_t>(tid) >> 2), k0 = tid & 3u;
      const uint64_t region = static_cast<uint64_t>(w) * P.n_sub + sbk;
      const uint32_t c = w < P.src.W ? min(P.cnt1[region], static_cast<uint32_t>(P.cap1)) : 0u;
      uint32_t sum;
      const uint32_t at = n + block_exclusive_scan<BLOCK>(k0 == 0 ? c : 0u, wsum, &sum) - (k0 == 0 ? 0u : c);
      const uint64_t wl = static_cast<uint64_t>(w) << P.src.li_bits, li_mask = (1ull << P.src.li_bits) - 1;
      for (uint32_t k = k0; k < c; k += 4) {
        const uint64_t x = P.l1[region * P.cap1 + k];
        if (at + k < static_cast<uint32_t>(kJoinCap))
          gathered[at + k] = ((((x >> P.src.li_bits) & P.kl_mask) & P.low_mask) << P.wl_bits) | wl | (x & li_mask);
      }
      n += sum;
      __syncthreads();
    }
    if (n > static_cast<uint32_t>(kJoinCap)) {  // the pass is split
      if (tid == 0) atomicOr(&P.flags[kFlagL2Overflow], 1u);
      return;
    }
    src = gathered;
    if (tid == 0 && n) atomicAdd(P.joined, static_cast<unsigned long long>(n));
  } else {
    n = min(P.cnt2[sbk], P.cap2);
    src = P.l2c + sbk * P.cap2;
    __syncthreads();
    if (tid == 0) {
      P.cnt2[sbk] = 0;
      if (n) atomicAdd(P.joined, static_cast<unsigned long long>(n));
    }
  }
  if (n < 2) return;
  const uint32_t pb = P.wl_bits;
  if (tid == 0) matches = 0;  // (barriers follow before the first match)
  auto emit = [&](uint64_t a, uint64_t b) {
    const uint32_t k = atomicAdd(&matches, 1u);
    if (k < kMatchMax) match[k] = WordMatch{a, b};
  };
  for (uint32_t i0 = 0; i0 < n; i0 += kJoinCap) {
    const uint32_t m = min(static_cast<uint32_t>(kJoinCap), n - i0);
    uint32_t slots = 1024;
    while (slots < 2 * m && slots < static_cast<uint32_t>(kJoinSlots)) slots <<= 1;
    const uint32_t smask = slots - 1;
    uint64_t e[EPT];
#pragma unroll
    for (int k = 0; k < EPT; ++k) {
      const uint32_t i = tid + k * BLOCK;
      e[k] = src[i0 + (i < m ? i : 0u)];
    }
    for (uint32_t s = 4 * tid; s < slots; s += 4 * BLOCK)
      *reinterpret_cast<uint4*>(&table[s]) = make_uint4(kEmpty, kEmpty, kEmpty, kEmpty);
    __syncthreads();
    constexpr int kClaim = EPT < 4 ? EPT : 4;
    static_assert(EPT % kClaim == 0, "claim groups");
#pragma unroll
    for (int k0 = 0; k0 < EPT; k0 += kClaim) {
      uint32_t got[kClaim];
#pragma unroll
      for (int u = 0; u < kClaim; ++u) {
        const uint32_t i = tid + (k0 + u) * BLOCK;
        const uint32_t h = static_cast<uint32_t>(e[k0 + u] >> pb);
        got[u] = i < m ? atomicCAS(&table[h & smask], kEmpty, (h & ~kIdxMask) | i) : kEmpty;
      }
#pragma unroll
      for (int u = 0; u < kClaim; ++u) {
        if (got[u] == kEmpty) continue;
        const int k = k0 + u;
        const uint64_t fk = e[k] >> pb;
        const uint32_t h = static_cast<uint32_t>(fk);
        const uint32_t mine = (h & ~kIdxMask) | (tid + k * BLOCK);
        uint32_t v = got[u], s = h & smask;
        for (;;) {
          if (((v ^ mine) & ~kIdxMask) == 0) {
            const uint64_t f = src[i0 + (v & kIdxMask)];
            if ((f >> pb) == fk) emit(e[k], f);
          }
          s = (s + 1) & smask;
          v = atomicCAS(&table[s], kEmpty, mine);
          if (v == kEmpty) break;
        }
      }
    }
    __syncthreads();
    for (uint32_t jj = i0 + m + tid; jj < n; jj += BLOCK) {
      const uint64_t g = src[jj];
      const uint64_t fk = g >> pb;
      const uint32_t h = static_cast<uint32_t>(fk);
      uint32_t s = h & smask;
      for (;;) {
        const uint32_t v = table[s];
        if (v == kEmpty) break;
        if (((v ^ h) & ~kIdxMask) == 0) {
          const uint64_t f = src[i0 + (v & kIdxMask)];
          if ((f >> pb) == fk) emit(g, f);
        }
        s = (s + 1) & smask;
      }
    }
    __syncthreads();
    const uint32_t met = matches;
    if (met == 0) continue;  // uniform
    if (met <= kMatchMax) {
      for (uint32_t k = tid >> 6; k < met; k += BLOCK / 64) {  // uniform over a wave
        const WordMatch w = match[k];
        MatchPair r;
        if (match_pair(P.src, pb, w.a, w.b, &r) && may_be_equal(P, r.x, r.y) && lane_id() == 0) emit_match(P, w.a, w.b, r);
      }
    } else {
      // Each entry of the chunk against those before it, each later one against all.
      for (uint32_t i = i0 + tid; i < n; i += BLOCK) {
        const uint64_t g = src[i];
        const uint32_t h = static_cast<uint32_t>(g >> pb);
        uint32_t s = h & smask;
        for (uint32_t v = table[s]; v != kEmpty; s = (s + 1) & smask, v = table[s]) {
          const uint32_t o = i0 + (v & kIdxMask);
          if (((v ^ h) & ~kIdxMask) != 0 || o >= i) continue;
          const uint64_t f = src[o];
          MatchPair r;
          if ((f >> pb) == (g >> pb) && match_pair(P.src, pb, g, f, &r) && small_primes_agree(P, r.x, r.y)) emit_match(P, g, f, r);
        }
      }
    }
    __syncthreads();
    if (tid == 0) {
      atomicAdd(&P.flags[kFlagWordMatch], met);
      matches = 0;
    }
    __syncthreads();
  }
}

// Sort join of one second-level partition, the ablation of the LDS hash join:
// Algorithm 2 (sort, then compare neighbours) applied per partition, with every
// pair of a run of equal keys reported rather than adjacent ones only.  The low
// 32 bits of each fingerprint, packed with the entry's index, are bitonic-
// sorted in LDS; runs of equal words are compared on the full fingerprint and
// query.  A partition larger than one LDS chunk is joined chunk by chunk: every
// later entry binary-searches each sorted chunk.
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_join_sort(JoinParams P) {
  constexpr int kIdx = 13;  // index bits (kJoinCap = 8192)
  static_assert(kJoinCap <= (1 << kIdx), "index field");
  __shared__ uint64_t key[kJoinCap];
  const int tid = threadIdx.x;
  note_time(P.flags, K_JOIN);
  const uint64_t sbk = blockIdx.x;
  if (sbk >= P.n_sub) return;
  const uint32_t n = min(P.cnt2[sbk], P.cap2);
  __syncthreads();
  // This workgroup is the only reader of the cursor: clear it for the next group.
  if (tid == 0) {
    P.cnt2[sbk] = 0;
    if (n) atomicAdd(P.joined, static_cast<unsigned long long>(n));
  }
  if (n < 2) return;
  const Entry* src = P.l2 + sbk * P.cap2;
  auto same = [&](const Entry& a, const Entry& b) {
    return entry_fp(a) == entry_fp(b) && entry_grp(a, P.gmask) == entry_grp(b, P.gmask);
  };
  for (uint32_t i0 = 0; i0 < n; i0 += kJoinCap) {
    const uint32_t m = min(static_cast<uint32_t>(kJoinCap), n - i0);
    uint32_t npad = 2;
    while (npad < m) npad <<= 1;
    for (uint32_t i = tid; i < npad; i += BLOCK)
      key[i] = i < m ? (static_cast<uint64_t>(static_cast<uint32_t>(entry_fp(src[i0 + i]))) << kIdx) | i : ~0ull;
    __syncthreads();
    for (uint32_t k = 2; k <= npad; k <<= 1) {
      for (uint32_t j = k >> 1; j > 0; j >>= 1) {
        for (uint32_t t = tid; t < npad / 2; t += BLOCK) {
          const uint32_t i = ((t & ~(j - 1)) << 1) | (t & (j - 1)), l = i | j;
          const uint64_t a = key[i], b = key[l];
          if ((a > b) == ((i & k) == 0)) {
            key[i] = b;
            key[l] = a;
          }
        }
        __syncthreads();
      }
    }
    // Runs of equal 32-bit fingerprint words inside the chunk: the thread at a
    // run's first element compares every pair of the run in full.
    for (uint32_t i = tid; i + 1 < m; i += BLOCK) {
      const uint64_t h = key[i] >> kIdx;
      if ((i > 0 && (key[i - 1] >> kIdx) == h) || (key[i + 1] >> kIdx) != h) continue;
      uint32_t end = i + 1;
      while (end < m && (key[end] >> kIdx) == h) ++end;
      for (uint32_t a = i; a < end; ++a) {
        const Entry ea = src[i0 + static_cast<uint32_t>(key[a] & ((1u << kIdx) - 1))];
        for (uint32_t b = a + 1; b < end; ++b) {
          const Entry eb = src[i0 + static_cast<uint32_t>(key[b] & ((1u << kIdx) - 1))];
          if (same(ea, eb)) emit_equal(P, ea, eb);
        }
      }
    }
    // Every later entry searches this sorted chunk.
    for (uint32_t jj = i0 + m + tid; jj < n; jj += BLOCK) {
      const Entry g = src[jj];
      const uint64_t h = static_cast<uint32_t>(entry_fp(g));
      uint32_t lo = 0, hi = m;  // first word with key >> kIdx >= h
      while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if ((key[mid] >> kIdx) < h)
          lo = mid + 1;
        else
          hi = mid;
      }
      for (uint32_t a = lo; a < m && (key[a] >> kIdx) == h; ++a) {
        const Entry f = src[i0 + static_cast<uint32_t>(key[a] & ((1u << kIdx) - 1))];
        if (same(g, f)) emit_equal(P, g, f);
      }
    }
    __syncthreads();
  }
}

struct VerifyParams {
  const Cand* cand;
  const uint32_t* n_cand;  // candidate count, read on the device (graph replays)
  uint32_t cand_cap;
  const uint32_t* primes;  // all primes <= sqrt(hi_max), ascending
  const PrimeInv* pinv;    // their inverses for the divisibility tests
  uint32_t n_primes;
  const Query* queries;
  int batch;
  uint32_t kinds;
  uint32_t third_off;  // the third condition compares rad(m + third_off), rad(n + third_off) (2 in use)
  uint64_t fp_mask;  // fingerprint bits every candidate's entries hold
  uint64_t whole_mask;  // those the call keeps
  int compact;       // entries hold fewer than that
  OutPair* out;
  uint32_t out_cap;
  uint32_t* flags;
  Report* report;  // host memory
};

// The last workgroup of the verification to finish writes the report, and
// readies the flags for the candidates of another pass.
template <int BLOCK>
__device__ __forceinline__ void report(const VerifyParams& P, uint32_t active) {
  __shared__ uint32_t last;
  __syncthreads();
  if (threadIdx.x == 0) {
    __threadfence();
    last = atomicAdd(&P.flags[kFlagDone], 1u) + 1 == active;
    __threadfence();
  }
  __syncthreads();
  if (!last) return;
  static_assert(BLOCK >= static_cast<int>(kReportPairs), "one pair per thread");
  const volatile uint32_t* flags = P.flags;
  Counters* n = reinterpret_cast<Counters*>(P.flags);
  const uint32_t pairs = min(flags[kFlagOut], min(P.out_cap, kReportPairs));
  if (threadIdx.x < 16) P.report->n.flags[threadIdx.x] = flags[threadIdx.x];
  if (threadIdx.x < kAccCount) P.report->n.acc[threadIdx.x] = *(const volatile unsigned long long*)&n->acc[threadIdx.x];
  if (threadIdx.x < kKernels) {
    unsigned long long t = *(const volatile unsigned long long*)&n->ticks[threadIdx.x];
    if (threadIdx.x == K_VERIFY) {  // up to here
      t += wall_clock64() - *(const volatile unsigned long long*)&n->since;
      n->ticks[K_VERIFY] = t;
      n->running = 0;
    }
    P.report->n.ticks[threadIdx.x] = t;
  }
  if (threadIdx.x < pairs) P.report->pairs[threadIdx.x] = P.out[threadIdx.x];
  __syncthreads();
  if (threadIdx.x == 0) P.flags[kFlagCand] = P.flags[kFlagDone] = 0;
}

// value's word in lane l (the same in every lane).
__device__ __forceinline__ uint64_t read_lane64(uint64_t value, int l) {
  const uint32_t lo = __builtin_amdgcn_readlane(static_cast<uint32_t>(value), l);
  const uint32_t hi = __builtin_amdgcn_readlane(static_cast<uint32_t>(value >> 32), l);
  return (static_cast<uint64_t>(hi) << 32) | lo;
}

// One workgroup per candidate pair: rad of m, m+1, n, n+1 by trial division
// (the definition of the radical), with the cofactor left after dividing out
// every prime <= sqrt(v) being 1 or one more prime.
//
// Bound by latency, a few pairs a call: at most 15 primes divide a value, so a
// wave multiplies the few lanes that hold one in turn, and the values' last
// divisions run side by side.  Ten pairs of 3000000 or fewer: 9 -> 6 us
// (a tree over LDS with eight barriers, four divisions in a row).
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_verify(VerifyParams P) {
  constexpr int NV = 6;  // m, m+1, n, n+1 and, for the third condition, m+d, n+d (d = 2)
  __shared__ uint64_t red_r[NV][BLOCK / 64], red_s[NV][BLOCK / 64], rad[NV];
  const int tid = threadIdx.x;
  note_time(P.flags, K_VERIFY);
  const uint32_t n_cand = min(*P.n_cand, P.cand_cap);
  const uint32_t active = max(1u, min(n_cand, gridDim.x));  // workgroups with candidates, or the first
  if (blockIdx.x >= active) return;
  const bool third = (P.kinds & kKindThird) != 0;
  const int nv = third ? NV : 4;
  for (uint32_t c = blockIdx.x; c < n_cand; c += gridDim.x) {
    __syncthreads();
    const Cand cd = P.cand[c];
    const uint32_t qa_idx = entry_grp(cd.a, P.batch ? kGrpMask : 0u);
    const uint64_t off = P.batch ? P.queries[qa_idx].a : 0ull;
    const uint64_t xa = entry_pos(cd.a, P.batch) + off, xb = entry_pos(cd.b, P.batch) + off;
    const uint64_t m = xa < xb ? xa : xb, n = xa < xb ? xb : xa;
    const uint64_t d = P.third_off;
    const uint64_t v[NV] = {m, m + 1, n, n + 1, m + d, n + d};
    const uint64_t vmax = third && d > 1 ? n + d : n + 1;
    uint64_t pr[NV] = {1, 1, 1, 1, 1, 1}, sm[NV] = {1, 1, 1, 1, 1, 1};
    for (uint32_t i = tid; i < P.n_primes; i += BLOCK) {
      const uint64_t p = P.primes[i];
      if (p * p > vmax) break;
      if (p == 2) {
#pragma unroll
        for (int k = 0; k < NV; ++k) {
          if (k < nv && 4 <= v[k] && (v[k] & 1) == 0) {
            pr[k] *= 2;
            sm[k] <<= __builtin_ctzll(v[k]);
          }
        }
        continue;
      }
      // An odd p divides t iff t * p^-1 (mod 2^64) <= floor((2^64 - 1) / p),
      // and that product is then t / p.
      const PrimeInv pi = P.pinv[i];
#pragma unroll
      for (int k = 0; k < NV; ++k) {
        uint64_t t = v[k] * pi.inv;
        if (k < nv && p * p <= v[k] && t <= pi.lim) {
          pr[k] *= p;
          uint64_t pk = p;
          for (uint64_t u = t * pi.inv; u <= pi.lim; u *= pi.inv) pk *= p;
          sm[k] *= pk;
        }
      }
    }
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      uint64_t r = 1, sq = 1;  // of the wave
      for (uint64_t m_hit = __ballot(pr[k] != 1); m_hit; m_hit &= m_hit - 1) {
        const int l = __builtin_ctzll(m_hit);
        r *= read_lane64(pr[k], l);
        sq *= read_lane64(sm[k], l);
      }
      if ((tid & 63) == 0) {
        red_r[k][tid >> 6] = r;
        red_s[k][tid >> 6] = sq;
      }
    }
    __syncthreads();
    if (tid < NV) {
      uint64_t r = red_r[tid][0], sq = red_s[tid][0];
      for (int w = 1; w < BLOCK / 64; ++w) {
        r *= red_r[tid][w];
        sq *= red_s[tid][w];
      }
      const uint64_t cof = (tid == 0 ? v[0] : tid == 1 ? v[1] : tid == 2 ? v[2] : tid == 3 ? v[3] : tid == 4 ? v[4] : v[5]) / sq;
      rad[tid] = r * (cof > 1 ? cof : 1);
    }
    __syncthreads();
    if (tid == 0) {
      const uint64_t lo_m = rad[0] < rad[1] ? rad[0] : rad[1], hi_m = rad[0] < rad[1] ? rad[1] : rad[0];
      const uint64_t lo_n = rad[2] < rad[3] ? rad[2] : rad[3], hi_n = rad[2] < rad[3] ? rad[3] : rad[2];
      const bool same = (lo_m == lo_n) && (hi_m == hi_n) && m != n &&
                        entry_grp(cd.b, P.batch ? kGrpMask : 0u) == qa_idx;
      const uint64_t fp_m = key64(lo_m, hi_m, P.batch ? qa_idx : 0u) >> 11;
      if (!same) {
        // Different sets (or queries).  A candidate made from compact words
        // (or from cut fingerprints) counts as one only if the whole ones agree.
        if (P.compact && ((fp_m ^ (key64(lo_n, hi_n, P.batch ? qa_idx : 0u) >> 11)) & P.whole_mask))
          atomicAdd(&P.flags[kFlagDropped], 1u);
        else
          atomicAdd(&P.flags[kFlagFalseCand], 1u);
      } else if ((fp_m ^ entry_fp(cd.a)) & P.fp_mask) {
        atomicAdd(&P.flags[kFlagVerifyFail], 1u);  // the entry does not hold this set's fingerprint
      } else {
        // Kind 1 iff rad(m) = rad(n) (Algorithm 2); the third-condition bit
        // marks a first-kind pair with rad(m + 2) = rad(n + 2) as well.
        const uint32_t base = rad[0] == rad[2] ? 1u : 2u;
        const bool three = third && base == 1u && rad[4] == rad[5];
        const uint32_t kind = base | (three ? kKindThird : 0u);
        if ((P.kinds & base) || three) {
          const uint32_t k = atomicAdd(&P.flags[kFlagOut], 1u);
          if (k < P.out_cap) {
            OutPair o;
            o.m = m;
            o.n = n;
            o.kind = kind;
            o.query = P.batch ? qa_idx : 0u;
            P.out[k] = o;
          }
        }
      }
    }
  }
  report<BLOCK>(P, active);
}

// Start of a call: counters and group cursors to zero, and the query tables,
// from the host's staging buffer or (at most kFewQueries) from the arguments.
constexpr uint32_t kFewQueries = 2;
struct BeginParams {
  Counters* n;
  uint32_t* cnt2;  // n_cnt2 cursors
  uint32_t n_cnt2;
  Query* queries;
  uint64_t* seg_prefix;
  uint32_t* small;
  uint32_t n_queries, n_small;
  Query few[kFewQueries];  // without staged_queries
  uint64_t few_prefix[kFewQueries + 1];
  uint32_t few_small[kFewQueries];
  const uint64_t* staged_queries;  // host memory: the queries, n_queries + 1 words, n_small half words
  const uint64_t* staged_prefix;
  const uint32_t* staged_small;
};
__global__ __launch_bounds__(256) void k_begin(BeginParams P) {
  const uint32_t t = blockIdx.x * 256 + threadIdx.x, step = gridDim.x * 256;
  if (P.n && t < 16) P.n->flags[t] = 0;
  if (P.n && t < kAccCount) P.n->acc[t] = 0;
  if (P.n && t < kKernels) P.n->ticks[t] = 0;
  if (P.n && t == 0) P.n->running = 0;
  for (uint32_t i = t; i < P.n_cnt2; i += step) P.cnt2[i] = 0;
  if (!P.staged_queries) {
    if (t < P.n_queries) P.queries[t] = P.few[t];
    if (t <= P.n_queries) P.seg_prefix[t] = P.few_prefix[t];
    if (t < P.n_small) P.small[t] = P.few_small[t];
    return;
  }
  uint64_t* q = reinterpret_cast<uint64_t*>(P.queries);
  constexpr uint32_t kWords = sizeof(Query) / sizeof(uint64_t);
  for (uint32_t i = t; i < kWords * P.n_queries; i += step) q[i] = P.staged_queries[i];
  for (uint32_t i = t; i < P.n_queries + 1; i += step) P.seg_prefix[i] = P.staged_prefix[i];
  for (uint32_t i = t; i < P.n_small; i += step) P.small[i] = P.staged_small[i];
}

__global__ void k_fill_u32(uint32_t* p, uint64_t n, uint32_t v) {
  for (uint64_t i = blockIdx.x * static_cast<uint64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<uint64_t>(gridDim.x) * blockDim.x)
    p[i] = v;
}

}  // namespace bx
