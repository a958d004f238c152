// Step 1: signature matching -- group R request keys.
//
// HeraSys Sec. 3.3 (I): a node whose signature matches a node already in the
// window is fused into it; Eq. (3) aggregates over the merged set M(v*).  The
// paper detects matches with a hash map (Appendix B.3, Phase 1).  On the GPU
// every path below gives the same canonical outputs (those of a stable sort
// of (key, request) pairs): distinct keys ascending, the survivor of a group
// is its earliest request, counts[g] = |M(v*)|, inverse[i] = group.
//
// Paths:
//   R <= kSmallMax : one workgroup groups the keys in an LDS hash table
//                    (first request by atomic min, group size by atomic add),
//                    orders the distinct keys by counting, for each, the
//                    distinct keys below it (in its bucket of the key range),
//                    and maps every request to its group through the table;
//   larger R       : the key range is found on the device; keys that take at
//                    most R values are grouped by direct addressing over the
//                    range; keys spread evenly over a wide range (signatures) by a
//                    hash table in the workspace, their distinct values
//                    ordered bucket by bucket of the range; others by an LSD
//                    radix sort (8-bit digits over key - min, so only the bits
//                    that vary are sorted; stable local ranking with wavefront
//                    ballots, then head flags, a compaction and group sizes)
//                    in one persistent launch.
#include "common.h"

namespace hs {

constexpr int kSmallMax = 4096;
constexpr int kSmallThreads = 1024;
constexpr int kRadixThreads = 256;
constexpr int kRadixItems = 16;
constexpr int kTile = kRadixThreads * kRadixItems;  // keys per block
constexpr int kRadixBits = 8;
constexpr int kBins = 1 << kRadixBits;

__device__ __forceinline__ uint64_t map_key(int64_t k) {
  return (uint64_t)k ^ 0x8000000000000000ull;
}
__device__ __forceinline__ int64_t unmap_key(uint64_t u) {
  return (int64_t)(u ^ 0x8000000000000000ull);
}

// Inclusive prefix sum over a block; returns the inclusive value for this
// thread and the block total.  `wsum` needs blockDim/64 + 1 entries.
template <int NT>
__device__ __forceinline__ uint32_t block_inclusive_scan(uint32_t v, uint32_t *wsum,
                                                         uint32_t &total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    uint32_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) wsum[w] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t acc = 0;
    for (int i = 0; i < NT / 64; ++i) {
      uint32_t t = wsum[i];
      wsum[i] = acc;
      acc += t;
    }
    wsum[NT / 64] = acc;
  }
  __syncthreads();
  total = wsum[NT / 64];
  uint32_t r = x + wsum[w];
  __syncthreads();
  return r;
}

// ---------------------------------------------------------------- up to 4,096

constexpr int kRankDirect = 512;     // distinct keys ranked over all of them up to here
constexpr int kRankBuckets = 512;    // buckets of the key range above
constexpr int kRankCrowded = 80;     // keys in a bucket that call for other buckets

// One workgroup; RMAX requests at most, in a table of twice as many slots.
// Bound by latency: a few barriers, and the ranking.  Ranking every distinct key
// by counting all of them takes n^2 LDS reads: 1.2 us of the 9 us for 329
// keys, but most of the time from about a thousand.  Above kRankDirect, the keys
// are first put into kRankBuckets buckets of their range, and a key counts only
// those of its bucket.  3,000 requests, 960 distinct: 56 us by a bitonic sort of
// the requests.
// Keys that crowd the range's buckets (ids under a few tenants, dense ids and a
// sentinel) get buckets between RMAX / 8 of their own number instead, taken evenly
// from the table's order, which is that of the hash.  4,096 keys, all but one
// dense: 46 us, 1,496 with the range's buckets; in 64 clusters: 47 us either way
// (the line: uniform keys have 16 or less in a bucket).
template <int RMAX>
__global__ __launch_bounds__(kSmallThreads) void dedup_hash_kernel(
    const int64_t *__restrict__ keys, int R, int64_t *__restrict__ uk, int32_t *__restrict__ fi,
    int32_t *__restrict__ cnt, int32_t *__restrict__ inv, int64_t *__restrict__ nu_out) {
  // Mapped keys (map_key: order-preserving to unsigned) in open addressing
  // with linear probing; mapped value 0 marks an empty slot, so the one key
  // that maps to 0 (INT64_MIN) has a slot of its own, number SLOTS.
  constexpr int SLOTS = 2 * RMAX;    // load factor at most 1/2
  constexpr int PER = RMAX / kSmallThreads;
  __shared__ unsigned long long hk[SLOTS + 1];
  __shared__ int32_t hmin[SLOTS + 1];   // first request; later the group id
  __shared__ int32_t hcnt[SLOTS + 1];
  __shared__ uint16_t order[RMAX];      // slots of the distinct keys
  __shared__ unsigned long long ck[kRankDirect + 8];   // distinct keys, up to kRankDirect
  __shared__ uint32_t bcnt[kRankBuckets], bat[kRankBuckets];
  __shared__ uint64_t smin[kSmallThreads / 64], smax[kSmallThreads / 64];
  __shared__ uint32_t wsum[kSmallThreads / 64 + 1];
  __shared__ int32_t ncomp, crowded;
  const int tid = threadIdx.x;
  for (int t = tid; t <= SLOTS; t += kSmallThreads) {
    hk[t] = 0ull;
    hmin[t] = 0x7FFFFFFF;
    hcnt[t] = 0;
  }
  if (tid < kRankBuckets) bcnt[tid] = 0u;
  if (tid == 0) ncomp = crowded = 0;
  __syncthreads();
  int myslot[PER];
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int p = tid + e * kSmallThreads;
    myslot[e] = -1;
    if (p < R) {
      const unsigned long long m = map_key(keys[p]);
      uint32_t sl = SLOTS;
      if (m != 0ull) {
        sl = (uint32_t)((m * 0x9E3779B97F4A7C15ull) >> 51) & (SLOTS - 1);
        for (;;) {   // at most R probes: fewer keys than slots
          const unsigned long long prev = atomicCAS(&hk[sl], 0ull, m);
          if (prev == 0ull || prev == m) break;
          sl = (sl + 1) & (SLOTS - 1);
        }
      }
      atomicMin(&hmin[sl], p);
      atomicAdd(&hcnt[sl], 1);
      myslot[e] = (int)sl;
    }
  }
  __syncthreads();
  // distinct keys in any order (one slot per distinct key holds requests)
  uint64_t mn = ~0ull, mx = 0ull;
  for (int t = tid; t <= SLOTS; t += kSmallThreads) {
    if (hcnt[t] != 0) {
      const int u = atomicAdd(&ncomp, 1);
      const uint64_t m = hk[t];
      order[u] = (uint16_t)t;
      if (u < kRankDirect) ck[u] = m;
      mn = m < mn ? m : mn;
      mx = m > mx ? m : mx;
    }
  }
  __syncthreads();
  const int n = ncomp;
  auto put = [&](int sl, uint64_t m, int r) {
    uk[r] = unmap_key(m);
    fi[r] = hmin[sl];
    if (cnt) cnt[r] = hcnt[sl];
    hmin[sl] = r;   // (this thread is the only one that reads the slot here)
  };
  if (n <= kRankDirect) {
    // group id = number of distinct keys below (keys are distinct); the list
    // is padded to a multiple of 8 with all-ones keys (never below a key) so
    // that eight independent reads are in flight at a time
    const int n8 = (n + 7) & ~7;
    if (tid < n8 - n) ck[n + tid] = ~0ull;
    __syncthreads();
    if (tid < n) {
      const unsigned long long m = ck[tid];
      int r = 0;
      for (int j = 0; j < n8; j += 8) {
        unsigned long long b[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) b[t] = ck[j + t];
#pragma unroll
        for (int t = 0; t < 8; ++t) r += b[t] < m ? 1 : 0;
      }
      put(order[tid], m, r);
    }
  } else {
    for (int o = 32; o > 0; o >>= 1) {
      const uint64_t a = __shfl_xor(mn, o, 64), c = __shfl_xor(mx, o, 64);
      mn = a < mn ? a : mn;
      mx = c > mx ? c : mx;
    }
    if ((tid & 63) == 0) {
      smin[tid >> 6] = mn;
      smax[tid >> 6] = mx;
    }
    __syncthreads();
    mn = smin[0];
    mx = smax[0];
    for (int w = 1; w < kSmallThreads / 64; ++w) {
      mn = smin[w] < mn ? smin[w] : mn;
      mx = smax[w] > mx ? smax[w] : mx;
    }
    // bucket = the top 9 bits of the range's key - min
    const int bits = 64 - __clzll((long long)(mx - mn));   // (n > 1: mx > mn)
    const int shift = bits > 9 ? bits - 9 : 0;
    int msl[PER];
    uint32_t mb[PER], mat[PER];
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const int u = tid + e * kSmallThreads;
      msl[e] = u < n ? (int)order[u] : -1;
      if (u < n) {
        mb[e] = (uint32_t)((hk[msl[e]] - mn) >> shift);
        mat[e] = atomicAdd(&bcnt[mb[e]], 1u);
      }
    }
#pragma unroll
    for (int e = 0; e < PER; ++e)
      if (msl[e] >= 0 && mat[e] >= (uint32_t)kRankCrowded) crowded = 1;
    __syncthreads();
    if (crowded) {
      // the sampled keys, sorted by counting, T threads to each
      constexpr int M = RMAX / 8, T = kSmallThreads / M;
      static_assert(M <= kRankBuckets && M <= kRankDirect && M % (8 * T) == 0, "sampled keys");
      const int u = tid / T, part = tid % T;
      const uint64_t x = hk[order[u * n / M]];   // (n > kRankDirect: distinct)
      if (part == 0) ck[u] = x;
      if (tid < kRankBuckets) bcnt[tid] = 0u;
      __syncthreads();
      int r = 0;
      for (int j = part * (M / T); j < (part + 1) * (M / T); j += 8) {
        uint64_t y[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) y[t] = ck[j + t];
#pragma unroll
        for (int t = 0; t < 8; ++t) r += y[t] < x ? 1 : 0;
      }
#pragma unroll
      for (int o = 1; o < T; o <<= 1) r += __shfl_xor(r, o, 64);
      __syncthreads();
      if (part == 0) ck[r] = x;
      __syncthreads();
      // a key's bucket: the last of them that is not above it, or the first
      int lo[PER];
#pragma unroll
      for (int e = 0; e < PER; ++e) lo[e] = 0;
#pragma unroll 1
      for (int half = M / 2; half > 0; half >>= 1) {
#pragma unroll
        for (int e = 0; e < PER; ++e)
          if (msl[e] >= 0 && ck[lo[e] + half] <= hk[msl[e]]) lo[e] += half;
      }
#pragma unroll
      for (int e = 0; e < PER; ++e) {
        if (msl[e] < 0) continue;
        mb[e] = (uint32_t)lo[e];
        mat[e] = atomicAdd(&bcnt[lo[e]], 1u);
      }
      __syncthreads();
    }
    uint32_t total;
    const uint32_t c = tid < kRankBuckets ? bcnt[tid] : 0u;
    const uint32_t incl = block_inclusive_scan<kSmallThreads>(c, wsum, total);
    if (tid < kRankBuckets) bat[tid] = incl - c;
    __syncthreads();
    // (every thread has read its entries of `order`)
#pragma unroll
    for (int e = 0; e < PER; ++e)
      if (msl[e] >= 0) order[bat[mb[e]] + mat[e]] = (uint16_t)msl[e];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      if (msl[e] < 0) continue;
      const uint64_t m = hk[msl[e]];
      const int b0 = (int)bat[mb[e]], b1 = b0 + (int)bcnt[mb[e]];
      int r = b0;
      for (int j = b0; j < b1; j += 4) {
        uint64_t y[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) y[t] = j + t < b1 ? hk[order[j + t]] : ~0ull;
#pragma unroll
        for (int t = 0; t < 4; ++t) r += y[t] < m ? 1 : 0;
      }
      put(msl[e], m, r);
    }
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int p = tid + e * kSmallThreads;
    if (p < R) inv[p] = hmin[myslot[e]];
  }
  if (tid == 0) *nu_out = (int64_t)n;
}

// ---------------------------------------------------------------- larger R
//
// Five launches whatever the keys:
//   prep    : mapped keys and request numbers, per-workgroup key min/max, and
//             the scratch the later launches need at its neutral value;
//   mark    : every workgroup reduces the min/max itself and picks the path;
//             dense path (the keys take at most R values, max - min < R):
//             first request and group size per key value; hash path: the same
//             per slot of the hash table, each new key also appended to its
//             bucket of the key range;
//   groups  : dense path: the present values numbered in ascending order by
//             a single-pass scan (each value block looks back at the running
//             totals of the blocks before it), with the per-group outputs;
//             hash path: each bucket's keys ranked, with the outputs;
//   inverse : dense and hash path: request -> group;
//   radix   : sort path (returns at once on the others): one persistent
//             launch of at most kRadixGridMax workgroups, all resident, that
//             runs every LSD pass (8-bit digits of key - min, one pass per
//             8 bits of max - min), then head flags, compaction and group
//             sizes, with grid barriers between the phases.

constexpr int kPrepMax = 1024;        // prep workgroups (min/max partials)
constexpr int kRadixGridMax = 256;    // workgroups of the persistent sort
constexpr int kBarGroups = 16;        // arrival counters of the grid barrier
constexpr int kCtlStride = 32;        // 32-bit words between counters (128 B)
// control words: [0] value-block ticket of the groups launch; [kCtlFull] set
// when the hash path has given up (a bucket is full, or a search too long);
// barrier arrival counter j at (1 + j) * kCtlStride; the barrier's release counter at
// (1 + kBarGroups) * kCtlStride
constexpr int kCtlWords = (2 + kBarGroups) * kCtlStride;
constexpr int kCtlFull = 1;
constexpr int kSampleKeys = 1024;   // the first keys of the window

struct RadixWs {
  uint64_t *keyA, *keyB;
  int32_t *idxA, *idxB;
  uint64_t *pmin, *pmax;   // per-prep-workgroup min/max of mapped keys
  uint64_t *range;         // [0] = global min, [1] = radix pass count,
                           // [2] = key values of the dense path (0: others),
                           // [3] = hash path, [4] = range of the sampled keys
                           // where they suit that path (else 0)
  uint32_t *hist;          // kBins x nb, digit-major (scanned in place)
  uint32_t *dtot;          // kBins digit totals of a pass
  uint32_t *bheads;        // heads per tile (scanned in place)
  int32_t *start;          // group start positions
  uint64_t *flags;         // dense value blocks: running-total words
  uint32_t *ctl;           // kCtlWords control words
  // hash path (hbits = 0: none); everything but gid and the buckets starts at 0
  int hbits;               // log2 of the table's slots
  unsigned long long *hk;  // [slots] mapped keys (0: empty); slot `slots` is
                           // that of the key that maps to 0
  uint32_t *hfirst;        // [slots + 1] R - first request
  uint32_t *hcnt;          // [slots + 1] group size
  int32_t *hgid;           // [slots + 1] group
  uint32_t *bcnt;          // [buckets] keys per bucket
  uint64_t *bkey;          // [buckets][kBucketCap]
  int32_t *bslot;          // [buckets][kBucketCap]
};

// Hash path.  The sort takes 8 passes for 64-bit signatures, each with two or
// three grid barriers: 410 us for 200,000 of them, of which the bytes are 5.
// (200,000 signatures, 95,000 distinct: marking 52 us, groups 8 us.)  The table
// has at least 2 R slots; with R rounded up to a power of two there
// is a bucket of the key range per 256 requests.  Uniform keys (the signatures
// are hash values) fill a bucket to at most 256 on average over the full range
// of 64 bits, and to at most 512 over a range just above a power of two (half of
// the buckets used), never to kBucketCap.  Keys that do are left to the sort.  Up
// to 2^20 requests: the table and the buckets take 90 bytes per request or more.
//
// A key's search in the table ends after kProbeMax slots.  In a table that is at
// most half full the longest search is about ln(R) / 0.19 slots (72 for 2^20 keys),
// but keys whose products with the hash's multiplier share their top bits (an
// arithmetic progression of a suitable step does) would search all R: such keys are
// left to the sort as well.
constexpr int kHashRMax = 1 << 20;
constexpr int kBucketCap = 1024;
constexpr int kProbeMax = 256;
__host__ __device__ __forceinline__ int hash_bits(int64_t R) {   // 2 R <= 2^bits < 4 R
  int b = 13;
  while (((int64_t)1 << b) < 2 * R) ++b;
  return b;
}
__host__ __device__ __forceinline__ int bucket_bits(int hbits) { return hbits - 9; }
// A key's bucket is (key - min) >> shift, with keys `span` apart.
__device__ __forceinline__ int bucket_shift(uint64_t span, int hbits) {
  const int bits = 64 - __clzll((long long)span), bb = bucket_bits(hbits);   // (span > 0)
  return bits > bb ? bits - bb : 0;
}

// ------------------------------------------------ grid-wide helpers

// Barrier over the G workgroups of a launch that are all resident at once
// (G at most what the device holds of them).  `k`
// counts the barriers this workgroup has passed (the counters only grow
// within a launch; prep zeroes them).  Arrivals are spread over kBarGroups
// counters so that no single address takes all G of them; the last arrival
// of each group bumps the release counter that everyone waits on.
__device__ __forceinline__ void grid_barrier(uint32_t *ctl, int G, uint32_t &k) {
  ++k;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
  __syncthreads();
  if (threadIdx.x == 0) {
    const int ng = G < kBarGroups ? G : kBarGroups;
    const int j = (int)blockIdx.x % ng;
    const uint32_t gsize = (uint32_t)(G / ng + (j < G % ng ? 1 : 0));
    uint32_t *sub = ctl + (1 + j) * kCtlStride;
    uint32_t *rel = ctl + (1 + kBarGroups) * kCtlStride;
    const uint32_t old =
        __hip_atomic_fetch_add(sub, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
    if (old + 1 == k * gsize)
      __hip_atomic_fetch_add(rel, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    while (__hip_atomic_load(rel, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) < k * (uint32_t)ng)
      __builtin_amdgcn_s_sleep(1);
  }
  __syncthreads();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
}

// Exclusive prefix sum of a[0, n) in place by one workgroup; returns the
// total.
__device__ uint32_t block_scan_inplace(uint32_t *a, int64_t n) {
  __shared__ uint32_t wsum[kRadixThreads / 64 + 1];
  constexpr int P = 4;
  uint32_t carry = 0;
  for (int64_t c0 = 0; c0 < n; c0 += kRadixThreads * P) {
    const int64_t i0 = c0 + (int64_t)threadIdx.x * P;
    uint32_t v[P], sum = 0;
#pragma unroll
    for (int e = 0; e < P; ++e) {
      v[e] = i0 + e < n ? a[i0 + e] : 0u;
      sum += v[e];
    }
    uint32_t total;
    uint32_t run = carry + block_inclusive_scan<kRadixThreads>(sum, wsum, total) - sum;
#pragma unroll
    for (int e = 0; e < P; ++e)
      if (i0 + e < n) {
        a[i0 + e] = run;
        run += v[e];
      }
    carry += total;
  }
  return carry;
}

// ------------------------------------------------ prep and path choice

// First slot to search for a mapped key in a table of 2^bits slots.
__device__ __forceinline__ uint32_t hash_of(uint64_t m, int bits) {
  return (uint32_t)((m * 0x9E3779B97F4A7C15ull) >> (64 - bits));
}

// Whether the keys suit the hash path, from a sample: the window's first 1,024.
// They must lie R or more apart and no bucket may be expected to fill.  Clustered
// keys (ids under a few tenants, dense ids and a sentinel) put most of the range's
// keys in a few buckets: one counter then takes an atomic add for every key, 11 ns
// each, and the sort still follows.  200,000 dense ids and one far key: 2,680 us,
// the sort alone 404; a million ids under two tenants 5,452, 903.
//
// n distinct keys of the sample with p ordered pairs of them in one bucket: the
// keys that share a random key's bucket are about D p / n^2 of D distinct ones,
// and D is at most R n / 1024 (new keys get rarer).  Signatures have 512 at most
// (twice R / buckets, half of the buckets used) with a deviation of 32; the limit
// lies between that and the bucket's size.  One crowded bucket among many weighs
// little in that mean: t = 2^20 / R keys of the sample in one bucket stand for the
// 1,024 that it holds, and t + 4 sqrt(t) + 4 are not there by chance.  5,000 keys,
// 30 % of them within one bucket: 268 us with an attempt, 232 without.  What gets
// past both costs the attempt: 1 % of 200,000 keys in one bucket 526 us (the sort
// alone 441), of 10^6 1,874 (1,359), 2 % of 65,536 333 (280).  A search of more than 128 slots here
// (36 are usual for 1,024 keys in 2,048 slots) tells keys that the hash does not
// spread.
constexpr uint64_t kSpreadMax = 768;
//
// Workgroup e of E: the first decides, the others clear the table and the bucket
// counts if the keys lie far enough apart.  They are not the workgroups that read
// the keys: 256 of those, each reading the same 8 KiB for this, took the dense path
// 1 us longer (262,144 ids and the gather of their rows: 86.5 us).
__device__ void sample_spread(const int64_t *__restrict__ keys, int R, const RadixWs &ws, int e0,
                              int E) {
  constexpr int per = kSampleKeys / kRadixThreads, slots = 2 * kSampleKeys, W = kRadixThreads / 64;
  constexpr int lbits = 11, kBucketsMax = 1 << 12;
  static_assert(slots == 1 << lbits && kHashRMax == 1 << 20, "sample table, buckets of 2^20 keys");
  __shared__ unsigned long long set[slots];
  __shared__ uint32_t cnt[kBucketsMax];
  __shared__ uint64_t smin[W], smax[W];
  __shared__ uint32_t total, unfit;   // distinct keys << 21 | pairs (< 2^20)
  const int tid = threadIdx.x;
  uint64_t m[per], mn = ~0ull, mx = 0ull;
#pragma unroll
  for (int e = 0; e < per; ++e) {
    m[e] = map_key(keys[e * kRadixThreads + tid]);   // (R > kSmallMax)
    mn = m[e] < mn ? m[e] : mn;
    mx = m[e] > mx ? m[e] : mx;
  }
  if (e0 == 0) {
    for (int i = tid; i < slots; i += kRadixThreads) set[i] = 0ull;
    for (int i = tid; i < 1 << bucket_bits(ws.hbits); i += kRadixThreads) cnt[i] = 0u;
    if (tid == 0) total = unfit = 0u;
  }
  for (int o = 32; o > 0; o >>= 1) {
    const uint64_t a = __shfl_xor(mn, o, 64), c = __shfl_xor(mx, o, 64);
    mn = a < mn ? a : mn;
    mx = c > mx ? c : mx;
  }
  if ((tid & 63) == 0) {
    smin[tid >> 6] = mn;
    smax[tid >> 6] = mx;
  }
  __syncthreads();
  for (int w = 0; w < W; ++w) {
    mn = smin[w] < mn ? smin[w] : mn;
    mx = smax[w] > mx ? smax[w] : mx;
  }
  const uint64_t span = mx - mn;
  if (span < (uint64_t)R) {
    if (e0 == 0 && tid == 0) ws.range[4] = 0ull;
    return;
  }
  if (e0 > 0) {
    const int64_t slots = (int64_t)1 << ws.hbits, gs = (int64_t)(E - 1) * kRadixThreads;
    for (int64_t i = (int64_t)(e0 - 1) * kRadixThreads + tid; i <= slots; i += gs) {
      if (i < slots) ws.hk[i] = 0ull;
      ws.hfirst[i] = 0u;
      ws.hcnt[i] = 0u;
      if (i < ((int64_t)1 << bucket_bits(ws.hbits))) ws.bcnt[i] = 0u;
    }
    return;
  }
  const int shift = bucket_shift(span, ws.hbits);
  const uint32_t t = (1u << 20) / (uint32_t)R, crowd = t + 4u * (uint32_t)sqrtf((float)t) + 4u;
  // (the four keys' first steps are in flight together; 0, the mark of an empty
  // slot, is one key at most and is not counted)
  uint32_t h[per], sum = 0u;
  unsigned long long prev[per];
#pragma unroll
  for (int e = 0; e < per; ++e) {
    h[e] = hash_of(m[e], lbits) & (slots - 1);
    prev[e] = atomicCAS(&set[h[e]], 0ull, m[e]);
  }
#pragma unroll
  for (int e = 0; e < per; ++e) {
    int left = 128;
    while (prev[e] != 0ull && prev[e] != m[e] && --left > 0) {
      h[e] = (h[e] + 1) & (slots - 1);
      prev[e] = atomicCAS(&set[h[e]], 0ull, m[e]);
    }
    if (left == 0) unfit = 1u;
  }
#pragma unroll
  for (int e = 0; e < per; ++e)
    if (prev[e] == 0ull && m[e] != 0ull) {
      const uint32_t others = atomicAdd(&cnt[(uint32_t)((m[e] - mn) >> shift)], 1u);
      sum += (1u << 21) + 2u * others;
      if (others >= crowd) unfit = 1u;
    }
  for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
  if ((tid & 63) == 0) atomicAdd(&total, sum);
  __syncthreads();
  if (tid == 0) {
    const uint64_t n = total >> 21, pairs = total & ((1u << 21) - 1u);
    const bool fit = unfit == 0u && (uint64_t)R * pairs <= kSpreadMax * kSampleKeys * n;
    ws.range[4] = fit ? span : 0ull;
  }
}

// Workgroup b of P: chunks of kPrepChunk requests b, b + P, ... -> mapped
// keys (keyA), request numbers (idxA) and the min/max over them; the dense
// tables for up to R values, the value-block words and the control words to
// their neutral values.
constexpr int kPrepChunk = 4 * kRadixThreads;
__global__ __launch_bounds__(kRadixThreads) void dedup_prep_kernel(
    const int64_t *__restrict__ keys, int R, int P, RadixWs ws) {
  __shared__ uint64_t smin[kRadixThreads / 64], smax[kRadixThreads / 64];
  const int tid = threadIdx.x;
  if ((int)blockIdx.x >= P) {   // (hash path only)
    sample_spread(keys, R, ws, (int)blockIdx.x - P, (int)gridDim.x - P);
    return;
  }
  uint64_t mn = ~0ull, mx = 0ull;
  for (int64_t c = blockIdx.x; c * kPrepChunk < R; c += P) {
#pragma unroll
    for (int e = 0; e < kPrepChunk / kRadixThreads; ++e) {
      const int64_t p = c * kPrepChunk + e * kRadixThreads + tid;
      if (p < R) {
        const uint64_t k = map_key(keys[p]);
        ws.keyA[p] = k;
        ws.idxA[p] = (int32_t)p;
        mn = k < mn ? k : mn;
        mx = k > mx ? k : mx;
      }
    }
  }
  for (int o = 32; o > 0; o >>= 1) {
    const uint64_t a = __shfl_xor(mn, o, 64), c = __shfl_xor(mx, o, 64);
    mn = a < mn ? a : mn;
    mx = c > mx ? c : mx;
  }
  if ((tid & 63) == 0) {
    smin[tid >> 6] = mn;
    smax[tid >> 6] = mx;
  }
  __syncthreads();
  if (tid == 0) {
    for (int w = 1; w < kRadixThreads / 64; ++w) {
      mn = smin[w] < mn ? smin[w] : mn;
      mx = smax[w] > mx ? smax[w] : mx;
    }
    ws.pmin[blockIdx.x] = mn;
    ws.pmax[blockIdx.x] = mx;
  }
  // dense tables (first request, group size) over [0, R) >= [0, nv)
  int32_t *first = (int32_t *)ws.keyB, *count = (int32_t *)ws.keyB + R;
  const int64_t gt = (int64_t)blockIdx.x * kRadixThreads + tid;
  const int64_t gs = (int64_t)P * kRadixThreads;
  for (int64_t v = gt; v < R; v += gs) {
    first[v] = 0x7fffffff;
    count[v] = 0;
  }
  const int64_t nvb = ((int64_t)R + 1023) / 1024;
  for (int64_t i = gt; i < nvb; i += gs) ws.flags[i] = 0ull;
  if (blockIdx.x == 0)
    for (int i = tid; i < kCtlWords; i += kRadixThreads) ws.ctl[i] = 0u;
}

struct Range {
  uint64_t mn;
  uint64_t npass;   // radix passes (0 on the dense path)
  uint64_t nv;      // key values of the dense path (0: others)
  int hash;         // hash path
  uint64_t span;    // max - min
};

// Global min/max over the P prep partials and the path: dense when the keys
// take at most R values (max - min < R), else by hashing where the sampled keys
// suit it (prep has then cleared the table), else radix with one pass per 8 bits of max - min.  Computed by
// every workgroup that calls it.
__device__ Range range_of(int R, int P, const RadixWs &ws) {
  __shared__ uint64_t smin[kRadixThreads / 64], smax[kRadixThreads / 64];
  __shared__ Range res;
  const int tid = threadIdx.x;
  uint64_t mn = ~0ull, mx = 0ull;
  for (int i = tid; i < P; i += kRadixThreads) {
    mn = ws.pmin[i] < mn ? ws.pmin[i] : mn;
    mx = ws.pmax[i] > mx ? ws.pmax[i] : mx;
  }
  for (int o = 32; o > 0; o >>= 1) {
    uint64_t a = __shfl_xor(mn, o, 64), c = __shfl_xor(mx, o, 64);
    mn = a < mn ? a : mn;
    mx = c > mx ? c : mx;
  }
  if ((tid & 63) == 0) {
    smin[tid >> 6] = mn;
    smax[tid >> 6] = mx;
  }
  __syncthreads();
  if (tid == 0) {
    for (int w = 1; w < kRadixThreads / 64; ++w) {
      mn = smin[w] < mn ? smin[w] : mn;
      mx = smax[w] > mx ? smax[w] : mx;
    }
    const uint64_t span = mx - mn;
    const int bits = span ? 64 - __clzll((long long)span) : 0;
    const bool dense = span < (uint64_t)R;
    res.mn = mn;
    res.npass = dense ? 0ull : (uint64_t)((bits + kRadixBits - 1) / kRadixBits);
    res.nv = dense ? span + 1 : 0ull;
    // (a range of twice the sample's or more has keys that the sample did not see;
    // the dense path does not wait for the word)
    res.hash = !dense && ws.hbits && span >> 1 <= ws.range[4] ? 1 : 0;
    res.span = span;
  }
  __syncthreads();
  return res;
}

// ---------------------------------------------------------------- dense path
//
// When the R mapped keys take at most R values (e.g. chunk row ids), the
// groups are found by direct addressing over [min, max] instead of sorting:
// per key value v, the first request (atomic min) and the group size (atomic
// add); a scan over the values numbers the present ones in ascending key
// order; each request then reads its group.  Same canonical outputs as the
// sort.  Value arrays reuse the sort's second buffers: first/count in keyB
// (2 x int32 per value), group ids in idxB.

constexpr int kDenseBlk = 1024;                        // values per value block
constexpr int kDensePer = kDenseBlk / kRadixThreads;   // values per thread
constexpr int kAggRound = 1024, kAggSlots = 2048;

// Hash path of the marking launch.  Rounds of kAggRound consecutive requests
// are first combined per key in an LDS table; the thread that entered a key
// there looks it up in the workspace's table (its up to four keys' first
// probes are in flight together), adds the round's first request and count to
// its slot and, if the key is new, appends it to its bucket.  idxB gets every
// request's slot.  Bound by the latency of a few dependent device-scope
// atomics per key.  Once any workgroup has given up (kCtlFull) the others do no
// more than they have begun.
// lk, lfirst, lcnt: [kAggSlots] mapped key (0: empty), first request (later the
// slot), count.
__device__ __forceinline__ void hash_insert(int R, const Range &rg, const RadixWs &ws,
                                            unsigned long long *lk, int32_t *lfirst,
                                            int32_t *lcnt) {
  constexpr int per = kAggRound / kRadixThreads;
  __shared__ int32_t zfirst, zcnt;               // the key that maps to 0
  const int tid = threadIdx.x, hbits = ws.hbits, shift = bucket_shift(rg.span, hbits);
  const uint32_t hmask = (1u << hbits) - 1u;
  constexpr int lbits = 11;
  static_assert((1 << lbits) == kAggSlots, "LDS table");
  auto full = [&]() {
    return __hip_atomic_load(&ws.ctl[kCtlFull], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u;
  };
  auto give_up = [&]() {
    __hip_atomic_store(&ws.ctl[kCtlFull], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  for (int64_t round = blockIdx.x; round * kAggRound < R; round += gridDim.x) {
    const int64_t base = round * kAggRound;
    for (int j = tid; j < kAggSlots; j += kRadixThreads) {
      lk[j] = 0ull;
      lfirst[j] = 0x7fffffff;
      lcnt[j] = 0;
    }
    if (tid == 0) {
      zfirst = 0x7fffffff;
      zcnt = 0;
    }
    __syncthreads();
    unsigned long long m[per];
    int ls[per];          // LDS slot of the request's key (-1: none, -2: key 0)
    bool own[per];        // this request entered it
#pragma unroll
    for (int e = 0; e < per; ++e) {
      const int64_t p = base + e * kRadixThreads + tid;
      m[e] = p < R ? ws.keyA[p] : 0ull;
      ls[e] = p < R ? -2 : -1;
      own[e] = false;
    }
#pragma unroll
    for (int e = 0; e < per; ++e) {
      const int32_t p = (int32_t)(base + e * kRadixThreads + tid);
      if (m[e] != 0ull) {
        uint32_t h = hash_of(m[e], lbits);
        for (;;) {   // at most kAggRound keys in kAggSlots slots: a slot is found
          const unsigned long long prev = atomicCAS(&lk[h], 0ull, m[e]);
          own[e] = prev == 0ull;
          if (prev == 0ull || prev == m[e]) break;
          h = (h + 1) & (kAggSlots - 1);
        }
        ls[e] = (int)h;
        atomicMin(&lfirst[h], p);
        atomicAdd(&lcnt[h], 1);
      } else if (ls[e] == -2) {
        atomicMin(&zfirst, p);
        atomicAdd(&zcnt, 1);
      }
    }
    __syncthreads();
    uint32_t gs[per];
    unsigned long long prev[per];
#pragma unroll
    for (int e = 0; e < per; ++e) {
      gs[e] = hash_of(m[e], hbits) & hmask;
      prev[e] = own[e] ? atomicCAS(&ws.hk[gs[e]], 0ull, m[e]) : m[e];
    }
#pragma unroll
    for (int e = 0; e < per; ++e) {
      for (int left = kProbeMax; prev[e] != 0ull && prev[e] != m[e]; --left) {
        if (left == 0 || ((left & 15) == 8 && full())) {
          give_up();
          own[e] = false;   // (nobody reads what would follow)
          break;
        }
        gs[e] = (gs[e] + 1) & hmask;
        prev[e] = atomicCAS(&ws.hk[gs[e]], 0ull, m[e]);
      }
    }
    auto add = [&](uint32_t slot, int32_t first, int32_t cnt) {
      atomicMax(&ws.hfirst[slot], (uint32_t)(R - first));
      atomicAdd(&ws.hcnt[slot], (uint32_t)cnt);
    };
    auto append = [&](uint64_t key, uint32_t slot) {
      const uint32_t b = (uint32_t)((key - rg.mn) >> shift);
      const uint32_t at = atomicAdd(&ws.bcnt[b], 1u);
      if (at < (uint32_t)kBucketCap) {
        ws.bkey[(int64_t)b * kBucketCap + at] = key;
        ws.bslot[(int64_t)b * kBucketCap + at] = (int32_t)slot;
      } else {
        give_up();
      }
    };
#pragma unroll
    for (int e = 0; e < per; ++e) {
      if (!own[e]) continue;
      add(gs[e], lfirst[ls[e]], lcnt[ls[e]]);
      if (prev[e] == 0ull) append(m[e], gs[e]);
      lfirst[ls[e]] = (int32_t)gs[e];   // (only its owner reads the entry here)
    }
    if (tid == 0 && zcnt > 0) {
      const uint32_t slot = 1u << hbits;
      atomicMax(&ws.hfirst[slot], (uint32_t)(R - zfirst));
      if (atomicAdd(&ws.hcnt[slot], (uint32_t)zcnt) == 0u) append(0ull, slot);
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < per; ++e) {
      const int64_t p = base + e * kRadixThreads + tid;
      if (p < R) ws.idxB[p] = ls[e] >= 0 ? lfirst[ls[e]] : (1 << hbits);
    }
    __syncthreads();
  }
}

// Hash path of the groups launch: bucket b's keys are ranked by counting the
// smaller ones (they are distinct), and its groups follow those of the buckets
// before it.
__device__ void hash_groups(int R, const RadixWs &ws, int64_t *__restrict__ uk,
                            int32_t *__restrict__ fi, int32_t *__restrict__ cnt,
                            int64_t *__restrict__ nu_out) {
  __shared__ uint64_t sk[kBucketCap + 8];
  __shared__ uint32_t wsum[kRadixThreads / 64 + 1];
  if (ws.ctl[kCtlFull]) return;
  const int tid = threadIdx.x, B = 1 << bucket_bits(ws.hbits);
  for (int b = blockIdx.x; b < B; b += gridDim.x) {
    uint32_t before = 0;
    for (int i = tid; i < b; i += kRadixThreads) before += ws.bcnt[i];
    const int n = (int)ws.bcnt[b];   // <= kBucketCap
    for (int i = tid; i < n; i += kRadixThreads) sk[i] = ws.bkey[(int64_t)b * kBucketCap + i];
    const int n8 = (n + 7) & ~7;
    for (int i = n + tid; i < n8; i += kRadixThreads) sk[i] = ~0ull;   // (never below a key)
    uint32_t total;
    block_inclusive_scan<kRadixThreads>(before, wsum, total);   // (and a barrier for sk)
    for (int i = tid; i < n; i += kRadixThreads) {
      const uint64_t m = sk[i];
      uint32_t r = total;
      for (int j = 0; j < n8; j += 8) {
        uint64_t y[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) y[t] = sk[j + t];
#pragma unroll
        for (int t = 0; t < 8; ++t) r += y[t] < m ? 1u : 0u;
      }
      const int32_t slot = ws.bslot[(int64_t)b * kBucketCap + i];
      uk[r] = unmap_key(m);
      fi[r] = R - (int32_t)ws.hfirst[slot];
      if (cnt) cnt[r] = (int32_t)ws.hcnt[slot];
      ws.hgid[slot] = (int32_t)r;
    }
    if (b == B - 1 && tid == 0) *nu_out = (int64_t)total + n;
    __syncthreads();
  }
}

// Rounds of kAggRound consecutive requests are first combined per key value
// in an LDS table (a hot key appears many times per round), then each table
// entry goes to the value arrays with one atomic min and one atomic add.
// Workgroup 0 also stores the path for the later launches.
__global__ __launch_bounds__(kRadixThreads) void dense_mark_kernel(int R, int P, RadixWs ws) {
  __shared__ unsigned long long thash[kAggSlots];   // hash path: mapped keys
  __shared__ int32_t tfirst[kAggSlots], tcount[kAggSlots];
  int32_t *const tkey = (int32_t *)thash;           // dense path: key values
  const Range rg = range_of(R, P, ws);
  const int tid = threadIdx.x;
  if (blockIdx.x == 0 && tid == 0) {
    ws.range[0] = rg.mn;
    ws.range[1] = rg.npass;
    ws.range[2] = rg.nv;
    ws.range[3] = (uint64_t)rg.hash;
  }
  if (__builtin_expect(!rg.nv, 0)) {   // (the dense path's code follows without a jump)
    if (rg.hash) hash_insert(R, rg, ws, thash, tfirst, tcount);
    return;
  }
  int32_t *first = (int32_t *)ws.keyB, *count = (int32_t *)ws.keyB + R;
  for (int64_t round = blockIdx.x; round * kAggRound < R; round += gridDim.x) {
    const int64_t base = round * kAggRound;
    for (int j = tid; j < kAggSlots; j += kRadixThreads) {
      tkey[j] = -1;
      tfirst[j] = 0x7fffffff;
      tcount[j] = 0;
    }
    __syncthreads();
    for (int j = tid; j < kAggRound; j += kRadixThreads) {
      const int64_t p = base + j;
      if (p >= R) break;
      const int32_t v = (int32_t)(ws.keyA[p] - rg.mn);   // < nv <= R
      uint32_t h = ((uint32_t)v * 2654435761u) & (kAggSlots - 1);
      for (;;) {   // at most kAggRound keys in kAggSlots slots: a slot is found
        const int32_t prev = atomicCAS(&tkey[h], -1, v);
        if (prev == -1 || prev == v) break;
        h = (h + 1) & (kAggSlots - 1);
      }
      atomicMin(&tfirst[h], (int32_t)p);
      atomicAdd(&tcount[h], 1);
    }
    __syncthreads();
    for (int j = tid; j < kAggSlots; j += kRadixThreads) {
      const int32_t v = tkey[j];
      if (v >= 0) {
        atomicMin(&first[v], tfirst[j]);
        atomicAdd(&count[v], tcount[j]);
      }
    }
    __syncthreads();
  }
}

// Value-block words: state in the high half (1: the block's own count, 2:
// the running total through the block), the number in the low half.
constexpr uint64_t kFlagAgg = 1ull << 32, kFlagPrefix = 2ull << 32;

// One value block per workgroup, in the order the workgroups start (a ticket,
// so every block it waits on has started): count the present values, publish
// the count, add up the counts or running totals of the blocks before it,
// publish the running total, then number its present values and write the
// per-group outputs.  The last block writes n_u.
__global__ __launch_bounds__(kRadixThreads) void dense_groups_kernel(
    int R, RadixWs ws, int64_t *__restrict__ uk, int32_t *__restrict__ fi,
    int32_t *__restrict__ cnt, int64_t *__restrict__ nu_out) {
  __shared__ uint32_t wsum[kRadixThreads / 64 + 1];
  __shared__ uint32_t s_vb, s_before;
  const uint64_t nv = ws.range[2], hash = ws.range[3];   // (read together)
  if (hash) {
    hash_groups(R, ws, uk, fi, cnt, nu_out);
    return;
  }
  const uint64_t nvb = (nv + kDenseBlk - 1) / kDenseBlk;
  if (blockIdx.x >= nvb) return;
  const int tid = threadIdx.x;
  if (tid == 0)
    s_vb = __hip_atomic_fetch_add(ws.ctl, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  const uint64_t vb = s_vb;
  const uint64_t mn = ws.range[0];
  const int32_t *first = (const int32_t *)ws.keyB, *count = (const int32_t *)ws.keyB + R;
  int32_t *gid = ws.idxB;
  const uint64_t v0 = vb * kDenseBlk + (uint64_t)tid * kDensePer;
  int32_t c[kDensePer];
  uint32_t pr = 0;
#pragma unroll
  for (int e = 0; e < kDensePer; ++e) {
    c[e] = v0 + e < nv ? count[v0 + e] : 0;
    pr += c[e] > 0 ? 1u : 0u;
  }
  uint32_t total;
  const uint32_t incl = block_inclusive_scan<kRadixThreads>(pr, wsum, total);
  if (tid < 64) {
    // wave 0: publish this block's count, then add up the words of the
    // blocks before it, 64 at a time, back to the nearest running total
    // (blocks before the first count as a running total of 0)
    uint64_t *fl = ws.flags;
    const int lane = tid;
    uint32_t before = 0;
    if (vb == 0) {
      if (lane == 0)
        __hip_atomic_store(&fl[0], kFlagPrefix | total, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    } else {
      if (lane == 0)
        __hip_atomic_store(&fl[vb], kFlagAgg | total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      for (int64_t j0 = (int64_t)vb - 1;; j0 -= 64) {
        const int64_t j = j0 - lane;
        uint64_t f = j >= 0 ? __hip_atomic_load(&fl[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                            : kFlagPrefix;
        while (__any(f == 0ull)) {
          __builtin_amdgcn_s_sleep(1);
          if (f == 0ull) f = __hip_atomic_load(&fl[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        const uint64_t pm = __ballot(f >= kFlagPrefix);
        const int stop = pm ? __ffsll((long long)pm) - 1 : 64;
        uint32_t v = lane <= stop ? (uint32_t)f : 0u;
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        before += v;
        if (pm) break;
      }
      if (lane == 0)
        __hip_atomic_store(&fl[vb], kFlagPrefix | (before + total), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
    if (lane == 0) s_before = before;
  }
  __syncthreads();
  uint32_t g = s_before + incl - pr;
#pragma unroll
  for (int e = 0; e < kDensePer; ++e) {
    const uint64_t v = v0 + e;
    if (c[e] > 0) {
      uk[g] = unmap_key(mn + v);
      fi[g] = first[v];
      if (cnt) cnt[g] = c[e];
      gid[v] = (int32_t)g;
      ++g;
    }
  }
  if (vb + 1 == nvb && tid == 0) *nu_out = (int64_t)(s_before + total);
}

// Request -> group.
__global__ __launch_bounds__(256) void dense_inverse_kernel(int R, RadixWs ws,
                                                            int32_t *__restrict__ inv) {
  const uint64_t nv = ws.range[2], hash = ws.range[3];
  if (hash) {
    if (ws.ctl[kCtlFull]) return;
    for (int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x; p < R; p += (int64_t)gridDim.x * 256)
      inv[p] = ws.hgid[ws.idxB[p]];
    return;
  }
  if (!nv) return;
  const uint64_t mn = ws.range[0];
  for (int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x; p < R; p += (int64_t)gridDim.x * 256)
    inv[p] = ws.idxB[ws.keyA[p] - mn];
}

// ---------------------------------------------------------------- sort path

__device__ __forceinline__ uint32_t digit_of(uint64_t k, uint64_t mn, int pass) {
  return (uint32_t)(((k - mn) >> (pass * kRadixBits)) & (kBins - 1));
}

// Digit histogram of tile b for one pass.
__device__ __forceinline__ void hist_phase(int R, int nb, int pass, uint64_t mn, int b,
                                           const RadixWs &ws) {
  __shared__ uint32_t h[kBins];
  const uint64_t *src = (pass & 1) ? ws.keyB : ws.keyA;
  const int tid = threadIdx.x;
  h[tid] = 0;
  __syncthreads();
  for (int e = 0; e < kRadixItems; ++e) {
    int p = b * kTile + e * kRadixThreads + tid;
    if (p < R) atomicAdd(&h[digit_of(src[p], mn, pass)], 1u);
  }
  __syncthreads();
  ws.hist[tid * nb + b] = h[tid];
  __syncthreads();
}

// Stable scatter of tile b by its digit for one pass.  With at most
// kDirectTiles tiles the digit offsets come straight from the histogram;
// otherwise its rows are already exclusive scans over the tiles and dtot
// holds the digit totals.
constexpr int kDirectTiles = 64;
__device__ __forceinline__ void scatter_phase(int R, int nb, int pass, uint64_t mn, int b,
                                              const RadixWs &ws) {
  __shared__ uint32_t goff[kBins];
  __shared__ uint32_t running[kBins];
  __shared__ uint32_t wcount[kRadixThreads / 64][kBins];
  __shared__ uint32_t wsum[kRadixThreads / 64 + 1];
  const uint64_t *ksrc = (pass & 1) ? ws.keyB : ws.keyA;
  uint64_t *kdst = (pass & 1) ? ws.keyA : ws.keyB;
  const int32_t *isrc = (pass & 1) ? ws.idxB : ws.idxA;
  int32_t *idst = (pass & 1) ? ws.idxA : ws.idxB;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;

  // global base of each digit for this tile: all smaller digits everywhere,
  // plus this digit in earlier tiles
  uint32_t tot, prior;
  if (nb <= kDirectTiles) {
    tot = 0;
    prior = 0;
    for (int bb = 0; bb < nb; ++bb) {
      const uint32_t c = ws.hist[tid * nb + bb];
      tot += c;
      prior += bb < b ? c : 0u;
    }
  } else {
    tot = ws.dtot[tid];
    prior = ws.hist[tid * nb + b];
  }
  uint32_t total;
  const uint32_t incl = block_inclusive_scan<kRadixThreads>(tot, wsum, total);
  goff[tid] = incl - tot + prior;
  running[tid] = 0;
  const uint64_t lt = (1ull << lane) - 1ull;
  for (int e = 0; e < kRadixItems; ++e) {
    for (int i = tid; i < (kRadixThreads / 64) * kBins; i += kRadixThreads)
      (&wcount[0][0])[i] = 0;
    __syncthreads();
    int p = b * kTile + e * kRadixThreads + tid;
    bool valid = p < R;
    uint64_t key = valid ? ksrc[p] : 0ull;
    int32_t idx = valid ? isrc[p] : 0;
    uint32_t d = valid ? digit_of(key, mn, pass) : 0u;
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int bit = 0; bit < kRadixBits; ++bit) {
      bool s = (d >> bit) & 1u;
      uint64_t bal = __ballot(s);
      peers &= s ? bal : ~bal;
    }
    uint32_t rank = (uint32_t)__popcll(peers & lt);
    if (valid && rank == 0) wcount[w][d] = (uint32_t)__popcll(peers);
    __syncthreads();
    if (valid) {
      uint32_t pos = goff[d] + running[d] + rank;
      for (int ww = 0; ww < w; ++ww) pos += wcount[ww][d];
      if (pos < (uint32_t)R) {  // always true for a consistent histogram
        kdst[pos] = key;
        idst[pos] = idx;
      }
    }
    __syncthreads();
    uint32_t add = 0;
    for (int ww = 0; ww < kRadixThreads / 64; ++ww) add += wcount[ww][tid];
    running[tid] += add;
    __syncthreads();
  }
}

__device__ __forceinline__ const uint64_t *sorted_keys(const RadixWs &ws, uint64_t npass) {
  return (npass & 1) ? ws.keyB : ws.keyA;
}
__device__ __forceinline__ const int32_t *sorted_idx(const RadixWs &ws, uint64_t npass) {
  return (npass & 1) ? ws.idxB : ws.idxA;
}

// Group heads (first of each run of equal keys) in tile b of the sorted keys.
__device__ __forceinline__ void heads_phase(int R, uint64_t npass, int b, const RadixWs &ws) {
  __shared__ uint32_t wsum[kRadixThreads / 64 + 1];
  const uint64_t *k = sorted_keys(ws, npass);
  const int tid = threadIdx.x;
  uint32_t h = 0;
  for (int e = 0; e < kRadixItems; ++e) {
    int p = b * kTile + e * kRadixThreads + tid;
    if (p < R) h += (p == 0 || k[p] != k[p - 1]) ? 1u : 0u;
  }
  uint32_t total;
  block_inclusive_scan<kRadixThreads>(h, wsum, total);
  if (tid == 0) ws.bheads[b] = total;
}

// Distinct keys, survivors and the request -> group map from tile b; bheads
// holds the heads before each tile.
__device__ __forceinline__ void compact_phase(int R, uint64_t npass, int b, const RadixWs &ws,
                                              int64_t *__restrict__ uk, int32_t *__restrict__ fi,
                                              int32_t *__restrict__ inv,
                                              int64_t *__restrict__ nu_out) {
  __shared__ uint32_t wsum[kRadixThreads / 64 + 1];
  const uint64_t *k = sorted_keys(ws, npass);
  const int32_t *ix = sorted_idx(ws, npass);
  const int tid = threadIdx.x;
  const uint32_t g0 = ws.bheads[b];
  // thread t owns positions [base + t*I, base + t*I + I) so that the scan
  // order is the sorted order
  const int base = b * kTile + tid * kRadixItems;
  uint32_t h = 0;
  for (int e = 0; e < kRadixItems; ++e) {
    int p = base + e;
    if (p < R) h += (p == 0 || k[p] != k[p - 1]) ? 1u : 0u;
  }
  uint32_t total;
  uint32_t incl = block_inclusive_scan<kRadixThreads>(h, wsum, total);
  uint32_t g = g0 + incl - h;
  for (int e = 0; e < kRadixItems; ++e) {
    int p = base + e;
    if (p >= R) break;
    uint64_t kk = k[p];
    const int32_t src = ix[p];
    if (p == 0 || kk != k[p - 1]) {
      if (g < (uint32_t)R) {
        uk[g] = unmap_key(kk);
        fi[g] = src;
        ws.start[g] = p;
      }
      ++g;
    }
    if ((uint32_t)src < (uint32_t)R) inv[src] = (int32_t)(g - 1);
    if (p == R - 1) {
      *nu_out = (int64_t)g;
      if (g <= (uint32_t)R) ws.start[g] = R;
    }
  }
}

// The whole sort path in one persistent launch of G workgroups (all resident
// at once): per pass a
// digit histogram per tile, with more than kDirectTiles tiles an exclusive
// scan of each digit's row over the tiles (rows spread over the wavefronts),
// and the stable scatter; then
// head counts per tile, their scan (workgroup 0), the compaction and the
// group sizes.  Tiles are taken b, b + G, ...; the barrier count is the same
// for every workgroup.
__global__ __launch_bounds__(kRadixThreads) void radix_sort_kernel(
    int R, int nb, RadixWs ws, int64_t *__restrict__ uk, int32_t *__restrict__ fi,
    int32_t *__restrict__ cnt, int32_t *__restrict__ inv, int64_t *__restrict__ nu_out) {
  if (ws.range[2] || (ws.range[3] && !ws.ctl[kCtlFull])) return;   // dense or hash path
  const uint64_t mn = ws.range[0], npass = ws.range[1];
  const int G = gridDim.x, b = blockIdx.x;
  uint32_t k = 0;
  const int wid = b * (kRadixThreads / 64) + (threadIdx.x >> 6), nw = G * (kRadixThreads / 64);
  const int lane = threadIdx.x & 63;
  for (int pass = 0; pass < (int)npass; ++pass) {
    for (int t = b; t < nb; t += G) hist_phase(R, nb, pass, mn, t, ws);
    grid_barrier(ws.ctl, G, k);
    if (nb > kDirectTiles) {
      // each digit's row: exclusive scan over the tiles by one wavefront
      for (int d = wid; d < kBins; d += nw) {
        uint32_t *row = ws.hist + (int64_t)d * nb;
        uint32_t carry = 0;
        for (int c0 = 0; c0 < nb; c0 += 4 * 64) {
          const int i0 = c0 + lane * 4;
          uint32_t v[4], sum = 0;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            v[e] = i0 + e < nb ? row[i0 + e] : 0u;
            sum += v[e];
          }
          uint32_t x = sum;
#pragma unroll
          for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
          }
          uint32_t run = carry + x - sum;
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (i0 + e < nb) {
              row[i0 + e] = run;
              run += v[e];
            }
          carry += __shfl(x, 63, 64);
        }
        if (lane == 0) ws.dtot[d] = carry;
      }
      grid_barrier(ws.ctl, G, k);
    }
    for (int t = b; t < nb; t += G) scatter_phase(R, nb, pass, mn, t, ws);
    grid_barrier(ws.ctl, G, k);
  }
  for (int t = b; t < nb; t += G) heads_phase(R, npass, t, ws);
  grid_barrier(ws.ctl, G, k);
  if (b == 0) block_scan_inplace(ws.bheads, nb);
  grid_barrier(ws.ctl, G, k);
  for (int t = b; t < nb; t += G) compact_phase(R, npass, t, ws, uk, fi, inv, nu_out);
  if (cnt) {
    grid_barrier(ws.ctl, G, k);
    const int64_t n = *nu_out;
    for (int64_t g = (int64_t)b * kRadixThreads + threadIdx.x; g < R && g < n;
         g += (int64_t)G * kRadixThreads)
      cnt[g] = ws.start[g + 1] - ws.start[g];
  }
}

// ---------------------------------------------------------------- host side

static size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

size_t dedup_workspace_bytes(int64_t R) {
  if (R <= kSmallMax) return 0;
  size_t nb = (size_t)((R + kTile - 1) / kTile);
  size_t nvb = (size_t)((R + kDenseBlk - 1) / kDenseBlk);
  size_t s = 0;
  s += 2 * align_up(sizeof(uint64_t) * R);
  s += 2 * align_up(sizeof(int32_t) * R);
  s += 2 * align_up(sizeof(uint64_t) * kPrepMax);
  s += align_up(sizeof(uint64_t) * 5);
  s += align_up(sizeof(uint32_t) * kBins * nb);
  s += align_up(sizeof(uint32_t) * kBins);
  s += align_up(sizeof(uint32_t) * nb);
  s += align_up(sizeof(int32_t) * (R + 1));
  s += align_up(sizeof(uint64_t) * nvb);
  s += align_up(sizeof(uint32_t) * kCtlWords);
  if (R <= kHashRMax) {
    const size_t slots = (size_t)1 << hash_bits(R);
    const size_t buckets = (size_t)1 << bucket_bits(hash_bits(R));
    s += align_up(8 * slots) + 3 * align_up(4 * (slots + 1)) + align_up(4 * buckets);
    s += align_up(8 * buckets * kBucketCap) + align_up(4 * buckets * kBucketCap);
  }
  return s;
}

// Workgroups of radix_sort_kernel that the current device holds at once (0:
// unknown).
static int radix_capacity() {
  static int cache[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
  if (cache[dev]) return cache[dev] > 0 ? cache[dev] : 0;
  int cus = 0, per = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, radix_sort_kernel, kRadixThreads, 0) !=
          hipSuccess ||
      cus <= 0 || per <= 0) {
    cache[dev] = -1;
    return 0;
  }
  cache[dev] = cus * per;
  return cache[dev];
}

hipError_t launch_dedup(const int64_t *keys, int64_t R, int64_t *uk, int32_t *fi, int32_t *cnt,
                        int32_t *inv, int64_t *nu, void *ws, hipStream_t st) {
  if (R <= kSmallMax) {
    hipLaunchKernelGGL(R <= kSmallMax / 2 ? dedup_hash_kernel<kSmallMax / 2>
                                          : dedup_hash_kernel<kSmallMax>,
                       dim3(1), dim3(kSmallThreads), 0, st, keys, (int)R, uk, fi, cnt, inv, nu);
    return hipGetLastError();
  }
  const int capacity = radix_capacity();
  if (capacity <= 0) return hipErrorNotSupported;
  const int nb = (int)((R + kTile - 1) / kTile);
  const int64_t nvb = (R + kDenseBlk - 1) / kDenseBlk;
  char *p = (char *)ws;
  RadixWs w;
  w.keyA = (uint64_t *)p; p += align_up(sizeof(uint64_t) * R);
  w.keyB = (uint64_t *)p; p += align_up(sizeof(uint64_t) * R);
  w.idxA = (int32_t *)p; p += align_up(sizeof(int32_t) * R);
  w.idxB = (int32_t *)p; p += align_up(sizeof(int32_t) * R);
  w.pmin = (uint64_t *)p; p += align_up(sizeof(uint64_t) * kPrepMax);
  w.pmax = (uint64_t *)p; p += align_up(sizeof(uint64_t) * kPrepMax);
  w.range = (uint64_t *)p; p += align_up(sizeof(uint64_t) * 5);
  w.hist = (uint32_t *)p; p += align_up(sizeof(uint32_t) * kBins * nb);
  w.dtot = (uint32_t *)p; p += align_up(sizeof(uint32_t) * kBins);
  w.bheads = (uint32_t *)p; p += align_up(sizeof(uint32_t) * nb);
  w.start = (int32_t *)p; p += align_up(sizeof(int32_t) * (R + 1));
  w.flags = (uint64_t *)p; p += align_up(sizeof(uint64_t) * nvb);
  w.ctl = (uint32_t *)p; p += align_up(sizeof(uint32_t) * kCtlWords);
  w.hbits = R <= kHashRMax ? hash_bits(R) : 0;
  int64_t buckets = 0;
  if (w.hbits) {
    const size_t slots = (size_t)1 << w.hbits;
    buckets = (int64_t)1 << bucket_bits(w.hbits);
    w.hk = (unsigned long long *)p; p += align_up(8 * slots);
    w.hfirst = (uint32_t *)p; p += align_up(4 * (slots + 1));
    w.hcnt = (uint32_t *)p; p += align_up(4 * (slots + 1));
    w.hgid = (int32_t *)p; p += align_up(4 * (slots + 1));
    w.bcnt = (uint32_t *)p; p += align_up(4 * buckets);
    w.bkey = (uint64_t *)p; p += align_up(8 * buckets * kBucketCap);
    w.bslot = (int32_t *)p;
  }
  int Ri = (int)R;
  const int64_t chunks = (R + kPrepChunk - 1) / kPrepChunk;
  const int P = chunks < kPrepMax ? (int)chunks : kPrepMax;
  // (hash path: workgroups that look at the sample and clear the table)
  const int E = !w.hbits ? 0 : 1 + (P / 2 < 32 ? 32 : P / 2);
  hipLaunchKernelGGL(dedup_prep_kernel, dim3(P + E), dim3(kRadixThreads), 0, st, keys, Ri, P, w);
  int64_t rounds = (R + kAggRound - 1) / kAggRound;
  if (rounds > 4096) rounds = 4096;
  hipLaunchKernelGGL(dense_mark_kernel, dim3((unsigned)rounds), dim3(kRadixThreads), 0, st, Ri,
                     P, w);
  // (a workgroup per value block or per bucket)
  hipLaunchKernelGGL(dense_groups_kernel, dim3((unsigned)(nvb > buckets ? nvb : buckets)), dim3(kRadixThreads), 0, st, Ri,
                     w, uk, fi, cnt, nu);
  int64_t ib = (R + 255) / 256;
  if (ib > 8192) ib = 8192;
  hipLaunchKernelGGL(dense_inverse_kernel, dim3((unsigned)ib), dim3(256), 0, st, Ri, w, inv);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  int G = nb < kRadixGridMax ? nb : kRadixGridMax;
  if (G > capacity) G = capacity;
  // an ordinary launch: G is at most what the device holds at once, so every
  // workgroup becomes resident (a cooperative launch would only add ~17 us of
  // set-up to every call, the dense path's included)
  hipLaunchKernelGGL(radix_sort_kernel, dim3(G), dim3(kRadixThreads), 0, st, Ri, nb, w, uk, fi,
                     cnt, inv, nu);
  return hipGetLastError();
}

}  // namespace hs
