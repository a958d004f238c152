// Steps 3 and 4 for bf16 and fp8-e4m3 corpora: score every distinct query
// against the corpus on the matrix cores and keep the k best rows per query
// and corpus slice.
//
// HeraSys runs one retrieval per fused node (Sec. 3.3 (I)) and batches ready
// nodes of the same type (Appendix A, batching constraint); a retrieval
// node's result is its Top-K chunks (Eq. 2 parameters; Sec. 4.1 workloads).
// Here the batch is the n_u distinct queries and the retrieval is an exact
// inner product, s[u, c] = scale_c * sum_j Q[u, j] C[c, j], accumulated in
// fp32.
//
// Work decomposition: a persistent grid, one workgroup of four waves per CU.
// A work item is (query tile of 128, corpus slice); a slice is a run of
// tiles of 384 corpus rows.  Wave w owns rows [96w, 96w + 96) of a tile
// against all 128 queries: 3 x 4 blocks of v_mfma_f32_32x32x16_bf16 with the
// 192 fp32 accumulators in AGPRs (the rest of the register file holds two
// sets of operand fragments and the epilogue's working set without spills).
// Items of one slice get consecutive logical ids on one XCD, so the query
// tiles that read the same corpus rows share that XCD's L2.
//
// Operand staging: both operands stream through a ring of LDS stages (two
// for bf16, three for fp8), one K range of 64 per stage, written by
// buffer_load ... lds (asynchronous copies from global memory straight into
// LDS, no registers).  A bf16 corpus row contributes one 128-byte line per
// stage (fp8: 64 bytes).  Rows are stored in LDS as 16-byte pieces with an
// XOR swizzle so that fragment reads (ds_read_b128) are bank-conflict free.
// The query rows, and the corpus when it is given in the tiled layout, are
// kept in global memory in exactly that LDS order (tile_queries_kernel,
// tile_corpus_kernel), zero-padded past n_u, N and d, so every copy reads
// 1 KiB of consecutive bytes; a row-major corpus is copied as row pieces
// through a descriptor whose range covers the tile's valid rows (rows past N
// read as zeros).  Either way there are no bounds branches and no access
// outside the operands.  Inside one MFMA the K order is free as long as
// both operands agree; each lane takes the K slice that makes its fp8 corpus
// piece one 16-byte read.
//
// Synchronisation per stage: a wave copies, and alone reads, its own 96
// corpus rows of a stage, so it refills them as soon as its own reads of
// the stage's slot are complete (after the first of the four MFMA steps),
// without a barrier.  The query rows are shared by the four waves: after the
// third step the waves wait for their own copies of the next stage
// (s_waitcnt vmcnt with the number of younger copies), then one barrier,
// then the query rows of the stage ns ahead and the next stage's first
// fragments, overlapped with the last step.  The fences of __syncthreads are
// not used because they would wait for every copy in flight.
//
// Top-k (fused, scores never reach memory), per tile: rows past N are
// masked and each lane screens its 16-score row blocks by their maximum
// (fp8: accumulator x row scale) against the query's threshold; only the
// blocks that reach it are examined, and their scores at or above it are
// appended to a small per-query LDS queue (one atomic per lane and block
// reserves the slots), merged into the query's sorted k-list when a queue
// is due.  Thresholds come from lower bounds of the query's final k-th best
// score: the slice's own k-list; a seed, the k-th largest of the lane maxima
// of a first pass over the first tiles of the slices (at most 128 of them:
// a sample spread over the corpus); the order statistics of the slices
// finished so far; and the
// largest bound any slice of the query has published so far (a per-query
// array in the workspace, read asynchronously with each tile's copies).
// Keys order by (score desc, row asc): ties go to the lower
// corpus row independently of tile, slice or lane.
#include <mutex>
#include <type_traits>

#include "score_lists.h"

namespace hs {

typedef __bf16 bf16x8m __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2m __attribute__((ext_vector_type(2)));
typedef float f32x16m __attribute__((ext_vector_type(16)));

constexpr int kMW = 4;                   // waves per workgroup (one per SIMD)
constexpr int kMT = kMW * 64;            // threads
constexpr int kMRB = 3;                  // 32-row blocks per wave
constexpr int kMQB = 4;                  // 32-query blocks per tile
constexpr int kMNC = kMW * 32 * kMRB;    // 384 corpus rows per tile
constexpr int kMKC = 64;                 // K per ring stage (four 16-deep MFMA steps)
constexpr int kMVals = 16 * kMRB;        // scores per lane and query per tile
constexpr int kMLanesQ = kMW * 2;        // lanes holding one query in a tile

// Seed pass sample: the lane maxima of the first T tiles of every slice (at
// most kSeedMax of them per query).
//
// A sample of M = 384 S T rows lets about N k / M rows of the corpus pass its
// bound, each an insertion into a list, while every sampled tile is computed
// twice.
// - Short slices (n < 4 S, n = tiles per slice): the list of a slice of n rows
//   hardly ever bounds better than the seed of T S, so a workgroup's 128
//   queries take in proportion to k n / (S T) insertions, and T tiles of nch
//   stages plus the maxima (about 1.6 stages): T^2 = c k n / (S (nch + 1.6)).
//   c = 6, measured: 960 queries, 500,009 x 400 fp8, k = 50 (n = 40, S = 32),
//   seed pass + selection + main pass: T = 2 (as before) 1,042 us, c = 6 (T =
//   7) 805, c = 12 811, c = 25 827, c = 50 904; 329 queries, 1M x 768 bf16, k =
//   10 (n = 30, S = 85): T = 1 (c = 6) 709 us, T = 2 715; 336 queries, 333,333
//   x 1,000, k = 20 (n = 10, S = 85): T = 1 430 us, T = 2 447.
// - Longer slices: their own lists and the bounds they publish take over.  One
//   tile for k <= 48 (8 or 16 changed nothing at k = 32, n = 651, S = 16); for
//   larger k the lists fill late, and T grows to 20 within 1/16 of the slice.
// The maxima share the lists' bytes, 32 T against 8 k per query and slice, and T
// stays within k / 4 for short slices: many queries run as short slices, and
// their lists are what a workspace is sized by.
constexpr int kSeedMax = 16384;
constexpr int kSeedTilesMax = 20;
__host__ __device__ __forceinline__ int seed_tiles(int k, int64_t ntiles, int64_t S, int nch) {
  if (S < 1) return 1;
  const int n = (int)(ntiles / S);
  int t = 1;
  if (n < 4 * S) {
    // the integer whose square is nearest below twice-rounded T^2 (no square
    // root: host and device must agree)
    const int64_t num = 60 * (int64_t)k * n, den = S * (10 * (int64_t)nch + 16);
    while (t < kSeedTilesMax && (int64_t)(2 * t + 1) * (2 * t + 1) * den <= 4 * num) ++t;
    if (t > n / 2) t = n / 2;
    if (t > k / 4) t = k / 4;   // (within the lists' bytes)
  } else if (k > 48) {
    t = n / 16;
  }
  const int room = (int)(kSeedMax / (S * kMLanesQ));
  if (t > room) t = room;
  if (t > kSeedTilesMax) t = kSeedTilesMax;
  return t < 1 ? 1 : t;
}
// Slices that take part in the seed sample: one in every seed_stride(S), at
// most kSeedSlices of them.  A single query tile runs as up to 256 slices, and
// the seed pass (one tile per workgroup, all at once) then reads that many
// tiles of the corpus; half of them are as good a sample for the seed.
constexpr int kSeedSlices = 128;
__host__ __device__ __forceinline__ int64_t seed_stride(int64_t S) {
  return S > kSeedSlices ? (S + kSeedSlices - 1) / kSeedSlices : 1;
}
constexpr int kMRowsW = 32 * kMRB;       // rows per wave in a tile
constexpr int kMSS = kMNC + 128 - kMRowsW;  // row-scale slot stride (floats): the
                                         // last wave's two 64-row copies overhang
constexpr int kMGts = kMMQ + 32;         // shared-threshold slot stride (entries): the
                                         // last wave's 64-entry copy overhangs

template <bool FP8>
struct Geo {
  static constexpr int esz = FP8 ? 1 : 2;
  static constexpr int arow = kMKC * esz;         // bytes of one corpus row per stage
  static constexpr int abytes = kMNC * arow;
  static constexpr int brow = kMKC * 2;           // bytes of one query row per stage
  static constexpr int bbytes = kMMQ * brow;
  static constexpr int stage = abytes + bbytes;
  static constexpr int ns = FP8 ? 3 : 2;          // ring stages
  static constexpr int nsc = FP8 ? ns + 1 : 0;    // row-scale slots (tiles in flight)
  static constexpr int ngt = ns + 1;              // shared-threshold slots (tiles in flight)
  static constexpr int adma = abytes / 1024 / kMW;  // 1 KiB copies per wave and stage
  static constexpr int bdma = bbytes / 1024 / kMW;
  static constexpr int ldma = adma + bdma;        // copies per wave and stage (scales aside)
  static constexpr int apieces = arow / 16;       // 16-byte pieces of a corpus row stage
  static constexpr int bpieces = brow / 16;
};

// Order statistics a finished item publishes per query: level l holds the
// ordered score of the ceil(k / r)-th best key of the slice's final list,
// r = 2^l, l < kLvl (0 where the list is shorter).  If r slices publish level-l
// values of at least x, those slices hold r * ceil(k / r) >= k distinct
// rows scoring at least x, so the r-th largest level-l value over the
// slices is a lower bound of the query's k-th best score.  An item starts
// by raising the query's shared threshold to the best such bound over the
// slices finished so far.
// Long items with kWaveLists also publish, and raise their queries' thresholds,
// while they run: after kLvlFirst tiles and whenever that number has doubled.
// Slices that run at the same time then share one bound instead of each filling
// a list of its own.  A raise reads 5 S words per query, so where items follow in
// later rounds anyway, and start from what the finished slices published, it is
// done only for up to kLvlSlices slices.  Without -> with it, k = 100 unless said:
// 20M x 768 fp8, 2,100 queries (15 slices of 3,472 tiles, one round) 69.2 -> 64.7
// ms, but 2,190 queries (71 slices of 733, five rounds) 70.7 -> 72.1; 5M fp8, 3,000
// queries (32 slices, three rounds) 25.4 -> 25.0, 9,000 (18, five) 74.1 -> 73.4;
// k = 40, 1,100 queries (142, five) 9.4 -> 9.8; 4M x 512 bf16, k = 64, 2,190
// queries (71, five) 10.7 -> 11.6.
constexpr int kLvl = 5;
constexpr int kLvlFirst = 32, kLvlSlices = 48;
constexpr int kMWarmBytes = kMW * kMMQ * 4;   // per-wave warm-up minima (alias the queue)
static_assert(kMWarmBytes <= kMMQ * kMQcap * 8, "warm-up minima fit in the queue");

// Where the k-lists of an item live.
// kLdsLists: in LDS, merged by a thread per query as soon as a queue is half
//   full; for every k that fits beside the ring (18 or 19).
// kTailLists: in the global partial buffer with the last kMTail entries in LDS,
//   merged by a thread per query when a queue is full; up to k = kTailMax.
// kWaveLists: in the global partial buffer alone, merged by a wave per query,
//   whose cost is a read of the list whatever the number of keys, so the queues
//   take the tail's place in LDS (24 keys).
// The line between the last two, measured: 20M x 768 fp8, k = 100, 75.0 ms with
// tails, 65.4-67.6 without; 500,009 x 400 fp8, k = 50, 885 us either way; 4M x
// 1,024 bf16, k = 32, 79.0 ms either way; 333,333 x 1,000 bf16, k = 20, 460 us
// with tails, 472 without (an end of item of 32 queries per wave).
constexpr int kTailLists = 0, kLdsLists = 1, kWaveLists = 2;
constexpr int kTailMax = 32;
template <int LISTS>
constexpr int kQcap = LISTS == kWaveLists ? 24 : kMQcap;   // queue slots per query
static_assert(kQcap<kWaveLists> * 8 == kMQcap * 8 + kMTail * 8, "the same LDS as with tails");

__host__ __device__ constexpr int mfma_lds_bytes(bool fp8, bool lds_lists, int k) {
  return (fp8 ? Geo<true>::ns * Geo<true>::stage + Geo<true>::nsc * kMSS * 4 +
                    Geo<true>::ngt * kMGts * 4
              : Geo<false>::ns * Geo<false>::stage + Geo<false>::ngt * kMGts * 4) +
         kMMQ * kMQcap * 8 + kMMQ * (4 + 4 + 4 + 8 + 4) + 16 +
         (lds_lists ? kMMQ * k * 8 : kMMQ * kMTail * 8);
}
// k-lists of up to kMTail entries always fit in LDS, so global lists (which
// keep kMTail entries in LDS) always have k > kMTail; and the global-list
// layout fits for every k.
static_assert(mfma_lds_bytes(false, true, kMTail) <= 160 * 1024 &&
                  mfma_lds_bytes(true, true, kMTail) <= 160 * 1024,
              "short k-lists fit in LDS");
static_assert(mfma_lds_bytes(false, false, 0) <= 160 * 1024 &&
                  mfma_lds_bytes(true, false, 0) <= 160 * 1024,
              "global-list layout fits in LDS");

// Warm-up groups per lane and query: the kMVals scores a lane holds for one
// query are cut into gpl groups so that kMLanesQ * gpl >= k group maxima
// exist.  0 = no warm-up (k too large for one tile).
__host__ __device__ constexpr int mwarm_groups(int k) {
  int g = 1;
  while (g <= kMVals && kMLanesQ * g < k) g <<= 1;
  return g <= kMVals ? g : 0;
}

__device__ __forceinline__ void cvt8_fp8_bf16(uint32_t lo, uint32_t hi, bf16x8m &out) {
  // exact e4m3 -> bf16 (every e4m3 value is representable in bf16)
  bf16x2m a = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, 1.0f, false);
  bf16x2m b = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, 1.0f, true);
  bf16x2m c = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, 1.0f, false);
  bf16x2m e = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, 1.0f, true);
  uint4 v = make_uint4(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b),
                       __builtin_bit_cast(uint32_t, c), __builtin_bit_cast(uint32_t, e));
  out = __builtin_bit_cast(bf16x8m, v);
}

// Fragments of one half stage (two 16-deep steps).  The K order inside a
// stage is permuted identically for both operands: step t in 0..3 and lane
// half h take elements [32h + 8t, 32h + 8t + 8), so that one 16-byte fp8
// corpus piece feeds two consecutive steps.
template <bool FP8, int NQB>
struct Frag {
  // bf16: A pieces [step][rb]; fp8: raw 16-byte pieces [rb] (both steps)
  uint4 a[FP8 ? 1 : 2][kMRB];
  uint4 b[2][NQB];
  // ds_read_b128 operations that fill one Frag
  static constexpr int na = (FP8 ? 1 : 2) * kMRB;
  static constexpr int nreads = na + 2 * NQB;
};

// Read k (0 <= k < nreads) of half u of the stage in ring slot `st`: the A
// pieces first (step-major), then the B pieces (step-major).
template <bool FP8, int NQB>
__device__ __forceinline__ void read_frag_piece(Frag<FP8, NQB> &f, const unsigned char *st,
                                                int wv, int c, int h, int u, int k) {
  using G = Geo<FP8>;
  using F = Frag<FP8, NQB>;
  if (k < F::na) {
    const int s = FP8 ? 0 : k / kMRB, rb = k % kMRB;
    const int slot = FP8 ? swz_slot<G::apieces>(2 * h + u, c)
                         : swz_slot<G::apieces>(4 * h + 2 * u + s, c);
    const unsigned char *abase = st + (wv * 32 * kMRB + c) * G::arow;
    f.a[s][rb] = *reinterpret_cast<const uint4 *>(abase + rb * 32 * G::arow + slot * 16);
  } else {
    const int s = (k - F::na) / NQB, qb = (k - F::na) % NQB;
    const int slot = swz_slot<G::bpieces>(4 * h + 2 * u + s, c);
    const unsigned char *bbase = st + G::abytes + c * G::brow;
    f.b[s][qb] = *reinterpret_cast<const uint4 *>(bbase + qb * 32 * G::brow + slot * 16);
  }
}

// Read half u of the stage in ring slot `st`.
template <bool FP8, int NQB>
__device__ __forceinline__ void read_frags(Frag<FP8, NQB> &f, const unsigned char *st, int wv,
                                           int c, int h, int u) {
#pragma unroll
  for (int k = 0; k < Frag<FP8, NQB>::nreads; ++k) read_frag_piece<FP8>(f, st, wv, c, h, u, k);
}

// Redefine the second step's operands of a half stage in place (no code):
// MFMAs that use them cannot then be moved above a preceding barrier.
typedef unsigned u32x4m __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void pin_u4(uint4 &v) {
  u32x4m t = __builtin_bit_cast(u32x4m, v);
  asm volatile("" : "+v"(t));
  v = __builtin_bit_cast(uint4, t);
}
template <bool FP8, int NQB>
__device__ __forceinline__ void pin_step1(Frag<FP8, NQB> &f) {
#pragma unroll
  for (int rb = 0; rb < kMRB; ++rb) pin_u4(f.a[FP8 ? 0 : 1][rb]);
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb) pin_u4(f.b[1][qb]);
}

// One 16-deep MFMA step over the wave's kMRB x NQB blocks, with op(i) issued after
// the i-th matrix instruction, in its shadow (a scheduling barrier after each keeps
// the order).
template <bool FP8, bool ZERO, int NQB, typename Op>
__device__ __forceinline__ void mfma_step_il(f32x16m (&acc)[kMRB][NQB], const Frag<FP8, NQB> &f,
                                             int s, Op &&op) {
  bf16x8m av[kMRB];
#pragma unroll
  for (int rb = 0; rb < kMRB; ++rb) {
    if constexpr (FP8) {
      const uint4 v = f.a[0][rb];
      if (s == 0) cvt8_fp8_bf16(v.x, v.y, av[rb]);
      else cvt8_fp8_bf16(v.z, v.w, av[rb]);
    } else {
      av[rb] = __builtin_bit_cast(bf16x8m, f.a[s][rb]);
    }
  }
  const f32x16m zero = {};
#pragma unroll
  for (int i = 0; i < kMRB * NQB; ++i) {
    const int rb = i / NQB, qb = i % NQB;
    acc[rb][qb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
        av[rb], __builtin_bit_cast(bf16x8m, f.b[s][qb]), ZERO ? zero : acc[rb][qb], 0, 0, 0);
    op(i);
    __builtin_amdgcn_sched_barrier(0);
  }
}

template <bool FP8, int LISTS>
__device__ __forceinline__ MLds carve_mlds(unsigned char *p, int k) {
  using G = Geo<FP8>;
  MLds L;
  L.ring = p; p += G::ns * G::stage;
  L.sscale = reinterpret_cast<float *>(p); p += G::nsc * kMSS * 4;
  L.gtl = reinterpret_cast<uint32_t *>(p); p += G::ngt * kMGts * 4;
  L.queue = reinterpret_cast<uint64_t *>(p);
  L.warm = reinterpret_cast<float *>(p);   // (used before the queue in an epilogue)
  p += kMMQ * kQcap<LISTS> * 8;
  L.lmin = reinterpret_cast<uint64_t *>(p); p += kMMQ * 8;
  L.qcount = reinterpret_cast<int32_t *>(p); p += kMMQ * 4;
  L.thr0 = reinterpret_cast<float *>(p); p += kMMQ * 4;
  L.thr = reinterpret_cast<float *>(p); p += kMMQ * 4;
  L.pub = reinterpret_cast<uint32_t *>(p); p += kMMQ * 4;
  L.flags = reinterpret_cast<int32_t *>(p); p += 16;
  L.lists = LISTS == kLdsLists ? reinterpret_cast<uint64_t *>(p) : nullptr;
  L.tail = LISTS == kTailLists ? reinterpret_cast<uint64_t *>(p) : nullptr;
  (void)k;
  return L;
}

// Keep t (descending) the R largest of the values offered so far.
template <int R>
__device__ __forceinline__ void offer_top(uint32_t (&t)[R], uint32_t x) {
#pragma unroll
  for (int u = 0; u < R; ++u) {
    const uint32_t hi = t[u] > x ? t[u] : x;
    x = t[u] > x ? x : t[u];
    t[u] = hi;
  }
}

// Best lower bound of a query's k-th best score from the order statistics
// its finished slices published: the largest over levels l of the 2^l-th
// largest level-l value over the S slices (0 if none).  lv = the query's
// [kLvl][S] row; device-scope loads (other workgroups publish), issued 8
// slices x kLvl levels at a time.
__device__ __forceinline__ uint32_t level_bound(const uint32_t *lv, int S) {
  static_assert(kLvl == 5, "one top buffer per level");
  uint32_t t0[1] = {0u}, t1[2] = {0u, 0u}, t2[4] = {}, t3[8] = {}, t4[16] = {};
  for (int s0 = 0; s0 < S; s0 += 8) {
    uint32_t v[kLvl][8];
#pragma unroll
    for (int l = 0; l < kLvl; ++l)
#pragma unroll
      for (int u = 0; u < 8; ++u)
        v[l][u] = s0 + u < S ? __hip_atomic_load(lv + l * S + s0 + u, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT)
                             : 0u;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      offer_top(t0, v[0][u]);
      offer_top(t1, v[1][u]);
      offer_top(t2, v[2][u]);
      offer_top(t3, v[3][u]);
      offer_top(t4, v[4][u]);
    }
  }
  uint32_t b = t0[0];
  b = t1[1] > b ? t1[1] : b;
  b = t2[3] > b ? t2[3] : b;
  b = t3[7] > b ? t3[7] : b;
  b = t4[15] > b ? t4[15] : b;
  return b;
}

// An opaque copy of a lane value: values derived from it are recomputed
// where they are used instead of being hoisted (and spilled) by the compiler.
__device__ __forceinline__ int opaque(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// Merge the queued keys into the lists in the global partial buffer, a wave per
// query (kWaveLists).  The list is sorted in descending order; L.lmin[q] holds its
// length (what lies beyond it is not valid until the end of the item).  A list entry
// moves down by the number of new keys above it, a new key goes to its rank
// among the new keys plus the number of entries above it.  The list is read in
// blocks of 64 entries from its end, up to the block whose first entry is above
// every new key.  Entries and keys below the query's threshold cannot be in the
// result and are dropped.
//
// One thread per query inserted its keys one after the other before, climbing
// the list in windows of 8 dependent global reads, and the wave took as long as
// its longest thread: 174,000 cycles per round of merges, 12.5 % of the main
// pass over 20M fp8 rows, k = 100, with queues of 8 (the shader clock read around
// the rounds in a copy of the kernel).
__device__ __forceinline__ uint64_t lane_key(uint64_t x, int f) {
  const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)x, f);
  const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), f);
  return ((uint64_t)hi << 32) | lo;
}
//
// A wave has up to 32 queries (q = wave + 4 j); lane j holds the state of query
// j, and the next query's keys and list block are on their way while one is
// merged.  gt: shared thresholds of the item's queries.
__device__ __forceinline__ void merge_lists(const MLds &L, const MfmaArgs &a, const MItem &it,
                                            const uint32_t *gt) {
  constexpr int QC = kQcap<kWaveLists>;
  const int tid = opaque(threadIdx.x);   // (nothing below is worth a register outside)
  const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int k = a.k, mine = wv + kMW * lane;
  const bool own = lane < kMMQ / kMW && mine < it.qvalid;
  const float ninf = -__builtin_inff();
  int cnt = own ? L.qcount[mine] : 0;
  cnt = cnt < QC ? cnt : QC;
  int fill = own ? (int)L.lmin[mine] : 0;
  const float th0 = own ? L.thr[mine] : ninf;
  uint32_t tho = th0 > ninf ? ord_score(th0) : 0u;
  if (own && gt[mine] > tho) tho = gt[mine];
  uint64_t todo = __builtin_amdgcn_ballot_w64(cnt > 0);
  if (todo == 0ull) return;
  float kth = ninf;   // lane j: score of query j's k-th key, if it has one now
  uint64_t *const lists = a.part + ((int64_t)it.qbase * it.S + it.s) * k;
  auto list = [&](int j) { return lists + (int64_t)(wv + kMW * j) * it.S * k; };
  auto fetch = [&](int j, uint64_t &x, uint64_t &v) __attribute__((always_inline)) {
    const int n = __builtin_amdgcn_readlane(cnt, j), f = __builtin_amdgcn_readlane(fill, j);
    x = lane < n ? L.queue[(wv + kMW * j) * QC + lane] : 0ull;
    const int i = ((f - 1) & ~63) + lane;
    v = f > 0 && i < f ? list(j)[i] : 0ull;
  };
  int j = __builtin_ctzll(todo);
  uint64_t x, v;
  fetch(j, x, v);
  for (;;) {
    todo &= todo - 1ull;
    const int jn = todo ? __builtin_ctzll(todo) : j;
    const int n = __builtin_amdgcn_readlane(cnt, j), f0 = __builtin_amdgcn_readlane(fill, j);
    const uint32_t drop = (uint32_t)__builtin_amdgcn_readlane((int)tho, j);
    uint64_t xn = 0ull, vn = 0ull;
    if (todo) fetch(jn, xn, vn);
    uint64_t *l = list(j);
    if ((uint32_t)(x >> 32) < drop) x = 0ull;
    int pos = 0;   // the place of this lane's new key
    for (int f = 0; f < n; ++f) pos += lane_key(x, f) > x ? 1 : 0;
    uint64_t last = 0ull;   // the lane that holds the k-th key: that key
    int live = 0;
    for (int b = f0 > 0 ? (f0 - 1) & ~63 : -1; b >= 0; b -= 64) {
      const int i = b + lane;
      if (b != ((f0 - 1) & ~63)) v = l[i];
      if ((uint32_t)(v >> 32) < drop) v = 0ull;
      int shift = 0;
      for (int f = 0; f < n; ++f) {
        const uint64_t y = lane_key(x, f);
        const int above = __builtin_popcountll(__builtin_amdgcn_ballot_w64(v > y));
        pos += lane == f ? above : 0;
        shift += y > v ? 1 : 0;
      }
      live += __builtin_popcountll(__builtin_amdgcn_ballot_w64(v != 0ull));
      if (v != 0ull) {
        const int p = i + shift;
        if (shift > 0 && p < k) l[p] = v;
        if (p == k - 1) last = v;
      }
      if (__builtin_amdgcn_readfirstlane(v != 0ull && shift == 0 ? 1 : 0)) {
        pos += b;   // the entries of the earlier blocks are above every new key
        live += b;
        break;
      }
    }
    if (x != 0ull) {
      if (pos < k) l[pos] = x;
      if (pos == k - 1) last = x;
    }
    live += __builtin_popcountll(__builtin_amdgcn_ballot_w64(x != 0ull));
    const uint64_t has = __builtin_amdgcn_ballot_w64(last != 0ull);   // (at most one lane)
    const float lk = has ? unord_score((uint32_t)(lane_key(last, __builtin_ctzll(has)) >> 32)) : ninf;
    if (lane == j) {
      fill = live < k ? live : k;
      kth = lk;
    }
    if (!todo) break;
    j = jn;
    x = xn;
    v = vn;
  }
  if (cnt > 0) {
    L.qcount[mine] = 0;
    L.lmin[mine] = (uint64_t)fill;
    if (kth > th0) {
      L.thr[mine] = kth;
      publish_thr(L, a, it, mine, kth);
    }
  }
}

// The same, outside the tile epilogue.  Lists that are all empty (short
// slices, whose only merge is that at their end) take no list reads, and half a
// wave per query ranks its keys by counting.
__device__ __forceinline__ void merge_any(const MLds &L, const MfmaArgs &a, const MItem &it,
                                          const uint32_t *gt) {
  constexpr int QC = kQcap<kWaveLists>;
  static_assert(QC <= 32 && QC % 8 == 0, "a key per lane of half a wave, read by eights");
  static_assert(QC <= kTailMax, "these lists are longer than a queue");
  const int tid = opaque(threadIdx.x), lane = tid & 63, wv = tid >> 6, e = lane & 31;
  const int mine = wv + kMW * e;
  if (__builtin_amdgcn_ballot_w64(mine < it.qvalid && L.lmin[mine] != 0ull)) {
    merge_lists(L, a, it, gt);
    return;
  }
  for (int j = lane >> 5; j < kMMQ / kMW; j += 2) {
    const int q = wv + kMW * j;
    const float th = L.thr[q];
    uint32_t drop = gt[q];
    uint64_t x = e < QC ? L.queue[q * QC + e] : 0ull;
    int n = q < it.qvalid ? L.qcount[q] : 0;
    n = n < QC ? n : QC;
    const uint32_t to = th > -__builtin_inff() ? ord_score(th) : 0u;
    drop = to > drop ? to : drop;
    if (e >= n || (uint32_t)(x >> 32) < drop) x = 0ull;
    int pos = 0;
    for (int f = 0; __builtin_amdgcn_ballot_w64(f < n); f += 8) {
      uint64_t y[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) y[u] = L.queue[q * QC + f + u];
#pragma unroll
      for (int u = 0; u < 8; ++u) pos += f + u < n && y[u] > x ? 1 : 0;
    }
    const uint64_t mask = __builtin_amdgcn_ballot_w64(x != 0ull);
    const int live = __builtin_popcount((uint32_t)(lane < 32 ? mask : mask >> 32));
    // (fewer keys than k: no threshold yet)
    if (x != 0ull) a.part[((int64_t)(it.qbase + q) * it.S + it.s) * a.k + pos] = x;
    if (e == 0 && n > 0) {
      L.lmin[q] = (uint64_t)live;
      L.qcount[q] = 0;
    }
  }
}

// Order statistics of the wave's lists so far (global lists): eight queries at
// a time, a lane per query and level.
__device__ __forceinline__ void publish_levels_wave(const MLds &L, const MfmaArgs &a,
                                                    const MItem &it) {
  const int tid = opaque(threadIdx.x), lane = tid & 63, wv = tid >> 6, l = lane & 7;
  const int p = l < kLvl ? ((a.k + (1 << l) - 1) >> l) - 1 : a.k;   // ceil(k / 2^l) - 1
#pragma unroll
  for (int j0 = 0; j0 < kMMQ / kMW; j0 += 8) {
    const int j = j0 + (lane >> 3);
    const int q = wv + kMW * j;
    if (q < it.qvalid && p < (int)L.lmin[q])
      __hip_atomic_store(
          a.lvl + (int64_t)(it.qbase + q) * kLvl * it.S + l * it.S + it.s,
          (uint32_t)(a.part[((int64_t)(it.qbase + q) * it.S + it.s) * a.k + p] >> 32),
          __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Raise query t's threshold to the bound of the order statistics published so
// far by all its slices.
__device__ __forceinline__ void raise_by_levels(const MLds &L, const MfmaArgs &a, const MItem &it,
                                                int t) {
  const uint32_t b = level_bound(a.lvl + (int64_t)(it.qbase + t) * kLvl * it.S, (int)it.S);
  if (b) {
    L.thr[t] = fmaxf(L.thr[t], unord_score(b));
    publish_thr(L, a, it, t, L.thr[t]);
  }
}

// Keep the accumulators in AGPRs and make the compiler forget any VGPR copy
// of them: the epilogue then reads each element where it is used instead of
// holding all 256 in VGPRs across its loops.
template <int NQB>
__device__ __forceinline__ void pin_acc(f32x16m (&acc)[kMRB][NQB]) {
#pragma unroll
  for (int rb = 0; rb < kMRB; ++rb)
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) asm volatile("" : "+a"(acc[rb][qb]));
}

// NaN for the scores of rows past N (only for a tile that reaches past N).
template <int NQB>
__device__ __forceinline__ void mask_tail(f32x16m (&acc)[kMRB][NQB], int lim0) {
  if (lim0 < 32 * kMRB) {   // some of this lane's rows are past N
    const float nan = __builtin_nanf("");
#pragma unroll
    for (int rb = 0; rb < kMRB; ++rb)
#pragma unroll
      for (int qb = 0; qb < NQB; ++qb)
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (rb * 32 + 8 * (i >> 2) + (i & 3) >= lim0) acc[rb][qb][i] = nan;
    pin_acc(acc);
  }
}

// Turns the tile's accumulators into scores in place, once per tile: the fp8
// row scale applied, NaN for rows past N (NaN fails every >= test and fmaxf
// ignores it).  Accumulator element (rb, qb, i) of a lane is row
// rb * 32 + 8 * (i / 4) + i % 4 counted from the lane's first row; `lim0` =
// number of valid rows from there.  Everything after reads the accumulators
// directly.
template <bool FP8, int NQB>
__device__ __forceinline__ void finish_scores(f32x16m (&acc)[kMRB][NQB], const float *ssc_lane,
                                              int lim0) {
  if constexpr (FP8) {
#pragma unroll
    for (int rb = 0; rb < kMRB; ++rb)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        // (an opaque offset keeps the compiler from loading all 48 scales
        // ahead of the multiplies)
        const float4 s4 = *reinterpret_cast<const float4 *>(ssc_lane + opaque(rb * 32 + 8 * j));
#pragma unroll
        for (int qb = 0; qb < NQB; ++qb) {
          acc[rb][qb][4 * j + 0] *= s4.x;
          acc[rb][qb][4 * j + 1] *= s4.y;
          acc[rb][qb][4 * j + 2] *= s4.z;
          acc[rb][qb][4 * j + 3] *= s4.w;
          asm volatile("" : "+a"(acc[rb][qb]));
        }
      }
  }
  mask_tail(acc, lim0);
}

// The 16 fp8 row scales of row block rb of this lane (rows rb * 32 + 8 * (i /
// 4) + i % 4 from the lane's first row), or ones when the accumulators are
// already scaled.
template <bool FP8>
__device__ __forceinline__ void row_scales(float (&s16)[16], const float *ssc_lane, int rb,
                                           bool ones) {
  if constexpr (FP8) {
    if (!ones) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float4 s4 = *reinterpret_cast<const float4 *>(ssc_lane + rb * 32 + 8 * j);
        s16[4 * j + 0] = s4.x;
        s16[4 * j + 1] = s4.y;
        s16[4 * j + 2] = s4.z;
        s16[4 * j + 3] = s4.w;
      }
      return;
    }
  }
#pragma unroll
  for (int i = 0; i < 16; ++i) s16[i] = 1.0f;
}


// Warm-up: per query, the smallest of this lane's group maxima (groups of
// SPAN consecutive scores), combined over the two lane halves and stored per
// wave.
template <int SPAN, int NQB>
__device__ __forceinline__ void warm_minima(const MLds &L, f32x16m (&acc)[kMRB][NQB], int wv,
                                            int c, int h) {
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb) {
    float mn = __builtin_inff(), m = -__builtin_inff();
#pragma unroll
    for (int rb = 0; rb < kMRB; ++rb)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        m = fmaxf(m, acc[rb][qb][i]);
        if ((rb * 16 + i + 1) % SPAN == 0) {
          mn = fminf(mn, m);
          m = -__builtin_inff();
        }
      }
    mn = fminf(mn, __shfl_xor(mn, 32));
    if (h == 0) L.warm[wv * kMMQ + qb * 32 + c] = mn;
  }
}

// Seed pass: each lane's best score of the tile for each of its queries, as
// an ordered score, to lmax[((query * S + slice) * T + t) * 8 + lane-of-query]
// for the slice's t-th sampled tile (T tiles per slice).  These
// are scores of distinct corpus rows, so the k-th largest of all of a
// query's lane maxima (over all slices) is a lower bound of its k-th best
// score over the whole corpus.
template <bool FP8, int NQB>
__device__ __forceinline__ void mtile_lane_maxima(const MfmaArgs &a, const MItem &it,
                                                  f32x16m (&acc)[kMRB][NQB], int row0,
                                                  const float *ssc, int t) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int c = lane & 31, h = lane >> 5;
  const int lrow = wv * 32 * kMRB + 4 * h;
  const int lim0 = (int)a.N - row0 - lrow;
  const float *ssc_lane = FP8 ? ssc + lrow : nullptr;
  pin_acc(acc);
  finish_scores<FP8>(acc, ssc_lane, lim0);
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb) {
    float m = -__builtin_inff();
#pragma unroll
    for (int rb = 0; rb < kMRB; ++rb)
#pragma unroll
      for (int i = 0; i < 16; ++i) m = fmaxf(m, acc[rb][qb][i]);
    const int ql = qb * 32 + c;
    if (ql < it.qvalid)
      a.lmax[(((int64_t)(it.qbase + ql) * it.S + it.s) * it.T + t) * kMLanesQ + wv * 2 + h] =
          m > -__builtin_inff() ? ord_score(m) : 0u;
  }
}

// Top-k epilogue of one tile.  row0 = corpus row of the tile's first row;
// ssc = row scales of the tile (fp8).
template <bool FP8, int LISTS, int NQB>
__device__ __forceinline__ void mtile_epilogue(const MLds &L, const MfmaArgs &a, const MItem &it,
                                               f32x16m (&acc)[kMRB][NQB],
                                               float (&thr_r)[kMQB], int &epoch, int row0,
                                               const float *ssc, const uint32_t *gt,
                                               bool first) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int c = lane & 31, h = lane >> 5;
  const float ninf = -__builtin_inff();
  const int lrow = wv * 32 * kMRB + 4 * h;   // this lane's first row in the tile
  const int lim0 = (int)a.N - row0 - lrow;
  const float *ssc_lane = FP8 ? ssc + lrow : nullptr;
  pin_acc(acc);
  // fp8: scores are accumulator x row scale.  Only an item's first tile
  // (warm-up) scales the accumulators in place; otherwise the screening and
  // the examined blocks multiply as they read.
  const int gpl = mwarm_groups(a.k);
  const bool scaled = FP8 && first && gpl > 0;
  if (scaled)
    finish_scores<FP8>(acc, ssc_lane, lim0);
  else
    mask_tail(acc, lim0);
  if (first && gpl > 0) {
    // warm-up threshold: the smallest of kMLanesQ * gpl group maxima (the
    // queue, which these minima alias, is empty at an item's first tile)
    bar_lds();
    switch (gpl) {
      case 1: warm_minima<kMVals / 1, NQB>(L, acc, wv, c, h); break;
      case 2: warm_minima<kMVals / 2, NQB>(L, acc, wv, c, h); break;
      case 4: warm_minima<kMVals / 4, NQB>(L, acc, wv, c, h); break;
      case 8: warm_minima<kMVals / 8, NQB>(L, acc, wv, c, h); break;
      case 16: warm_minima<kMVals / 16, NQB>(L, acc, wv, c, h); break;
      case 32: warm_minima<kMVals / 32, NQB>(L, acc, wv, c, h); break;
      default: warm_minima<1, NQB>(L, acc, wv, c, h); break;
    }
    bar_lds();
    if (tid < it.qvalid) {
      float th = L.warm[tid];
#pragma unroll
      for (int w = 1; w < kMW; ++w) th = fminf(th, L.warm[w * kMMQ + tid]);
      L.thr0[tid] = th;
      L.thr[tid] = th;
      publish_thr(L, a, it, tid, th);
    }
    bar_lds();
#pragma unroll
    for (int qb = 0; qb < kMQB; ++qb) thr_r[qb] = L.thr[qb * 32 + c];
  }

  // shared thresholds of this lane's queries (read when the tile's copies
  // started; a stale value is just a lower bound)
  float g_r[kMQB];
#pragma unroll
  for (int qb = 0; qb < kMQB; ++qb) {
    const uint32_t gq = gt[qb * 32 + c];
    g_r[qb] = gq ? unord_score(gq) : -__builtin_inff();
    thr_r[qb] = fmaxf(thr_r[qb], g_r[qb]);
  }
  // Screening: elig[qb] bit 16 rb + i marks score (rb, qb, i) of this lane
  // as still to be examined; a 16-score row block is eligible when its best
  // score reaches the query threshold.
  pin_acc(acc);
  uint64_t elig[NQB];
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb) elig[qb] = 0ull;
#pragma unroll
  for (int rb = 0; rb < kMRB; ++rb) {
    float s16[16];
    row_scales<FP8>(s16, ssc_lane, rb, scaled);
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {
      float m = ninf;
#pragma unroll
      for (int i = 0; i < 16; ++i) m = fmaxf(m, FP8 ? acc[rb][qb][i] * s16[i] : acc[rb][qb][i]);
      elig[qb] |= m >= thr_r[qb] ? 0xFFFFull << (16 * rb) : 0ull;
    }
  }
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb)
    if (qb * 32 + c >= it.qvalid) elig[qb] = 0ull;
  // Scores at or above the current threshold are appended to the per-query
  // LDS queues (atomics, no barrier).  Merges into the k-lists are deferred:
  // one barrier per tile checks whether some queue overflowed (its
  // candidates stay eligible) or is due for a merge; only then do the
  // threads of the queries merge, the thresholds rise, and the candidates
  // left over are examined again.  A queue is due when half full if the
  // lists are in LDS, and only when full if they are in global memory,
  // where a merge round costs more than the candidates a later threshold rise
  // would save.
  constexpr int QC = kQcap<LISTS>, qdue = LISTS == kLdsLists ? QC / 2 : QC;
  for (;;) {
    bool ovf = false, full = false;
    pin_acc(acc);
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {
      const int ql = qb * 32 + c;
      const float th = thr_r[qb];
      uint64_t fail = 0;
#pragma unroll
      for (int rb = 0; rb < kMRB; ++rb) {
        const uint32_t el = (uint32_t)(elig[qb] >> (16 * rb)) & 0xFFFFu;
        if (!__builtin_amdgcn_ballot_w64(el != 0)) continue;
        float v[16], s16[16];
        row_scales<FP8>(s16, ssc_lane, rb, scaled);
        uint32_t cand = 0;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          v[i] = FP8 ? acc[rb][qb][i] * s16[i] : acc[rb][qb][i];
          cand |= v[i] >= th ? 1u << i : 0u;
        }
        cand &= el;
        if (!__builtin_amdgcn_ballot_w64(cand != 0)) continue;
        // one atomic per lane and block reserves queue slots for all its
        // candidates; the ones past the queue's room stay eligible
        const int rowb = opaque(row0 + lrow + rb * 32);
        int slot = 0;
        if (cand) slot = atomicAdd(&L.qcount[ql], __builtin_popcount(cand));
        while (cand) {
          if (slot >= QC) {
            fail |= (uint64_t)cand << (16 * rb);
            ovf = true;
            break;
          }
          const int jx = __builtin_ctz(cand);
          cand &= cand - 1u;
          // v[jx] by a tree of bitwise selects on the bits of jx (opaque
          // all-ones / zero masks: as plain selects, the compiler turns the
          // tree into an indexed load from scratch memory)
          uint32_t w8[8], w4[4];
          const uint32_t m0 = (uint32_t)opaque(-(jx & 1)), m1 = (uint32_t)opaque(-((jx >> 1) & 1));
          const uint32_t m2 = (uint32_t)opaque(-((jx >> 2) & 1)), m3 = (uint32_t)opaque(-(jx >> 3));
#pragma unroll
          for (int i = 0; i < 8; ++i)
            w8[i] = (__float_as_uint(v[2 * i]) & ~m0) | (__float_as_uint(v[2 * i + 1]) & m0);
#pragma unroll
          for (int i = 0; i < 4; ++i) w4[i] = (w8[2 * i] & ~m1) | (w8[2 * i + 1] & m1);
          const uint32_t w2a = (w4[0] & ~m2) | (w4[1] & m2), w2b = (w4[2] & ~m2) | (w4[3] & m2);
          const float sc = __uint_as_float((w2a & ~m3) | (w2b & m3));
          full |= slot + 1 >= qdue;
          L.queue[ql * QC + slot] = make_key(sc, (uint32_t)(rowb + 8 * (jx >> 2) + (jx & 3)));
          ++slot;
        }
      }
      elig[qb] = fail;
    }
    if (__builtin_amdgcn_ballot_w64(ovf) && lane == 0) L.flags[1] = epoch;
    if (__builtin_amdgcn_ballot_w64(full) && lane == 0) L.flags[2] = epoch;
    bar_lds();
    const bool again = L.flags[1] == epoch;
    if (!again && L.flags[2] != epoch) {   // no queue needs a merge yet
      ++epoch;
      break;
    }
    if constexpr (LISTS == kWaveLists) {
      merge_lists(L, a, it, gt);
    } else {
      if (tid < it.qvalid) merge_queue<LISTS == kLdsLists>(L, a, it, tid);
    }
    bar_lds();
#pragma unroll
    for (int qb = 0; qb < kMQB; ++qb) thr_r[qb] = fmaxf(L.thr[qb * 32 + c], g_r[qb]);
    ++epoch;
    if (!again) break;
  }
}

// One work item (a query tile against one corpus slice) whose queries fill
// NQB of the tile's 32-query blocks: the fragment reads, the matrix-core
// steps and the epilogue skip the blocks past the item's queries (few
// distinct queries).  The copies are those of a full
// tile (the query rows past the item's queries read as zeros).
template <bool FP8, int LISTS, bool SEED, int NQB>
__device__ __forceinline__ void run_item(const MfmaArgs &a, const MLds &L, const Split &sp,
                                         int64_t nu, int w, int &epoch) {
  using G = Geo<FP8>;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int c = lane & 31, h = lane >> 5;
  const int N = (int)a.N, d = (int)a.d;
  const int nch = (d + kMKC - 1) / kMKC;
  const float ninf = -__builtin_inff();
  // (the per-lane copy offsets are recomputed at each copy from the lane id,
  // a few VALU operations, rather than held in registers across the loop)
  {
    MItem it;
    const int qt = w % (int)sp.qtiles;
    it.s = w / (int)sp.qtiles;
    it.S = sp.S;
    it.T = seed_tiles(a.k, sp.ntiles, sp.S, nch);
    const int s0 = (int)((int64_t)it.s * sp.ntiles / sp.S);
    const int s1 = (int)((int64_t)(it.s + 1) * sp.ntiles / sp.S);
    const int t0 = s0;
    const int t1 = SEED ? s0 + (s1 - s0 < it.T ? s1 - s0 : it.T) : s1;
    it.qbase = qt * kMMQ;
    it.qvalid = (int)(nu - it.qbase < kMMQ ? nu - it.qbase : kMMQ);
    const int ntl = t1 - t0;
    const int T = ntl * nch;
    if constexpr (SEED) {
      if (it.s % seed_stride(it.S) != 0) {   // not sampled: no lane maxima
        const int per = it.T * kMLanesQ;
        for (int e = tid; e < it.qvalid * per; e += kMT) {
          const int qq = e / per, r = e - qq * per;
          a.lmax[((int64_t)(it.qbase + qq) * it.S + it.s) * per + r] = 0u;
        }
        return;
      }
    }

    // per-item state
    if (tid < kMMQ) {
      L.qcount[tid] = 0;
      L.thr0[tid] = ninf;
      L.thr[tid] = ninf;
      L.lmin[tid] = 0ull;
      L.pub[tid] = 0u;
      if (tid < it.qvalid && !SEED) {
        // (items of the first round start before any item has finished)
        if (w >= a.grid) {
          const uint32_t b =
              level_bound(a.lvl + (int64_t)(it.qbase + tid) * kLvl * it.S, (int)it.S);
          if (b) {
            atomicMax(a.gthr + it.qbase + tid, b);
            L.pub[tid] = b;
          }
        }
        if (LISTS == kLdsLists) {
          for (int j = 0; j < a.k; ++j) L.lists[tid * a.k + j] = 0ull;
        } else if (LISTS == kTailLists) {
          uint64_t *l = a.part + ((int64_t)(it.qbase + tid) * it.S + it.s) * a.k;
          for (int j = 0; j < a.k - kMTail; ++j) l[j] = 0ull;
          for (int j = 0; j < kMTail; ++j) L.tail[tid * kMTail + j] = 0ull;
        }
      }
    }
    float thr_r[kMQB];   // (read from L.thr after the prologue barrier)

    // the query tile's rows in the tiled order of tile_queries_kernel: stage
    // s of the tile is the 16 KiB block s, already in LDS order
    const i32x4m qrs =
        make_rsrc((const unsigned char *)a.q + (int64_t)(it.qbase / kMMQ) * nch * G::bbytes,
                  (uint32_t)(nch * G::bbytes));

    // copy stream: next chunk to issue.  A chunk is copied in two parts:
    // issue_a copies the corpus rows of this wave (the only wave that reads
    // them) and issue_b the wave's share of the query rows, the tile's shared
    // thresholds and row scales, and advances the stream.  issue_a of a
    // chunk always precedes its issue_b.
    int i_tl = 0, i_kc = 0, i_slot = 0, i_sc = 0, i_gt = 0, i_left = T;
    struct CopyA {
      i32x4m rs;
      uint32_t lds, voff, voff1;
    };
    auto prep_a = [&]() __attribute__((always_inline)) {
      CopyA ca;
      unsigned char *st = L.ring + i_slot * G::stage;
      const int ln = opaque(lane);
      constexpr int PA = G::apieces;
      const int wvs = __builtin_amdgcn_readfirstlane(wv);
      ca.lds = (uint32_t)(uintptr_t)st + wvs * G::adma * 1024;
      if (a.tiled) {
        // the tile's stages are consecutive blocks already in LDS order: this
        // wave's copies read adma consecutive KiB of the stage's block
        const uint32_t tb = (uint32_t)(nch * G::abytes);
        ca.rs = make_rsrc((const unsigned char *)a.corpus + (int64_t)(t0 + i_tl) * tb, tb);
        ca.voff = (uint32_t)((i_kc / kMKC) * G::abytes + wvs * G::adma * 1024 + ln * 16);
        ca.voff1 = ca.voff;
        return ca;
      }
      const int row0 = (t0 + i_tl) * kMNC;
      const int rows = N - row0 < kMNC ? N - row0 : kMNC;
      ca.rs = make_rsrc((const unsigned char *)a.corpus + (int64_t)row0 * d * G::esz,
                        (uint32_t)(rows * d * G::esz));
      const int arow0 = wvs * G::adma * (64 / PA) + ln / PA;
      ca.voff = (uint32_t)(arow0 * d * G::esz + swz_slot<PA>(ln % PA, ln / PA) * 16 + i_kc * G::esz);
      // the swizzle depends on the row mod 16: a bf16 copy holds 8 rows, so odd
      // copies hold rows 8..15 mod 16 (an fp8 copy holds 16 rows: one pattern)
      ca.voff1 = (uint32_t)(arow0 * d * G::esz +
                            swz_slot<PA>(ln % PA, (64 / PA) % 16 + ln / PA) * 16 + i_kc * G::esz);
      return ca;
    };
    auto issue_a_j = [&](const CopyA &ca, int j) __attribute__((always_inline)) {
      constexpr int PA = G::apieces;
      const uint32_t jstep = a.tiled ? 1024u : (uint32_t)((64 / PA) * d * G::esz);
      dma16s(ca.rs, ca.lds + j * 1024, ((j & 1) ? ca.voff1 : ca.voff) + (uint32_t)j * jstep);
    };
    auto issue_a = [&]() __attribute__((always_inline)) {
      if (i_left <= 0) return;
      const CopyA ca = prep_a();
#pragma unroll
      for (int j = 0; j < G::adma; ++j) issue_a_j(ca, j);
    };
    struct CopyB {
      uint32_t lds, voff;
    };
    // query part of the next chunk: this wave's bdma consecutive KiB of the
    // stage's block (queries past n_u and columns past d are zeros there);
    // once the stream has ended, zeros through an offset past the range
    auto prep_b = [&]() __attribute__((always_inline)) {
      CopyB cb;
      const int ln = opaque(lane);
      const int wvs = __builtin_amdgcn_readfirstlane(wv);
      cb.voff = i_left > 0
                    ? (uint32_t)((i_kc / kMKC) * G::bbytes + wvs * G::bdma * 1024 + ln * 16)
                    : 0x80000000u;
      cb.lds = (uint32_t)(uintptr_t)(L.ring + i_slot * G::stage + G::abytes) + wvs * G::bdma * 1024;
      return cb;
    };
    auto issue_b_j = [&](const CopyB &cb, int j) __attribute__((always_inline)) {
      dma16s(qrs, cb.lds + j * 1024, cb.voff + (uint32_t)(j * 1024));
    };
    auto extras_advance = [&]() __attribute__((always_inline)) {
      if (i_left <= 0) return;
      const int ln = opaque(lane);
      if (i_kc == 0) {
        // shared thresholds of the query tile, entries [32 wv, 32 wv + 64)
        const i32x4m grs = make_rsrc(a.gthr + it.qbase, (uint32_t)(it.qvalid * 4));
        dma4(grs, L.gtl + i_gt * kMGts + 32 * wv, (uint32_t)((32 * wv + ln) * 4));
        i_gt = i_gt + 1 == G::ngt ? 0 : i_gt + 1;
      }
      if constexpr (FP8) {
        if (i_kc == 0) {
          // rows [kMRowsW * wv, + 128) of the tile: the wave's own rows and an
          // overlap with the next wave's (same values, same place)
          const int row0 = (t0 + i_tl) * kMNC;
          const int rows = N - row0 < kMNC ? N - row0 : kMNC;
          const i32x4m srs = make_rsrc(a.scale + row0, (uint32_t)(rows * 4));
#pragma unroll
          for (int j = 0; j < 2; ++j)
            dma4(srs, L.sscale + i_sc * kMSS + wv * kMRowsW + j * 64,
                 (uint32_t)((wv * kMRowsW + j * 64 + ln) * 4));
          i_sc = i_sc + 1 == G::nsc ? 0 : i_sc + 1;
        }
      }
      i_kc += kMKC;
      if (i_kc >= d) {
        i_kc = 0;
        ++i_tl;
      }
      i_slot = i_slot + 1 == G::ns ? 0 : i_slot + 1;
      --i_left;
    };
    auto issue_b = [&]() __attribute__((always_inline)) {
      const CopyB cb = prep_b();
#pragma unroll
      for (int j = 0; j < G::bdma; ++j) issue_b_j(cb, j);
      extras_advance();
    };
#pragma unroll
    for (int j = 0; j < G::ns; ++j) {
      issue_a();
      issue_b();
    }
    // chunk 0 landed (chunks 1 .. ns-1 are younger)
    wait_vm(((T < G::ns ? T : G::ns) - 1) * G::ldma);
    bar_lds();

#pragma unroll
    for (int qb = 0; qb < kMQB; ++qb) thr_r[qb] = L.thr[qb * 32 + c];
    f32x16m acc[kMRB][NQB];
    Frag<FP8, NQB> f0, f1;
    read_frags<FP8>(f0, L.ring, wv, c, h, 0);
    int r_slot = 0, e_sc = 0, e_gt = 0, g = 0;

    // One stage: two halves of two MFMA steps each.  Once this wave's reads
    // of the stage's slot are complete (after step 0) it refills its own
    // corpus rows there with stage g+ns; no other wave reads them, so no
    // barrier is needed, and these copies (three quarters of the bytes)
    // get about half a stage more to arrive.  Before step 3 the wave waits
    // for stage g+1, the barrier lets every wave's copies of it be read and
    // lets the query rows of the slot be refilled, and the next stage's
    // first fragments are read, so that reads overlap the last MFMAs.
    // (Moving the whole copy earlier costs a second barrier per stage, which
    // was slower: the loop is bound by the matrix cores sharing the CU with
    // the LDS reads more than by copy latency.)
    // There is one wave per SIMD, so whatever stands between two matrix
    // instructions without being in the shadow of one is lost: the reads go two
    // or three to an instruction and so have landed when the next half needs
    // them, and the bookkeeping of the copies (stream position, descriptors,
    // offsets) is done behind matrix instructions of the steps that have
    // little else to issue, ahead of the step that uses it.
    constexpr int NR = Frag<FP8, NQB>::nreads, NM = kMRB * NQB;
    constexpr int RPM = (NR + NM - 1) / NM < 2 ? 2 : (NR + NM - 1) / NM;   // reads per MFMA
    constexpr int CPA = (G::adma + NM - 1) / NM, CPB = (G::bdma + NM - 1) / NM;
    auto stage = [&](auto first_c, auto rd_c) __attribute__((always_inline)) {
      constexpr bool FIRST = decltype(first_c)::value, RD = decltype(rd_c)::value;
      const unsigned char *cur = L.ring + r_slot * G::stage;
      const int ln1 = opaque(lane);
      CopyA ca;
      mfma_step_il<FP8, FIRST>(acc, f0, 0, [&](int i) __attribute__((always_inline)) {
#pragma unroll
        for (int k = RPM * i; k < RPM * (i + 1); ++k)
          if (k < NR) read_frag_piece<FP8>(f1, cur, wv, ln1 & 31, ln1 >> 5, 1, k);
        if (i == (NM > 8 ? 8 : NM - 1)) {
          // the previous stage's chunk is done with; this wave's corpus rows of
          // stage g+ns are next
          if (g > 0) extras_advance();
          ca = prep_a();
          if (i_left <= 0) ca.rs.z = 0;
        }
      });
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      mfma_step_il<FP8, false>(acc, f0, 1, [&](int i) __attribute__((always_inline)) {
#pragma unroll
        for (int k = CPA * i; k < CPA * (i + 1); ++k)
          if (k < G::adma) issue_a_j(ca, k);
      });
      CopyB cb;
      mfma_step_il<FP8, false>(acc, f1, 0, [&](int i) __attribute__((always_inline)) {
        // query rows of stage g+ns, into the slot stage g used
        if (i == (NM > 4 ? 4 : NM - 1)) cb = prep_b();
      });
      r_slot = r_slot + 1 == G::ns ? 0 : r_slot + 1;
      // stage g+1 landed (after the last stage: all copies landed): younger
      // are the parts of stages g+2 .. g+ns issued so far (a tile's thresholds
      // and row scales are not counted: waiting for fewer outstanding
      // operations only waits longer)
      if (g + G::ns < T)
        wait_vm((G::ns - 2) * G::ldma + G::adma);
      else
        wait_vm(0);
      bar_lds();
      pin_step1<FP8>(f1);
      const unsigned char *nxt = L.ring + r_slot * G::stage;
      const int ln0 = opaque(lane);
      constexpr int R0 = RD ? (NR + RPM - 1) / RPM : 0;   // instructions that carry reads
      constexpr int B0 = R0 < NM - (G::bdma + CPB - 1) / CPB ? R0
                                                             : NM - (G::bdma + CPB - 1) / CPB;
      mfma_step_il<FP8, false>(acc, f1, 1, [&](int i) __attribute__((always_inline)) {
        if constexpr (RD) {
#pragma unroll
          for (int k = RPM * i; k < RPM * (i + 1); ++k)
            if (k < NR) read_frag_piece<FP8>(f0, nxt, wv, ln0 & 31, ln0 >> 5, 0, k);
        }
#pragma unroll
        for (int k = CPB * (i - B0); k < CPB * (i - B0 + 1); ++k)
          if (k >= 0 && k < G::bdma) issue_b_j(cb, k);
      });
      ++g;
    };
    // (the first stage of a tile starts the accumulators from zero; its call
    // is peeled so that the previous tile's accumulators are dead here.  The
    // last stage of a tile leaves the next fragments in LDS: the epilogue runs
    // with only the accumulators live, and f0 is refilled after it.)
    const bool later = sp.qtiles * sp.S > a.grid;   // there are items that start later
    // tiles done at the next publication (none: more than any slice has; 0 for none,
    // in one expression, took 8 more scalar spills and 1 % of 500,009 fp8 rows)
    int due = kLvlFirst;
    if (sp.S == 1 || (later && sp.S > kLvlSlices)) due = 1 << 29;
    for (int tl = 0; tl < ntl; ++tl) {
      if (nch > 1) {
        stage(std::true_type{}, std::true_type{});
        for (int j = 1; j + 1 < nch; ++j) stage(std::false_type{}, std::true_type{});
        stage(std::false_type{}, std::false_type{});
      } else {
        stage(std::true_type{}, std::false_type{});
      }
      if constexpr (SEED)
        mtile_lane_maxima<FP8>(a, it, acc, (t0 + tl) * kMNC,
                               FP8 ? L.sscale + e_sc * kMSS : nullptr, tl);
      else
        mtile_epilogue<FP8, LISTS>(L, a, it, acc, thr_r, epoch, (t0 + tl) * kMNC,
                                       FP8 ? L.sscale + e_sc * kMSS : nullptr,
                                       L.gtl + e_gt * kMGts, tl == 0);
      if constexpr (!SEED && LISTS == kWaveLists) {
        // merge what is still queued and publish the lists' order statistics;
        // before the item's end, take what all slices have published
        const bool end = tl + 1 == ntl;
        if (end || tl + 1 == due) {
          due *= 2;
          bar_lds();
          merge_any(L, a, it, L.gtl + e_gt * kMGts);
          if (later || !end) publish_levels_wave(L, a, it);
          bar_lds();
          if (!end) {
            if (tid < it.qvalid) raise_by_levels(L, a, it, tid);
            bar_lds();
#pragma unroll
            for (int qb = 0; qb < kMQB; ++qb) thr_r[qb] = fmaxf(thr_r[qb], L.thr[qb * 32 + c]);
          }
        }
      }
      if constexpr (FP8) e_sc = e_sc + 1 == G::nsc ? 0 : e_sc + 1;
      e_gt = e_gt + 1 == G::ngt ? 0 : e_gt + 1;
      read_frags<FP8>(f0, L.ring + r_slot * G::stage, wv, c, h, 0);
    }

    if constexpr (SEED) {   // sampled tiles this slice does not have: no value
      const int st = it.T;
      for (int e = tid; e < it.qvalid * (st - ntl) * kMLanesQ; e += kMT) {
        const int q = e / ((st - ntl) * kMLanesQ), r = e % ((st - ntl) * kMLanesQ);
        a.lmax[(((int64_t)(it.qbase + q) * it.S + it.s) * st + ntl) * kMLanesQ + r] = 0u;
      }
    }
    // merge what is still queued, then flush the LDS lists of this item
    if constexpr (!SEED && LISTS != kWaveLists) {
      bar_lds();
      if (tid < it.qvalid) {
        merge_queue<LISTS == kLdsLists>(L, a, it, tid);
        // this slice's order statistics for the items that start later
        const uint64_t mn = L.lmin[tid];
        const int fill = (mn >> 32) ? a.k : (int)mn;
        const uint64_t *gl = a.part + ((int64_t)(it.qbase + tid) * it.S + it.s) * a.k;
        uint32_t *lv = a.lvl + (int64_t)(it.qbase + tid) * kLvl * it.S + it.s;
        for (int l = 0; l < kLvl; ++l) {
          const int p = opaque(((a.k + (1 << l) - 1) >> l) - 1);   // ceil(k / 2^l) - 1
          if (p < fill) {
            uint64_t key;
            if (LISTS == kLdsLists)
              key = L.lists[tid * a.k + p];
            else if (p >= a.k - kMTail)
              key = L.tail[tid * kMTail + p - (a.k - kMTail)];
            else
              key = gl[p];
            __hip_atomic_store(lv + l * it.S, (uint32_t)(key >> 32), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
          }
        }
      }
    }
    if (LISTS == kLdsLists && !SEED) {
      bar_lds();
      const int tot = it.qvalid * a.k;
      for (int t = tid; t < tot; t += kMT) {
        const int q = t / a.k, j = t - q * a.k;
        a.part[((int64_t)(it.qbase + q) * it.S + it.s) * a.k + j] = L.lists[t];
      }
    }
    if constexpr (!SEED && LISTS == kWaveLists) {   // empty slots
      const int mine = wv + kMW * lane;
      const int fill = lane < kMMQ / kMW && mine < it.qvalid ? (int)L.lmin[mine] : a.k;
      for (int j = 0; j < kMMQ / kMW && wv + kMW * j < it.qvalid; ++j) {
        uint64_t *l = a.part + ((int64_t)(it.qbase + wv + kMW * j) * it.S + it.s) * a.k;
        for (int i = __builtin_amdgcn_readlane(fill, j) + lane; i < a.k; i += 64) l[i] = 0ull;
      }
    }
    if (LISTS == kTailLists && !SEED) {
      bar_lds();
      const int tot = it.qvalid * kMTail;
      for (int t = tid; t < tot; t += kMT) {
        const int q = t / kMTail, j = t - q * kMTail;
        a.part[((int64_t)(it.qbase + q) * it.S + it.s) * a.k + a.k - kMTail + j] = L.tail[t];
      }
    }
    wait_vm(0);
    bar_lds();
  }
}

template <bool FP8, int LISTS, bool SEED>
__global__ __launch_bounds__(kMT, 1) void score_mfma_dma(MfmaArgs a) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const MLds L = carve_mlds<FP8, LISTS>(smem, a.k);
  const int64_t nu = read_nu(a.n_unique, a.n_unique_dev, a.cap);
  int64_t smax = kMSplitMaxSK / a.k;
  const Split sp = make_split(nu, a.N, kMMQ, kMNC, a.grid, smax < 1 ? 1 : smax);
  const int items = (int)(sp.qtiles * sp.S);
  if (threadIdx.x < 4) L.flags[threadIdx.x] = 0;
  int epoch = 1;
  for (int w = logical_wg(a.grid); w < items; w += a.grid) {
    // Queries of the item's tile (at least one: the tiles cover n_u).  With
    // several query tiles, the items of one corpus slice run on neighbouring
    // workgroups of one XCD and share its L2 only while they run at the same
    // pace, so every item then runs as a full tile; a single (partial) tile
    // skips its empty query blocks.
    const int64_t qv = sp.qtiles > 1 ? kMMQ : nu;
    if (qv > 96)
      run_item<FP8, LISTS, SEED, 4>(a, L, sp, nu, w, epoch);
    else if (qv > 64)
      run_item<FP8, LISTS, SEED, 3>(a, L, sp, nu, w, epoch);
    else if (qv > 32)
      run_item<FP8, LISTS, SEED, 2>(a, L, sp, nu, w, epoch);
    else
      run_item<FP8, LISTS, SEED, 1>(a, L, sp, nu, w, epoch);
  }
}

// ---------------------------------------------------------------- host side

int persistent_grid();

// Score workspace of the matrix-core path: [shared thresholds, cap x u32]
// (rounded to 256 bytes) followed by the partial lists.
size_t mfma_thr_bytes(int64_t cap) { return ((size_t)cap * 4 + 255) & ~(size_t)255; }

// Bytes of a query and slice in the partial-list area: the list, or the seed
// pass's maxima where these take more.  (The sample of short slices, the only one
// that depends on the dimension, is held within the list's bytes.)
static size_t mfma_list_bytes(int k, const Split &sp) {
  const size_t lists = (size_t)k * 8;
  const size_t maxima = (size_t)seed_tiles(k, sp.ntiles, sp.S, 1) * kMLanesQ * 4;
  return lists > maxima ? lists : maxima;
}

// worst case over n_u in [1, cap] and grids up to grid_max of n_u * S *
// per_slice bytes (0: those of the partial-list area).
// It takes up to (cap / 128) x 64 splits, and every score call lays out its
// workspace with it, so results are kept for the few shapes a process uses
// (on a window of a few hundred queries the loops cost tens of microseconds,
// on the launch path).
struct SplitWorstMemo {
  int64_t cap, N;
  int k, grid_max;
  size_t per_slice;
  bool valid;
  size_t bytes;
};
static std::mutex g_split_memo_mu;
static SplitWorstMemo g_split_memo[16];
static unsigned g_split_memo_next = 0;

static size_t mfma_split_worst(int64_t cap, int64_t N, int k, int grid_max, size_t per_slice) {
  {
    std::lock_guard<std::mutex> lock(g_split_memo_mu);
    for (const SplitWorstMemo &m : g_split_memo)
      if (m.valid && m.cap == cap && m.N == N && m.k == k && m.grid_max == grid_max &&
          m.per_slice == per_slice)
        return m.bytes;
  }
  size_t best = 0;
  const int64_t qtmax = (cap + kMMQ - 1) / kMMQ;
  int64_t smax = kMSplitMaxSK / k;
  if (smax < 1) smax = 1;
  for (int64_t qt = 1; qt <= qtmax; ++qt) {
    const int64_t nu = qt * kMMQ < cap ? qt * kMMQ : cap;
    for (int64_t g = 8; g <= grid_max; g += 8) {
      const Split sp = make_split(nu, N, kMMQ, kMNC, g, smax);
      const size_t b =
          (size_t)nu * (size_t)sp.S * (per_slice ? per_slice : mfma_list_bytes(k, sp));
      if (b > best) best = b;
    }
  }
  best = (best + 255) & ~(size_t)255;
  std::lock_guard<std::mutex> lock(g_split_memo_mu);
  g_split_memo[g_split_memo_next++ % 16] = {cap, N, k, grid_max, per_slice, true, best};
  return best;
}

// Score workspace of the matrix-core path: [shared thresholds, cap x u32 |
// order statistics of finished items, n_u x kLvl x S u32 | partial lists, n_u
// x S x k keys, and before them in the same bytes the seed pass's lane maxima,
// n_u x S x T x 8 u32], each rounded to 256 bytes.
// published order statistics, n_u x S x kLvl u32
static size_t mfma_lvl_bytes(int64_t cap, int64_t N, int k, int grid_max) {
  return mfma_split_worst(cap, N, k, grid_max, (size_t)kLvl * 4);
}

// Offset of the partial lists (and the lane maxima) in the score workspace.
size_t mfma_part_offset(int64_t cap, int64_t N, int k, int grid_max) {
  return mfma_thr_bytes(cap) + mfma_lvl_bytes(cap, N, k, grid_max);
}

static size_t mfma_partial_bytes(int64_t cap, int64_t N, int k, int grid_max) {
  return mfma_part_offset(cap, N, k, grid_max) + mfma_split_worst(cap, N, k, grid_max, 0);
}

void mfma_split_params(int *mq, int *nc, int64_t *smax, int k) {
  *mq = kMMQ;
  *nc = kMNC;
  int64_t s = kMSplitMaxSK / k;
  *smax = s < 1 ? 1 : s;
}

template <typename K>
static hipError_t launch_mfma(K kern, int grid, int lds, const MfmaArgs &a, hipStream_t st) {
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(kMT), lds, st, a);
  return hipGetLastError();
}

// Threshold seed per distinct query: the k-th largest of its lane maxima
// from the seed pass (at most kSeedMax of them), written to gthr, which it
// thereby (re)starts for the call: 0, no threshold, where there is no seed.
// The seed pass reads gthr only with its copies and never uses the values.
// Radix
// select on the 32-bit ordered scores, 8 bits per pass: a pass counts the
// values that carry the digits chosen so far by their next digit, and keeps
// the largest digit whose count of values at or above it reaches the rank
// still sought.
constexpr int kSeedThreads = 256;
template <bool F32>
__global__ __launch_bounds__(kSeedThreads) void mfma_seed_kernel(
    const uint32_t *__restrict__ lmax, int64_t n_unique, const int64_t *__restrict__ nu_dev,
    int64_t cap, int64_t N, int nch, int k, int64_t smax, uint32_t room, int grid,
    uint32_t *__restrict__ gthr,
    uint32_t *__restrict__ lvl) {
  __shared__ uint32_t vals[kSeedMax];
  __shared__ uint32_t hist[256];
  __shared__ uint32_t sel[2];   // chosen digit, values above it
  const int64_t nu = read_nu(n_unique, nu_dev, cap);
  const Split sp =
      make_split(nu, N, kMMQ, F32 ? kFNC : kMNC, grid, bound_slices(smax, nu, room));
  int64_t per;
  if (F32) {
    const int64_t stride = f32_seed_stride(sp.S);
    per = f32_seeded(sp) ? (sp.S + stride - 1) / stride * kFGroups : 0;
  } else {
    per = sp.S * kMLanesQ * seed_tiles(k, sp.ntiles, sp.S, nch);
  }
  const int n = (int)(per < kSeedMax ? per : kSeedMax);
  const int tid = threadIdx.x;
  // no item of this call has finished yet: no published order statistics
  if (!F32)
    for (int64_t e = (int64_t)blockIdx.x * kSeedThreads + tid; e < nu * kLvl * sp.S;
         e += (int64_t)gridDim.x * kSeedThreads)
      lvl[e] = 0u;
  if (n < k) {   // fewer lane maxima than k: no seed
    for (int64_t q = (int64_t)blockIdx.x * kSeedThreads + tid; q < nu;
         q += (int64_t)gridDim.x * kSeedThreads)
      gthr[q] = 0u;
    return;
  }
  for (int64_t q = blockIdx.x; q < nu; q += gridDim.x) {
    const uint32_t *src = lmax + q * per;
    for (int i = tid; i < n; i += kSeedThreads) vals[i] = src[i];
    uint32_t prefix = 0u, pmask = 0u;
    int kk = k;   // rank sought among the values that carry prefix
    for (int shift = 24; shift >= 0; shift -= 8) {
      hist[tid] = 0u;
      __syncthreads();
      for (int i = tid; i < n; i += kSeedThreads) {
        const uint32_t v = vals[i];
        if ((v & pmask) == prefix) atomicAdd(&hist[(v >> shift) & 0xFFu], 1u);
      }
      __syncthreads();
      if (tid < kWave) {
        // lane l holds digits 255 - 4l - j (j = 0..3), largest first; an
        // exclusive scan over lanes counts the values above its digits
        uint32_t c[4], sum = 0u;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          c[j] = hist[255 - 4 * tid - j];
          sum += c[j];
        }
        uint32_t incl = sum;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
          const uint32_t t = __shfl_up(incl, o);
          if (tid >= o) incl += t;
        }
        uint32_t above = incl - sum;
        if (above < (uint32_t)kk && (uint32_t)kk <= incl) {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            if (above + c[j] >= (uint32_t)kk) {
              sel[0] = 255u - 4u * tid - j;
              sel[1] = above;
              break;
            }
            above += c[j];
          }
        }
      }
      __syncthreads();
      prefix |= sel[0] << shift;
      pmask |= 0xFFu << shift;
      kk -= (int)sel[1];
      // (hist was last read before the barrier above; sel is rewritten only
      // after the next pass's counting barrier)
    }
    if (tid == 0) gthr[q] = prefix;
    __syncthreads();
  }
}

hipError_t launch_seed_select(const MfmaArgs &a, int64_t smax, uint32_t room, bool f32,
                              hipStream_t st) {
  const int64_t want = a.n_unique >= 0 ? a.n_unique : a.cap;
  const int64_t blocks = want < 4 * (int64_t)a.grid ? want : 4 * (int64_t)a.grid;
  if (blocks <= 0) return hipSuccess;
  hipLaunchKernelGGL(f32 ? mfma_seed_kernel<true> : mfma_seed_kernel<false>,
                     dim3((unsigned)blocks), dim3(kSeedThreads), 0, st, a.lmax, a.n_unique,
                     a.n_unique_dev, a.cap, a.N, (int)((a.d + kMKC - 1) / kMKC), a.k, smax, room,
                     a.grid, a.gthr, a.lvl);
  return hipGetLastError();
}

// Tiled corpus layout.  Tile t (corpus rows [384 t, 384 t + 384)) and stage s
// (columns [64 s, 64 s + 64)) form one block of Geo::abytes bytes at
// (t * nch + s) * Geo::abytes, nch = ceil(d / 64): the stage exactly as the
// copies place it in LDS, row r of the tile at r * Geo::arow with its 16-byte
// pieces in the swizzled slots the fragment reads expect (slot x of row r holds
// piece swz_slot(x, r)).  Rows past N and columns past d are zeros.  The score
// kernel then copies each wave's share of a stage as consecutive KiB instead of
// 8 (bf16) or 16 (fp8) row pieces per copy.
template <bool FP8>
__global__ __launch_bounds__(256) void tile_corpus_kernel(const unsigned char *__restrict__ src,
                                                          int64_t N, int64_t d, int nch,
                                                          int64_t npieces,
                                                          uint4 *__restrict__ dst) {
  using G = Geo<FP8>;
  constexpr int PA = G::apieces;
  constexpr int per_stage = G::abytes / 16;
  for (int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x; p < npieces;
       p += (int64_t)gridDim.x * 256) {
    const int64_t blk = p / per_stage;
    const int in = (int)(p - blk * per_stage);
    const int64_t t = blk / nch;
    const int s = (int)(blk - t * nch);
    const int r = in / PA;
    const int piece = swz_slot<PA>(in % PA, r);   // (an XOR: slot -> piece)
    const int64_t row = t * kMNC + r;
    const int64_t col = (int64_t)s * kMKC + piece * (16 / G::esz);
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (row < N && col < d)
      v = *reinterpret_cast<const uint4 *>(src + (row * d + col) * G::esz);
    dst[p] = v;
  }
}

// The distinct queries in the same order, per query tile: tile u (queries
// [128 u, 128 u + 128)) and stage s (128 bytes of each row: 64 bf16 or 32 fp32
// columns) form the 16 KiB block u * nch + s, row r of the tile at r * 128
// bytes with its pieces in the swizzled slots; queries past n_u and columns
// past d are zeros.  Written into the score workspace at the start of every
// score call (the queries' bytes read, the tiles' bytes written), so that the
// score kernels' query copies read consecutive KiB too.
__global__ __launch_bounds__(256) void tile_queries_kernel(
    const unsigned char *__restrict__ q, int64_t n_unique, const int64_t *__restrict__ nu_dev,
    int64_t cap, int64_t row_bytes, int nch, uint4 *__restrict__ dst) {
  constexpr int PB = Geo<false>::bpieces;
  constexpr int per_stage = Geo<false>::bbytes / 16;
  const int64_t nu = read_nu(n_unique, nu_dev, cap);
  const int64_t npieces = (nu + kMMQ - 1) / kMMQ * nch * per_stage;
  for (int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x; p < npieces;
       p += (int64_t)gridDim.x * 256) {
    const int64_t blk = p / per_stage;
    const int in = (int)(p - blk * per_stage);
    const int64_t u = blk / nch;
    const int s = (int)(blk - u * nch);
    const int r = in / PB;
    const int piece = swz_slot<PB>(in % PB, r);
    const int64_t row = u * kMMQ + r;
    const int64_t col = (int64_t)s * Geo<false>::brow + piece * 16;
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (row < nu && col < row_bytes)
      v = *reinterpret_cast<const uint4 *>(q + row * row_bytes + col);
    dst[p] = v;
  }
}

// Bytes of the tiled queries for up to cap distinct queries of row_bytes each.
size_t qtile_bytes(int64_t cap, int64_t row_bytes) {
  return (size_t)((cap + kMMQ - 1) / kMMQ) *
         (size_t)((row_bytes + Geo<false>::brow - 1) / Geo<false>::brow) * Geo<false>::bbytes;
}

hipError_t launch_tile_queries(const void *q, int64_t n_unique, const int64_t *nu_dev, int64_t cap,
                               int64_t row_bytes, void *dst, hipStream_t st) {
  if (cap <= 0) return hipSuccess;
  const int64_t want = (int64_t)(qtile_bytes(cap, row_bytes) / 16 + 255) / 256;
  const unsigned blocks = (unsigned)(want < 2048 ? want : 2048);
  const int nch = (int)((row_bytes + Geo<false>::brow - 1) / Geo<false>::brow);
  hipLaunchKernelGGL(tile_queries_kernel, dim3(blocks), dim3(256), 0, st,
                     (const unsigned char *)q, n_unique, nu_dev, cap, row_bytes, nch,
                     (uint4 *)dst);
  return hipGetLastError();
}

// Offset of the tiled queries in the score workspace (after the partial lists).
size_t mfma_qtile_offset(int64_t cap, int64_t N, int k, int grid_max) {
  return (mfma_partial_bytes(cap, N, k, grid_max) + 255) & ~(size_t)255;
}

size_t mfma_tiled_bytes(int64_t N, int64_t d, bool fp8) {
  const int64_t tiles = (N + kMNC - 1) / kMNC, nch = (d + kMKC - 1) / kMKC;
  return (size_t)(tiles * nch) * (size_t)(fp8 ? Geo<true>::abytes : Geo<false>::abytes);
}

hipError_t launch_tile_corpus(const void *corpus, int64_t N, int64_t d, bool fp8, void *tiled,
                              hipStream_t st) {
  const int64_t npieces = (int64_t)(mfma_tiled_bytes(N, d, fp8) / 16);
  if (npieces == 0) return hipSuccess;
  const int nch = (int)((d + kMKC - 1) / kMKC);
  const int64_t want = (npieces + 255) / 256;
  const unsigned blocks = (unsigned)(want < 8192 ? want : 8192);
  if (fp8)
    hipLaunchKernelGGL(tile_corpus_kernel<true>, dim3(blocks), dim3(256), 0, st,
                       (const unsigned char *)corpus, N, d, nch, npieces, (uint4 *)tiled);
  else
    hipLaunchKernelGGL(tile_corpus_kernel<false>, dim3(blocks), dim3(256), 0, st,
                       (const unsigned char *)corpus, N, d, nch, npieces, (uint4 *)tiled);
  return hipGetLastError();
}

hipError_t launch_score_mfma(const void *q, const void *corpus, const float *scale, int64_t N,
                             int64_t d, int k, int64_t n_unique, const int64_t *nu_dev,
                             int64_t cap, bool fp8, bool tiled, void *ws, hipStream_t st) {
  // shared thresholds: (re)started by the seed selection on every call
  uint32_t *gthr = (uint32_t *)ws;
  uint32_t *lvl = (uint32_t *)((unsigned char *)ws + mfma_thr_bytes(cap));
  void *part = (unsigned char *)ws + mfma_part_offset(cap, N, k, kMGridMax);
  uint32_t *lmax = (uint32_t *)part;
  void *qt = (unsigned char *)ws + mfma_qtile_offset(cap, N, k, kMGridMax);
  hipError_t e = launch_tile_queries(q, n_unique, nu_dev, cap, d * 2, qt, st);
  if (e != hipSuccess) return e;
  MfmaArgs a;
  a.q = qt;
  a.corpus = corpus;
  a.scale = scale;
  a.N = N;
  a.d = d;
  a.k = k;
  a.n_unique = n_unique;
  a.n_unique_dev = nu_dev;
  a.cap = cap;
  a.part = (uint64_t *)part;
  a.gthr = gthr;
  a.lmax = lmax;
  a.lvl = lvl;
  a.grid = persistent_grid();
  a.tiled = tiled ? 1 : 0;
  // k-lists in LDS when they fit beside the ring
  const bool ll = mfma_lds_bytes(fp8, true, k) <= kMLdsMax;
  const int lds = mfma_lds_bytes(fp8, ll, k);
  const int lds_seed = mfma_lds_bytes(fp8, false, k);
  auto run = [&](bool seed) {
    if (seed)
      return fp8 ? launch_mfma(score_mfma_dma<true, kTailLists, true>, a.grid, lds_seed, a, st)
                 : launch_mfma(score_mfma_dma<false, kTailLists, true>, a.grid, lds_seed, a, st);
    if (ll)
      return fp8 ? launch_mfma(score_mfma_dma<true, kLdsLists, false>, a.grid, lds, a, st)
                 : launch_mfma(score_mfma_dma<false, kLdsLists, false>, a.grid, lds, a, st);
    if (k > kTailMax)
      return fp8 ? launch_mfma(score_mfma_dma<true, kWaveLists, false>, a.grid, lds, a, st)
                 : launch_mfma(score_mfma_dma<false, kWaveLists, false>, a.grid, lds, a, st);
    return fp8 ? launch_mfma(score_mfma_dma<true, kTailLists, false>, a.grid, lds, a, st)
               : launch_mfma(score_mfma_dma<false, kTailLists, false>, a.grid, lds, a, st);
  };
  // Seed pass: score the first T tiles of every sampled slice (all slices, or
  // one in seed_stride(S)) and keep only lane maxima; their k-th largest per
  // query (a lower bound of the query's k-th best over the corpus, taken over
  // a sample of tiles spread over it)
  // seeds the shared thresholds.  The main pass then scores every tile with
  // lists that stay nearly untouched from the first tile on.
  e = run(true);
  if (e != hipSuccess) return e;
  int64_t smax = kMSplitMaxSK / k;
  e = launch_seed_select(a, smax < 1 ? 1 : smax, 0u, false, st);
  if (e != hipSuccess) return e;
  return run(false);
}

}  // namespace hs
