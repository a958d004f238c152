// What the matrix-core score kernels share (score_mfma.hip: bf16 and fp8
// corpora, score_f32.hip: fp32): asynchronous copies into LDS, their waits,
// the LDS piece order, and the per-query queues and sorted k-lists of the
// fused top-k.
#pragma once

#include "common.h"

namespace hs {

constexpr int kMMQ = 128;                // queries per tile
constexpr int kMQcap = 8;                // queue slots per query and round
constexpr int kMTail = 16;               // list entries kept in LDS when the lists are global
constexpr int kMSplitMaxSK = 8192;       // bound on S*k (merge list length)
constexpr int kMLdsMax = 160 * 1024;     // LDS per workgroup on gfx950
constexpr int kMGridMax = 512;           // persistent grid never exceeds this

// fp32 path (score_f32.hip): tiles of 64 corpus rows; its seed sample has 8 row
// groups per slice and query (the slice's first 32 rows).
constexpr int kFNC = 64;
constexpr int kFGroups = 8;
// Seed: worth a pass of its own when a slice has at least kFSeedTiles tiles
// (the pass costs one tile); at most kFSeedSlices slices are sampled.  200,000
// x 768, 120 queries, k = 10: 12 tiles per slice, about 160 of 200,000 rows
// pass the seed, where 46 of each slice's 390 rows entered unseeded lists.
constexpr int kFSeedTiles = 4;
constexpr int kFSeedSlices = 256;
__host__ __device__ __forceinline__ bool f32_seeded(const Split &sp) {
  return sp.ntiles >= kFSeedTiles * sp.S;
}
__host__ __device__ __forceinline__ int64_t f32_seed_stride(int64_t S) {
  return (S + kFSeedSlices - 1) / kFSeedSlices;
}

// Slot of 16-byte piece p in a row of P pieces.  gfx950's LDS serves a
// ds_read_b128 16 lanes at a time over 64 banks (256 bytes); the fragment
// reads have 16 consecutive rows read the same piece, so the 16 / P rows that
// share a 256-byte window must get distinct slots, for every p: the slot is p
// XOR the row's window number (mod P).  Only row mod 16 matters.
template <int P>
__device__ __forceinline__ int swz_slot(int p, int row) {
  return p ^ ((row / (16 / P)) & (P - 1));
}

// Barrier for LDS data: this wave's LDS operations complete, then s_barrier.
// No memory fence, so copies into the ring stay in flight across it.
__device__ __forceinline__ void bar_lds() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// Wait until at most n of this wave's vector-memory operations are pending
// (they complete in issue order).  n is one of the few values a ring depth
// can produce.
__device__ __forceinline__ void wait_vm(int n) {
  __builtin_amdgcn_sched_barrier(0);
  switch (n) {
#define HS_VM_CASE(x) \
  case x: asm volatile("s_waitcnt vmcnt(" #x ")" ::: "memory"); break;
    HS_VM_CASE(1) HS_VM_CASE(2) HS_VM_CASE(3) HS_VM_CASE(4) HS_VM_CASE(5) HS_VM_CASE(6)
    HS_VM_CASE(7) HS_VM_CASE(8) HS_VM_CASE(9) HS_VM_CASE(10) HS_VM_CASE(11) HS_VM_CASE(12)
    HS_VM_CASE(13) HS_VM_CASE(14) HS_VM_CASE(15) HS_VM_CASE(16) HS_VM_CASE(17) HS_VM_CASE(18)
    HS_VM_CASE(19) HS_VM_CASE(20) HS_VM_CASE(21) HS_VM_CASE(22) HS_VM_CASE(23) HS_VM_CASE(24)
    HS_VM_CASE(25) HS_VM_CASE(26) HS_VM_CASE(27) HS_VM_CASE(28) HS_VM_CASE(29) HS_VM_CASE(30)
    HS_VM_CASE(31) HS_VM_CASE(32)
#undef HS_VM_CASE
    default: asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); break;
  }
  __builtin_amdgcn_sched_barrier(0);
}

// Buffer descriptor (raw, stride 0) over [base, base + bytes): loads at
// offsets past `bytes` return zeros and touch no memory.
typedef int i32x4m __attribute__((ext_vector_type(4)));
__device__ __forceinline__ i32x4m make_rsrc(const void *base, uint32_t bytes) {
  // (the operands are wave-uniform; readfirstlane puts them in SGPRs)
  const uint64_t p = (uint64_t)base;
  i32x4m r;
  r.x = __builtin_amdgcn_readfirstlane((int)(uint32_t)p);
  r.y = __builtin_amdgcn_readfirstlane((int)((uint32_t)(p >> 32) & 0xFFFFu));
  r.z = __builtin_amdgcn_readfirstlane((int)bytes);
  r.w = 0x00020000;
  return r;
}

// Asynchronous copies global -> LDS (buffer_load ... lds): lane l writes its
// 16 (or 4) bytes at lds + 16 l (or 4 l).  They are issued from inline asm
// on purpose: the compiler cannot tell which LDS bytes such a copy writes,
// so for the builtin form it drains every copy in flight before any later
// LDS read, which would defeat the ring.  The kernel orders the copies
// itself (wait_vm, then a barrier).  M0 holds the LDS base; the compiler
// reserves M0 and sets it before each of its own uses, so overwriting it
// here is harmless.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void dma4(i32x4m rsrc, const void *lds, uint32_t voff) {
  const uint32_t l = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)lds);
  asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dword %1, %2, 0 offen lds"
               :: "s"(l), "v"(voff), "s"(rsrc) : "memory", "m0");
}
__device__ __forceinline__ void dma16s(i32x4m rsrc, uint32_t lds, uint32_t voff) {
  const uint32_t l = __builtin_amdgcn_readfirstlane(lds);
  asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
               :: "s"(l), "v"(voff), "s"(rsrc) : "memory", "m0");
}
#pragma clang diagnostic pop

struct MfmaArgs {
  const void *q;
  const void *corpus;
  const float *scale;
  int64_t N, d;
  int k;
  int64_t n_unique;
  const int64_t *n_unique_dev;
  int64_t cap;
  int grid;
  int tiled;        // corpus in the tiled layout (tile_corpus_kernel), else row-major
  uint64_t *part;
  uint32_t *gthr;   // [cap] per-query shared thresholds (ordered score, 0 = none)
  uint32_t *lmax;   // [n_u][S][T][8] lane maxima of the seed pass (ordered scores)
  uint32_t *lvl;    // [n_u][kLvl][S] order statistics of finished items (ordered scores)
};

struct MLds {
  unsigned char *ring;
  float *sscale;     // [nsc][kMSS] row scales of the tiles in flight (fp8)
  uint32_t *gtl;     // [ngt][kMGts] shared thresholds of the tiles in flight
  uint64_t *queue;   // [MQ][kMQcap] keys queued this round
  int32_t *qcount;   // [MQ] keys queued (may exceed kMQcap: overflow)
  float *thr0;       // [MQ] warm-up threshold of the item
  float *thr;        // [MQ] current threshold
  uint32_t *pub;     // [MQ] last threshold published to the shared array
  uint64_t *lmin;    // [MQ] last key of the sorted list when full, else its fill count
  float *warm;       // [kMW][MQ] per-wave minima of group maxima (aliases queue)
  int32_t *flags;    // [1] overflow epoch, [2] merge-due epoch
  uint64_t *lists;   // [MQ][k] or nullptr (lists in the global partial buffer)
  uint64_t *tail;    // [MQ][kMTail] last entries of the global lists, or nullptr
};

struct MItem {
  int qbase, qvalid, s;
  int64_t S;
  int T;   // tiles per slice of the seed pass sample
};

// Publish query t's threshold (a lower bound of its k-th best score over its
// slice, hence over the whole corpus) to the per-query shared array: every
// slice of the query filters with the largest bound any slice has reached.
__device__ __forceinline__ void publish_thr(const MLds &L, const MfmaArgs &a, const MItem &it,
                                            int t, float th) {
  if (!a.gthr || !(th > -__builtin_inff())) return;
  const uint32_t o = ord_score(th);
  if (o > L.pub[t]) {
    L.pub[t] = o;
    atomicMax(a.gthr + it.qbase + t, o);
  }
}

// Merge the queued keys of query t into its k-list (one thread per query).
// The list is kept sorted in descending key order (empty slots are key 0 at
// the end), so its minimum is always the last entry and an insertion only
// shifts the entries it passes: near the threshold, where nearly every
// entrant lands, that is one or two steps.  A list in the global partial
// buffer keeps its last kMTail entries in LDS while the item runs (its head,
// positions [0, k - kMTail), stays in global memory): an insertion touches
// global memory only when its key climbs above that window.
template <bool LDS_LISTS>
__device__ __forceinline__ void merge_queue(const MLds &L, const MfmaArgs &a, const MItem &it,
                                            int t) {
  const int cnt = L.qcount[t];
  if (cnt <= 0) return;
  const int n = cnt < kMQcap ? cnt : kMQcap;
  const int k = a.k;
  const int hb = LDS_LISTS ? k : k - kMTail;   // first position held in the LDS tail
  uint64_t *l = LDS_LISTS ? L.lists + t * k
                          : a.part + ((int64_t)(it.qbase + t) * it.S + it.s) * k;
  uint64_t *tail = LDS_LISTS ? nullptr : L.tail + t * kMTail;
  auto get = [&](int i) -> uint64_t { return (!LDS_LISTS && i >= hb) ? tail[i - hb] : l[i]; };
  auto set = [&](int i, uint64_t v) {
    if (!LDS_LISTS && i >= hb)
      tail[i - hb] = v;
    else
      l[i] = v;
  };
  // lmin holds the list's last key once the list is full, else its fill
  // count (below 2^32, hence below every key: a real key's ordered score is
  // nonzero), so that an entrant of a list that is not full starts at the
  // first empty slot instead of climbing over the empty ones
  uint64_t mn = L.lmin[t];
  int fill = (mn >> 32) ? k : (int)mn;
  for (int e = 0; e < n; ++e) {
    const uint64_t key = L.queue[t * kMQcap + e];
    if (key > mn) {
      int i = fill < k ? fill : k - 1;   // the key's slot if no entry above is smaller
      if constexpr (LDS_LISTS) {
        while (i > 0) {
          const uint64_t prev = get(i - 1);
          if (prev > key) break;
          set(i, prev);
          --i;
        }
      } else {
        // climb in windows of 8 entries read together (independent global
        // loads): the window's entries above the key stay, the others move
        // down by one
        while (i > 0) {
          const int lo = i > 8 ? i - 8 : 0;
          uint64_t b[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) b[u] = lo + u < i ? get(lo + u) : 0ull;   // (0: not above)
          int above = 0;
#pragma unroll
          for (int u = 0; u < 8; ++u) above += b[u] > key ? 1 : 0;
#pragma unroll
          for (int u = 7; u >= 0; --u)
            if (u >= above && lo + u < i) set(lo + u + 1, b[u]);
          if (above > 0 || lo == 0) {
            i = lo + above;
            break;
          }
          i = lo;
        }
      }
      set(i, key);
      if (fill < k) ++fill;
      mn = fill == k ? get(k - 1) : (uint64_t)fill;
    }
  }
  L.lmin[t] = mn;
  const float tl = (mn >> 32) ? unord_score((uint32_t)(mn >> 32)) : -__builtin_inff();
  const float t0v = L.thr0[t];
  L.thr[t] = tl > t0v ? tl : t0v;
  publish_thr(L, a, it, t, L.thr[t]);
  L.qcount[t] = 0;
}

}  // namespace hs
