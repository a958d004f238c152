// Steps 3 and 4 for fp32 inputs: score every distinct query against the fp32
// corpus on the fp32 matrix cores and keep the k best rows per query and
// corpus slice.
//
// HeraSys runs one retrieval per fused node (Sec. 3.3 (I)) and batches ready
// nodes of the same type (Appendix A, batching constraint); a retrieval
// node's result is its Top-K chunks (Eq. 2 parameters; Sec. 4.1 workloads).
// s[u, c] = sum_j Q[u, j] C[c, j], products and sums in fp32
// (v_mfma_f32_32x32x2_f32: 157 TFLOP/s, twice the vector units' rate without
// packed arithmetic).
//
// Work decomposition: a persistent grid, one workgroup of eight waves per CU
// (two per SIMD, so that one wave's LDS reads pass under the other's matrix
// instructions).  A work item is (query tile of 128, corpus slice); a slice is
// a run of tiles of 64 corpus rows, small so that a corpus of a few thousand
// rows still covers many CUs.  Four waves share each half of a tile's rows: a
// tile with 65..128 live queries gives each of the four 32 of them; with fewer,
// they also share the K range (WQ query blocks x WK parts, WQ * WK = 4).
//
// A score is the sum of four partial sums, p_t over the K steps t mod 4 (a
// step is 8 columns), added as (p0 + p1) + (p2 + p3) whatever WQ is: a wave
// holds its 4 / WK partial sums in separate accumulators (independent chains
// of matrix instructions) and the waves exchange the rest through LDS.  So a
// query's scores do not depend on how many queries its batch has, and equal
// corpus rows get bit-identical scores.
//
// Operand staging: chunks of 32 columns (128 bytes per row) of the tile's
// rows and of the queries stream through a ring of LDS stages, written by
// buffer_load ... lds copies (rows of 128 consecutive bytes; rows past N,
// queries past n_u and columns past d read as zeros).  Pieces of 16 bytes are
// XOR-swizzled so that the fragment reads (ds_read_b128) are free of bank
// conflicts.  One barrier per chunk.  The stream runs across tiles.  More than
// 32 queries are first put in the order of the stages (tile_queries_kernel):
// every CU reads them for every tile, and as row pieces, at a stride of a row,
// they come from a few of the L2's channels.
//
// Top-k per tile: scores stay in registers; each lane compares its row
// groups with the query's threshold and appends what reaches it to the
// query's LDS queue; queues are merged into sorted k-lists when one is due.
// Thresholds: the slice's own k-list, and (slices of several tiles) a seed,
// the k-th largest of the row-group maxima of one tile in each of at most 256
// slices, taken by a first pass.  Where there is no seed, an item's first tile
// fills the lists by ranking its rows instead of queueing them.
//
// What bounds it, measured (122 distinct queries, 200,000 x 768, k = 10):
// the matrix cores.  1,936 us on the vector units before; 453 us now, of 319 us
// of matrix instructions at the 2.0 GHz this load runs at and 13 rounds of
// tiles; without the epilogue 435 us, without the copies too 369 us.  32
// requests over 4,096 x 384: 37.6 -> 15.5 us, the latency of twelve chunks.
#include "score_lists.h"

namespace hs {

typedef float f32x4f __attribute__((ext_vector_type(4)));
typedef float f32x16f __attribute__((ext_vector_type(16)));

constexpr int kFT = 512;          // threads
constexpr int kFKC = 32;          // columns per ring stage (four 8-deep steps)
constexpr int kFRow = kFKC * 4;   // bytes of one row per stage
constexpr int kFBlk = 32 * kFRow; // bytes of 32 rows per stage (4 KiB)
constexpr int kFKeyLd = 66;       // keys per query of the first tile's ranking area
                                  // (16-byte rows, 4 banks apart)

// Ring stages per number of query blocks.  The area after the ring serves the
// exchange of partial sums (WK = 4: 24 KiB, WK = 2: 16 KiB) and the ranking of a
// first tile.
template <int WQ>
struct GeoF {
  static constexpr int WK = 4 / WQ;
  static constexpr int nv = 16 / WK;              // scores a lane ends up with per tile
  static constexpr int stage = (2 + WQ) * kFBlk;  // corpus rows, then queries
  static constexpr int ns = WQ == 4 ? 4 : WQ == 2 ? 5 : 7;
  static constexpr int ring = ns * stage;         // 96, 80 or 84 KiB
  static constexpr int xchg = WK == 1 ? 0 : WK == 2 ? 16 * 1024 : 24 * 1024;
  static constexpr int rank = 32 * kFKeyLd * 8;
  static constexpr int area = ring + (xchg > rank ? xchg : rank);
};
constexpr int kFRingArea = GeoF<4>::area;
static_assert(GeoF<2>::area <= kFRingArea && GeoF<1>::area <= kFRingArea, "ring and area fit");
constexpr int kFNgt = 9;              // shared-threshold slots (tiles in flight)
static_assert(GeoF<4>::ns + 2 <= kFNgt && GeoF<2>::ns + 2 <= kFNgt && GeoF<1>::ns + 2 <= kFNgt,
              "threshold slots cover the tiles in flight");

__host__ __device__ constexpr int f32_lds_bytes() {
  return kFRingArea + kMMQ * kMQcap * 8 + kMMQ * kMTail * 8 + kFNgt * kMMQ * 4 +
         kMMQ * (8 + 4 + 4 + 4 + 4) + 16;
}
static_assert(f32_lds_bytes() <= kMLdsMax, "fits the CU");

__device__ __forceinline__ MLds carve_flds(unsigned char *p, int k) {
  MLds L;
  L.ring = p; p += kFRingArea;
  L.queue = reinterpret_cast<uint64_t *>(p); p += kMMQ * kMQcap * 8;
  // lists of k <= kMTail keys, else the last kMTail keys of the global lists
  L.lists = k <= kMTail ? reinterpret_cast<uint64_t *>(p) : nullptr;
  L.tail = k <= kMTail ? nullptr : reinterpret_cast<uint64_t *>(p);
  p += kMMQ * kMTail * 8;
  L.lmin = reinterpret_cast<uint64_t *>(p); p += kMMQ * 8;
  L.gtl = reinterpret_cast<uint32_t *>(p); p += kFNgt * kMMQ * 4;
  L.qcount = reinterpret_cast<int32_t *>(p); p += kMMQ * 4;
  L.thr0 = reinterpret_cast<float *>(p); p += kMMQ * 4;
  L.thr = reinterpret_cast<float *>(p); p += kMMQ * 4;
  L.pub = reinterpret_cast<uint32_t *>(p); p += kMMQ * 4;
  L.flags = reinterpret_cast<int32_t *>(p);
  L.sscale = nullptr;
  L.warm = nullptr;
  return L;
}

// First tile of an item without a seed: every query's 64 keys are ranked by
// counting the larger ones and the k best written to the (empty) list, 32
// queries at a time: the waves that hold a block's scores write its keys, then
// each wave ranks 4 of its queries, one key per lane.
template <int WQ, bool LDS_LISTS>
__device__ __forceinline__ void rank_first_tile(const MLds &L, const MfmaArgs &a, const MItem &it,
                                                const float (&sc)[GeoF<WQ>::nv], int row0) {
  using G = GeoF<WQ>;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, c = lane & 31, h = lane >> 5;
  const int wr = wv >> 2, wq = (wv & 3) % WQ, wk = (wv & 3) / WQ;
  uint64_t *keys = reinterpret_cast<uint64_t *>(L.ring + G::ring);
  const int k = a.k;
  const int hb = LDS_LISTS ? k : k - kMTail;
  const int lim = (int)a.N - row0;
  // (global lists: their clearing by other waves has completed, and what is
  // written here has before the merges read it)
  if (!LDS_LISTS) wait_vm(0);
  for (int b = 0; b < WQ && b * 32 < it.qvalid; ++b) {
    bar_lds();   // the area is free
    if (wq == b) {
#pragma unroll
      for (int i = 0; i < G::nv; ++i) {
        const int ii = wk * G::nv + i;
        const int r = wr * 32 + 8 * (ii >> 2) + 4 * h + (ii & 3);
        const bool ok = r < lim && sc[i] == sc[i];
        keys[c * kFKeyLd + r] = ok ? make_key(sc[i], (uint32_t)(row0 + r)) : 0ull;
      }
    }
    bar_lds();
    for (int u = 0; u < 4; ++u) {
      const int qc = wv * 4 + u, q = b * 32 + qc;   // (wave-uniform)
      if (q >= it.qvalid) break;
      const uint64_t *row = keys + qc * kFKeyLd;
      const uint64_t x = row[lane];
      int r = 0;
      for (int j = 0; j < kFNC; j += 16) {
        uint64_t y[16];
#pragma unroll
        for (int t = 0; t < 16; ++t) y[t] = row[j + t];
#pragma unroll
        for (int t = 0; t < 16; ++t) r += y[t] > x ? 1 : 0;
      }
      const int n = __builtin_popcountll(__builtin_amdgcn_ballot_w64(x != 0ull));
      if (x != 0ull && r < k) {
        if (LDS_LISTS)
          L.lists[q * k + r] = x;
        else if (r >= hb)
          L.tail[q * kMTail + r - hb] = x;
        else
          a.part[((int64_t)(it.qbase + q) * it.S + it.s) * k + r] = x;
      }
      if (n < k) {
        if (lane == 0) L.lmin[q] = (uint64_t)n;   // (the threshold stays -inf)
      } else if (x != 0ull && r == k - 1) {
        L.lmin[q] = x;
        L.thr[q] = unord_score((uint32_t)(x >> 32));
      }
    }
  }
  if (!LDS_LISTS) wait_vm(0);
  bar_lds();
}

// Top-k of one tile: scores at or above the query's threshold are queued;
// queues are merged into the k-lists when one is due.
template <int WQ, bool LDS_LISTS>
__device__ __forceinline__ void f32_epilogue(const MLds &L, const MfmaArgs &a, const MItem &it,
                                             const float (&sc)[GeoF<WQ>::nv], int row0,
                                             const uint32_t *gt, int &epoch) {
  using G = GeoF<WQ>;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, c = lane & 31, h = lane >> 5;
  const int wr = wv >> 2, wq = (wv & 3) % WQ, wk = (wv & 3) / WQ;
  const int q = wq * 32 + c, lim = (int)a.N - row0;
  const uint32_t g = a.gthr ? gt[q] : 0u;
  const float gth = g ? unord_score(g) : -__builtin_inff();
  float th = fmaxf(L.thr[q], gth);
  uint32_t pend = q < it.qvalid ? (1u << G::nv) - 1u : 0u;
  constexpr int qdue = LDS_LISTS ? kMQcap / 2 : kMQcap;
  for (;;) {
    bool ovf = false, full = false;
    uint32_t cand = 0;
#pragma unroll
    for (int i = 0; i < G::nv; ++i) cand |= sc[i] >= th ? 1u << i : 0u;
    cand &= pend;
    pend = 0u;
    if (__builtin_amdgcn_ballot_w64(cand != 0u)) {
#pragma unroll
      for (int i = 0; i < G::nv; ++i) {
        if (!((cand >> i) & 1u)) continue;
        const int ii = wk * G::nv + i;
        const int r = wr * 32 + 8 * (ii >> 2) + 4 * h + (ii & 3);
        if (r >= lim) continue;
        const int slot = atomicAdd(&L.qcount[q], 1);
        if (slot < kMQcap) {
          L.queue[q * kMQcap + slot] = make_key(sc[i], (uint32_t)(row0 + r));
          full |= slot + 1 >= qdue;
        } else {
          pend |= 1u << i;
          ovf = true;
        }
      }
    }
    if (__builtin_amdgcn_ballot_w64(ovf) && lane == 0) L.flags[1] = epoch;
    if (__builtin_amdgcn_ballot_w64(full) && lane == 0) L.flags[2] = epoch;
    bar_lds();
    const bool again = L.flags[1] == epoch;
    const bool due = again || L.flags[2] == epoch;
    ++epoch;
    if (!due) break;
    if (tid < it.qvalid) merge_queue<LDS_LISTS>(L, a, it, tid);
    bar_lds();
    th = fmaxf(L.thr[q], gth);
    if (!again) break;
  }
}

// One work item: a tile of 32 * WQ queries (128 with WQ = 4) against one
// corpus slice.
template <int WQ, bool LDS_LISTS, bool SEED>
__device__ __forceinline__ void run_item_f32(const MfmaArgs &a, const MLds &L, const Split &sp,
                                             int64_t nu, int w, int &epoch) {
  using G = GeoF<WQ>;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, c = lane & 31, h = lane >> 5;
  const int wvs = __builtin_amdgcn_readfirstlane(wv);
  const int wr = wvs >> 2, wq = (wvs & 3) % WQ, wk = (wvs & 3) / WQ;
  const int N = (int)a.N, d = (int)a.d, nch = (d + kFKC - 1) / kFKC;
  const float ninf = -__builtin_inff();
  MItem it;
  it.s = w / (int)sp.qtiles;
  it.S = sp.S;
  it.T = 1;
  it.qbase = (w % (int)sp.qtiles) * kMMQ;
  it.qvalid = (int)(nu - it.qbase < kMMQ ? nu - it.qbase : kMMQ);
  const bool seeded = a.gthr != nullptr && f32_seeded(sp);
  const int64_t stride = f32_seed_stride(sp.S);
  if (SEED && it.s % stride != 0) return;
  const int t0 = (int)((int64_t)it.s * sp.ntiles / sp.S);
  const int t1 = SEED ? t0 + 1 : (int)((int64_t)(it.s + 1) * sp.ntiles / sp.S);
  const int ntl = t1 - t0, T = ntl * nch;

  if (!SEED && tid < kMMQ) {
    L.qcount[tid] = 0;
    L.thr0[tid] = ninf;
    L.thr[tid] = ninf;
    L.lmin[tid] = 0ull;
    L.pub[tid] = 0u;
    if (LDS_LISTS) {
      for (int j = 0; j < a.k; ++j) L.lists[tid * a.k + j] = 0ull;
    } else {
      for (int j = 0; j < kMTail; ++j) L.tail[tid * kMTail + j] = 0ull;
      if (tid < it.qvalid) {
        uint64_t *l = a.part + ((int64_t)(it.qbase + tid) * it.S + it.s) * a.k;
        for (int j = 0; j < a.k - kMTail; ++j) l[j] = 0ull;
      }
    }
  }

  // Copy stream.  A copy covers 8 rows of 128 bytes: lane l writes row l / 8,
  // slot l % 8, and so reads piece swz_slot(l % 8, row).  Wave w copies rows
  // [8 w, 8 w + 8) of the corpus tile and of every 64 queries (with one query
  // block, the first four waves copy it).
  const int qcopies = WQ == 1 ? (wvs < 4 ? 1 : 0) : WQ / 2;
  const int crow = wvs * 8 + (lane >> 3);
  const uint32_t ccol = (uint32_t)(swz_slot<8>(lane & 7, crow) * 16);
  const uint32_t rowb = (uint32_t)d * 4u;
  // queries: the tiled copy's 16 KiB blocks, else rows
  const uint32_t qtile = (uint32_t)nch * (kMMQ * kFRow);
  const i32x4m qrs =
      a.tiled ? make_rsrc((const unsigned char *)a.q + (int64_t)(it.qbase / kMMQ) * qtile, qtile)
              : make_rsrc((const unsigned char *)a.q + (int64_t)it.qbase * rowb,
                          (uint32_t)it.qvalid * rowb);
  const uint32_t qstep = a.tiled ? 64 * kFRow : 64u * rowb;
  const uint32_t qoff0 = a.tiled ? (uint32_t)(wvs * 1024 + lane * 16) : (uint32_t)crow * rowb + ccol;
  const uint32_t qinc = a.tiled ? kMMQ * kFRow : kFRow;
  const uint32_t coff0 = (uint32_t)crow * rowb + ccol;
  int i_row0 = t0 * kFNC, i_slot = 0, i_gt = 0, i_left = T;
  uint32_t i_col = 0, i_q = 0;   // byte column of the chunk, query offset
  i32x4m crs = {0, 0, 0, 0x00020000};
  auto issue = [&]() __attribute__((always_inline)) {
    if (i_left <= 0) return;
    if (i_col == 0) {   // a tile's first chunk
      const int rows = N - i_row0 < kFNC ? N - i_row0 : kFNC;
      crs = make_rsrc((const unsigned char *)a.corpus + (int64_t)i_row0 * rowb,
                      (uint32_t)rows * rowb);
      if (!SEED && a.gthr && wvs < 2) {   // shared thresholds, 64 queries per wave
        const i32x4m grs = make_rsrc(a.gthr + it.qbase, (uint32_t)(it.qvalid * 4));
        dma4(grs, L.gtl + i_gt * kMMQ + 64 * wvs, (uint32_t)((64 * wvs + lane) * 4));
      }
      i_gt = i_gt + 1 == kFNgt ? 0 : i_gt + 1;
    }
    const uint32_t lds = (uint32_t)(uintptr_t)(L.ring + i_slot * G::stage) + wvs * 1024;
    // a column past d would be the next row's: past the range instead (zeros)
    const bool in = i_col + ccol < rowb;
    dma16s(crs, lds, in ? coff0 + i_col : 0x80000000u);
#pragma unroll
    for (int b = 0; b < (WQ + 1) / 2; ++b)
      if (b < qcopies)
        dma16s(qrs, lds + (2 + 2 * b) * kFBlk,
               a.tiled || in ? qoff0 + i_q + (uint32_t)b * qstep : 0x80000000u);
    i_col += kFRow;
    i_q += qinc;
    if (i_col >= rowb) {
      i_col = 0;
      i_q = 0;
      i_row0 += kFNC;
    }
    i_slot = i_slot + 1 == G::ns ? 0 : i_slot + 1;
    --i_left;
  };
  // Chunk g's fragments are read into registers one chunk ahead: advance()
  // waits for chunk g + 1 to land, and after its barrier every wave has chunk
  // g's fragments, so chunk g + ns takes that slot and chunk g + 1's fragments
  // are read while the matrix instructions of chunk g run.  The copies of
  // chunk g + ns are issued after the first quarter of chunk g's matrix
  // instructions, whose time covers them.
  constexpr int NT = 4 / G::WK;
  struct FragF {
    f32x4f a[NT], b[NT];
  };
  int slot = 0, e_gt = 0, g = -1;
  auto advance = [&](FragF &f) __attribute__((always_inline)) {
    ++g;
    // chunks g + 1 .. g + ns - 2 are younger (waiting for more is harmless)
    if (T - 1 - g < G::ns - 2)
      wait_vm(0);
    else if (WQ != 1 || wvs < 4)
      wait_vm((G::ns - 2) * (1 + (WQ + 1) / 2));
    else
      wait_vm(G::ns - 2);
    bar_lds();
    const unsigned char *st = L.ring + slot * G::stage;
    const unsigned char *ab = st + (wr * 32 + c) * kFRow;
    const unsigned char *bb = st + (2 + wq) * kFBlk + c * kFRow;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int sl = swz_slot<8>(2 * (wk * NT + t) + h, c) * 16;
      f.a[t] = *reinterpret_cast<const f32x4f *>(ab + sl);
      f.b[t] = *reinterpret_cast<const f32x4f *>(bb + sl);
    }
    __builtin_amdgcn_sched_barrier(0);
    slot = slot + 1 == G::ns ? 0 : slot + 1;
  };
  f32x16f acc[NT];
  auto multiply = [&](const FragF &f, bool live) __attribute__((always_inline)) {
    auto quarter = [&](int e) __attribute__((always_inline)) {
#pragma unroll
      for (int t = 0; t < NT; ++t)
        acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(f.a[t][e], f.b[t][e], acc[t], 0, 0, 0);
    };
    if (live) quarter(0);
    __builtin_amdgcn_sched_barrier(0);
    issue();
    __builtin_amdgcn_sched_barrier(0);
    if (live) {
      quarter(1);
      quarter(2);
      quarter(3);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll
  for (int j = 0; j < G::ns; ++j) issue();
  FragF f0, f1;
  if (T > 0) advance(f0);
  for (int tl = 0; tl < ntl; ++tl) {
    // (a seed tile is the first 32 rows of its slice)
    const bool live = wq * 32 < it.qvalid && (wr == 0 || (!SEED && (t0 + tl) * kFNC + 32 < N));
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = f32x16f{};
    for (int j = 0; j < nch; j += 2) {
      advance(f1);
      multiply(f0, live);
      if (j + 1 < nch) {
        advance(f0);
        multiply(f1, live);
      } else {
        f0 = f1;
      }
    }
    // (p0 + p1) + (p2 + p3).  Accumulator element i of a lane is row
    // 8 (i / 4) + 4 h + i % 4, query 32 wq + c; wave part wk ends up with
    // elements [nv wk, nv wk + nv).
    float sc[G::nv];
    if constexpr (G::WK == 1) {
#pragma unroll
      for (int i = 0; i < 16; ++i)
        sc[i] = (acc[0][i] + acc[1][i]) + (acc[2][i] + acc[3][i]);
    } else if constexpr (G::WK == 2) {
      const f32x16f p = acc[0] + acc[1];
      // the other part's eight elements, as two float4 per lane
      f32x4f *x = reinterpret_cast<f32x4f *>(L.ring + G::ring) + (wr * 2 + wq) * 4 * 64 + lane;
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        f32x4f v;
#pragma unroll
        for (int b = 0; b < 4; ++b) v[b] = wk ? p[4 * u + b] : p[8 + 4 * u + b];
        x[(wk * 2 + u) * 64] = v;
      }
      bar_lds();
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const f32x4f o = x[((1 - wk) * 2 + u) * 64];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const float own = wk ? p[8 + 4 * u + b] : p[4 * u + b];
          sc[4 * u + b] = wk ? o[b] + own : own + o[b];
        }
      }
    } else {
      // quarter f of part wk's sums goes to part f
      f32x4f *x = reinterpret_cast<f32x4f *>(L.ring + G::ring) + wr * 12 * 64 + lane;
      f32x4f own = {};
#pragma unroll
      for (int f = 0; f < 4; ++f) {
        const f32x4f v = {acc[0][4 * f], acc[0][4 * f + 1], acc[0][4 * f + 2], acc[0][4 * f + 3]};
        if (f == wk)
          own = v;
        else
          x[(f * 3 + (wk < f ? wk : wk - 1)) * 64] = v;
      }
      bar_lds();
      f32x4f o[3];
#pragma unroll
      for (int u = 0; u < 3; ++u) o[u] = x[(wk * 3 + u) * 64];
      // o holds the other parts in order; own goes to place wk
      const f32x4f p0 = wk == 0 ? own : o[0];
      const f32x4f p1 = wk == 0 ? o[0] : wk == 1 ? own : o[1];
      const f32x4f p2 = wk <= 1 ? o[1] : wk == 2 ? own : o[2];
      const f32x4f p3 = wk == 3 ? own : o[2];
      const f32x4f v = (p0 + p1) + (p2 + p3);
#pragma unroll
      for (int b = 0; b < 4; ++b) sc[b] = v[b];
    }
    // (the area is written again only after later barriers: the chunk
    // barriers of the next tile, or the ranking's own first barrier)

    const int row0 = (t0 + tl) * kFNC;
    if constexpr (SEED) {
      // maxima over each 4-row group: scores of distinct rows, so the k-th
      // largest over the sample bounds the query's k-th best from below
      const int q = wq * 32 + c;
      if (q < it.qvalid && wr == 0) {
        const int64_t ns = (it.S + stride - 1) / stride;
        uint32_t *dst =
            a.lmax + ((int64_t)(it.qbase + q) * ns + it.s / stride) * kFGroups + h * 4;
#pragma unroll
        for (int u = 0; u < G::nv / 4; ++u) {
          float m = ninf;
#pragma unroll
          for (int b = 0; b < 4; ++b)
            if (8 * (wk * (G::nv / 4) + u) + 4 * h + b < N - row0) m = fmaxf(m, sc[4 * u + b]);
          dst[wk * (G::nv / 4) + u] = m > ninf ? ord_score(m) : 0u;
        }
      }
    } else if (!seeded && tl == 0) {
      rank_first_tile<WQ, LDS_LISTS>(L, a, it, sc, row0);
    } else {
      f32_epilogue<WQ, LDS_LISTS>(L, a, it, sc, row0, L.gtl + e_gt * kMMQ, epoch);
    }
    e_gt = e_gt + 1 == kFNgt ? 0 : e_gt + 1;
  }

  if constexpr (!SEED) {
    bar_lds();
    if (tid < it.qvalid) merge_queue<LDS_LISTS>(L, a, it, tid);
    bar_lds();
    const int per = LDS_LISTS ? a.k : kMTail, at = a.k - per;
    const uint64_t *src = LDS_LISTS ? L.lists : L.tail;
    for (int t = tid; t < it.qvalid * per; t += kFT) {
      const int q = t / per, j = t - q * per;
      a.part[((int64_t)(it.qbase + q) * it.S + it.s) * a.k + at + j] = src[t];
    }
  }
  wait_vm(0);
  bar_lds();
}

template <bool LDS_LISTS, bool SEED>
__global__ __launch_bounds__(kFT, 2) void score_f32_mfma(MfmaArgs a, int64_t smax, uint32_t room) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const MLds L = carve_flds(smem, a.k);
  const int64_t nu = read_nu(a.n_unique, a.n_unique_dev, a.cap);
  const Split sp = make_split(nu, a.N, kMMQ, kFNC, a.grid, bound_slices(smax, nu, room));
  if (SEED && !f32_seeded(sp)) return;
  const int items = (int)(sp.qtiles * sp.S);
  if (threadIdx.x < 4) L.flags[threadIdx.x] = 0;
  int epoch = 1;
  for (int w = logical_wg(a.grid); w < items; w += a.grid) {
    const int64_t qv = nu - (int64_t)(w % (int)sp.qtiles) * kMMQ;
    if (qv > 64)
      run_item_f32<4, LDS_LISTS, SEED>(a, L, sp, nu, w, epoch);
    else if (qv > 32)
      run_item_f32<2, LDS_LISTS, SEED>(a, L, sp, nu, w, epoch);
    else
      run_item_f32<1, LDS_LISTS, SEED>(a, L, sp, nu, w, epoch);
  }
}

// ---------------------------------------------------------------- host side

int persistent_grid();
hipError_t launch_seed_select(const MfmaArgs &a, int64_t smax, uint32_t room, bool f32,
                              hipStream_t st);
size_t qtile_bytes(int64_t cap, int64_t row_bytes);
hipError_t launch_tile_queries(const void *q, int64_t n_unique, const int64_t *nu_dev, int64_t cap,
                               int64_t row_bytes, void *dst, hipStream_t st);

// Workspace: [partial lists, n_u x S x k keys; the seed pass's group maxima,
// n_u x min(S, 256) x 8 u32, use the same bytes before them][shared
// thresholds, cap x u32][tiled queries].
//
// The lists have room for a number of (query, slice) places, and a call takes as
// many slices as its own n_u leaves room for (bound_slices): a plan made for many
// requests of which few are distinct fills the chip like one made for those few.
// The room is what kFRounds rounds of items on 256 CUs take, or 40 MiB, or a slice
// per query, whichever is most, and no more than every slice of every query.
//
// Within a limit (the library's own scratch; 0: none) the room shrinks to what is
// left, and the tiled queries go where they do not fit beside one round or 40 MiB
// of lists, and the seed where its thresholds do not fit beside a slice per query.
// (No tiled queries either for up to 32 of them, where the copy's launch costs more
// than it saves, nor above 256 MiB.)
constexpr size_t kFListBudget = (size_t)40 << 20, kFTiledMax = (size_t)256 << 20;
constexpr int kFCus = 256, kFRounds = 4;

struct F32Layout {
  int64_t smax;    // bound on S for any n_u
  uint32_t room;   // and on n_u x S (0: none)
  bool seed, tiled;
  size_t thr_at, q_at, bytes;
};

static F32Layout f32_layout(int64_t cap, int64_t N, int64_t d, int k, size_t limit) {
  F32Layout l;
  auto round = [](size_t x) { return (x + 255) & ~(size_t)255; };
  const int64_t c = cap > 0 ? cap : 1;
  const size_t keys = (size_t)k * 8, per = (size_t)(k < 4 ? 4 : k) * 8;   // (maxima included)
  const size_t thr = round((size_t)c * 4), qt = c > 32 ? qtile_bytes(c, d * 4) : 0;
  const int64_t most = kMSplitMaxSK / k < 1 ? 1 : kMSplitMaxSK / k;
  const int64_t tiles = (N + kFNC - 1) / kFNC;
  l.smax = most < tiles ? most : tiles < 1 ? 1 : tiles;
  auto places = [&](int64_t r) { return r < c ? c : r < c * l.smax ? r : c * l.smax; };
  auto want = [&](size_t p) {
    const int64_t r = (int64_t)(kFListBudget / p);
    return places(r > kFRounds * kFCus * kMMQ ? r : kFRounds * kFCus * kMMQ);
  };
  l.seed = true;
  l.tiled = qt > 0 && qt <= kFTiledMax;
  size_t p = per;
  int64_t room = want(p);
  if (limit && round((size_t)room * p) + thr + (l.tiled ? qt : 0) > limit) {
    l.seed = round((size_t)c * per) + thr <= limit;
    if (!l.seed) p = keys;
    size_t left = limit - (l.seed ? thr : 0);
    const size_t one = (size_t)places(kFCus * kMMQ) * p, least = (size_t)c * p;
    const size_t beside = one < kFListBudget ? one : kFListBudget > least ? kFListBudget : least;
    l.tiled = l.tiled && round(beside) + qt <= left;
    if (l.tiled) left -= qt;
    const int64_t fits = (int64_t)(left / p), w = want(p);
    room = places(fits < w ? fits : w);
  }
  l.room = room < c * l.smax ? (uint32_t)room : 0u;   // (0: every slice of every query)
  l.thr_at = round((size_t)room * p);
  l.q_at = l.thr_at + (l.seed ? thr : 0);
  l.bytes = l.q_at + (l.tiled ? qt : 0);
  return l;
}

size_t f32_score_bytes(int64_t cap, int64_t N, int64_t d, int k, size_t limit) {
  return f32_layout(cap, N, d, k, limit).bytes;
}

// What topk_merge_kernel needs to find this path's lists: thresholds (null:
// none), the bounds on S and the tile sizes.
void f32_split_params(int64_t cap, int64_t N, int64_t d, int k, size_t limit, const void *ws,
                      const uint32_t **thr, int *mq, int *nc, int64_t *smax, uint32_t *room,
                      int *grid) {
  const F32Layout l = f32_layout(cap, N, d, k, limit);
  *mq = kMMQ;
  *nc = kFNC;
  *smax = l.smax;
  *room = l.room;
  *grid = persistent_grid();
  *thr = l.seed && f32_seeded(make_split(cap, N, kMMQ, kFNC, *grid,
                                         bound_slices(l.smax, cap, l.room)))
             ? (const uint32_t *)((const unsigned char *)ws + l.thr_at)
             : nullptr;
}

template <bool LDS_LISTS, bool SEED>
static hipError_t launch_f32(const MfmaArgs &a, int64_t smax, uint32_t room, hipStream_t st) {
  const auto kern = score_f32_mfma<LDS_LISTS, SEED>;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, f32_lds_bytes());
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(a.grid), dim3(kFT), f32_lds_bytes(), st, a, smax, room);
  return hipGetLastError();
}

hipError_t launch_score_f32(const void *q, const void *corpus, int64_t N, int64_t d, int k,
                            int64_t n_unique, const int64_t *nu_dev, int64_t cap, size_t limit, void *ws,
                            hipStream_t st) {
  MfmaArgs a = {};
  a.q = q;
  a.corpus = corpus;
  a.N = N;
  a.d = d;
  a.k = k;
  a.n_unique = n_unique;
  a.n_unique_dev = nu_dev;
  a.cap = cap;
  a.part = (uint64_t *)ws;
  a.lmax = (uint32_t *)ws;
  const uint32_t *thr;
  int mq, nc;
  int64_t smax;
  uint32_t room;
  f32_split_params(cap, N, d, k, limit, ws, &thr, &mq, &nc, &smax, &room, &a.grid);
  a.gthr = const_cast<uint32_t *>(thr);
  const F32Layout l = f32_layout(cap, N, d, k, limit);
  if (l.tiled) {
    void *qt = (unsigned char *)ws + l.q_at;
    hipError_t e = launch_tile_queries(q, n_unique, nu_dev, cap, d * 4, qt, st);
    if (e != hipSuccess) return e;
    a.q = qt;
    a.tiled = 1;
  }
  const bool ll = k <= kMTail;
  if (thr) {
    // (fewer queries make more and shorter slices: a call may still turn out
    // to be unseeded on the device, which then clears its thresholds)
    hipError_t e = launch_f32<false, true>(a, smax, room, st);
    if (e != hipSuccess) return e;
    e = launch_seed_select(a, smax, room, true, st);
    if (e != hipSuccess) return e;
  }
  return ll ? launch_f32<true, false>(a, smax, room, st)
            : launch_f32<false, false>(a, smax, room, st);
}

}  // namespace hs
