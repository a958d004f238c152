// Steps 3 and 4: the host-side dispatch of the scoring kernels and the
// cross-slice merge of step 4.
//
// HeraSys runs one retrieval per fused node (Sec. 3.3 (I)) and batches ready
// nodes of the same type (Appendix A, batching constraint); a retrieval node's
// result is its Top-K chunks (Eq. 2 parameters; Sec. 4.1 workloads).  Here the
// batch is the n_u distinct queries and the retrieval is exact inner product.
//
// Phase 1 (score_mfma.hip for bf16 and fp8 corpora, score_f32.hip for fp32):
// persistent kernels.  Work items are (query tile, corpus slice) pairs
// (make_split), so the grid is filled whatever n_u turns out to be; each item
// leaves its slice's sorted list of the k best (score, row) keys per query.
// Phase 2 (topk_merge_kernel): per query, the S slice lists (S*k keys) are
// filtered (empty keys, and keys below the query's shared threshold), the
// rest sorted and the first k written out.
//
// Result keys order by (score desc, row asc), so ties always go to the lower
// corpus row, independently of which slice or lane saw them.
#include "common.h"

namespace hs {

constexpr int kMaxSK = 8192;        // bound on S*k (merge list length per query)
constexpr int kGridMax = 512;       // persistent grid never exceeds this

// ---------------------------------------------------------------- merge

constexpr int kMergeThreads = 1024;
constexpr int kMergeRankMax = 2048;   // survivors ranked by counting up to this many
constexpr int kMergeCutMin = 512;     // as many keys are ranked as soon as cut

// One workgroup per distinct query.  Its S*k slice keys are compacted into
// LDS, dropping empty keys, keys below the cut, and, when a shared threshold is
// given, keys whose score is below it (each a lower bound of the query's k-th
// best, so every key of the final k survives); the survivors are sorted
// (bitonic, descending; up to kMergeRankMax survivors are ranked by counting
// the survivors above each instead) and the first k decoded to (score, row),
// ranks past the survivors padded with (-inf, -1).
//
// The cut, from the slices' sorted lists: if r lists hold ceil(k / r) keys of
// at least x each, then k distinct rows do, so the r-th largest of the lists'
// ceil(k / r)-th keys is a lower bound of the k-th best key, as is the k-th
// largest list head when S >= k.  The heads alone leave few survivors when
// there are many more lists than k; with fewer than 4 k lists, the largest
// bound over r = 1, 2, 4, ... is taken (up to kMergeThreads values in all).
// Ranking takes m^2 LDS reads for m survivors: 960 queries, k = 50, S = 32 had
// about a thousand with the shared threshold alone, 109 us.
// ROOM: the lists leave room for a bounded n_u x S (without, the tiny window's merge
// takes 0.2 of its 5.4 us less).
template <bool ROOM>
__global__ __launch_bounds__(kMergeThreads) void topk_merge_kernel(
    const uint64_t *__restrict__ part, const uint32_t *__restrict__ thr, int64_t n_unique,
    const int64_t *__restrict__ n_unique_dev, int64_t cap, int64_t N, int k, int mq, int nc,
    int64_t smax, uint32_t room, int grid, float *__restrict__ out_s, int32_t *__restrict__ out_i) {
  __shared__ uint64_t buf[kMaxSK + 8];
  __shared__ uint64_t heads[kMergeThreads];
  __shared__ uint64_t head_cut;
  __shared__ int count;
  const int64_t nu = read_nu(n_unique, n_unique_dev, cap);
  const Split sp = make_split(nu, N, mq, nc, grid, ROOM ? bound_slices(smax, nu, room) : smax);
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int n = (int)(sp.S * k);
  for (int64_t q = blockIdx.x; q < nu; q += gridDim.x) {
    const uint32_t t = thr ? thr[q] : 0u;
    const uint64_t *src = part + q * sp.S * k;
    if (tid == 0) {
      count = 0;
      head_cut = 0ull;
    }
    // level l: r = 2^l lists and their ceil(k / r)-th keys; the last level
    // is that of the heads, where there are k
    const int S = (int)sp.S;
    int levels = 0, first = 0;
    if (S <= kMergeThreads && n > kMergeCutMin) {
      int below = 0;   // levels with r < k, r <= S
      while ((1 << below) < k && (1 << below) <= S) ++below;
      levels = below + (S >= k ? 1 : 0);
      first = S >= 4 * k ? levels - 1 : levels * S > kMergeThreads ? levels - kMergeThreads / S : 0;
    }
    const bool at = tid < (levels - first) * S;
    const int l = at ? first + tid / S : 0;
    const int r_l = 1 << l >= k ? k : 1 << l;
    uint64_t hk = 0ull;
    if (at) {
      hk = src[(int64_t)(tid % S) * k + (k + r_l - 1) / r_l - 1];
      heads[tid] = hk;
    }
    __syncthreads();
    if (hk != 0ull) {
      const uint64_t *hl = heads + (l - first) * S;
      int r = 0;
      for (int j = 0; j < S; ++j) r += hl[j] > hk ? 1 : 0;
      if (r == r_l - 1) atomicMax((unsigned long long *)&head_cut, (unsigned long long)hk);
    }
    __syncthreads();
    const uint64_t cut = head_cut;
    for (int i0 = 0; i0 < n; i0 += kMergeThreads) {
      const int i = i0 + tid;
      const uint64_t key = i < n ? src[i] : 0ull;
      const bool keep = key != 0ull && (uint32_t)(key >> 32) >= t && key >= cut;
      const uint64_t mask = __builtin_amdgcn_ballot_w64(keep);
      int base = 0;
      if (lane == 0 && mask) base = atomicAdd(&count, __popcll(mask));
      base = __shfl(base, 0);
      if (keep) buf[base + __popcll(mask & ((1ull << lane) - 1ull))] = key;
    }
    __syncthreads();
    const int m = count;
    if (m <= kMergeRankMax) {
      // rank = number of survivors above (keys are distinct: one per row);
      // the survivors are padded with empty keys to a multiple of 8 so that
      // eight independent reads are in flight at a time
      const int m8 = (m + 7) & ~7;
      for (int i = m + tid; i < m8; i += kMergeThreads) buf[i] = 0ull;
      __syncthreads();
      for (int u = tid; u < m; u += kMergeThreads) {
        const uint64_t key = buf[u];
        int r = 0;
        for (int j = 0; j < m8; j += 8) {
          uint64_t b[8];
#pragma unroll
          for (int t = 0; t < 8; ++t) b[t] = buf[j + t];
#pragma unroll
          for (int t = 0; t < 8; ++t) r += b[t] > key ? 1 : 0;
        }
        if (r < k) {
          float sc;
          int32_t row;
          decode_key(key, sc, row);
          out_s[q * k + r] = sc;
          out_i[q * k + r] = row;
        }
      }
      for (int j = m + tid; j < k; j += kMergeThreads) {
        out_s[q * k + j] = -__builtin_inff();
        out_i[q * k + j] = -1;
      }
    } else {
      int P = 2;
      while (P < m) P <<= 1;
      for (int i = m + tid; i < P; i += kMergeThreads) buf[i] = 0ull;
      __syncthreads();
      for (int size = 2; size <= P; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
          for (int u = tid; u < (P >> 1); u += kMergeThreads) {
            const int i = 2 * u - (u & (stride - 1));
            const int j = i + stride;
            const bool desc = (i & size) == 0;
            const uint64_t x = buf[i], y = buf[j];
            if ((x < y) == desc) {
              buf[i] = y;
              buf[j] = x;
            }
          }
          __syncthreads();
        }
      }
      for (int j = tid; j < k; j += kMergeThreads) {
        float sc;
        int32_t row;
        decode_key(j < m ? buf[j] : 0ull, sc, row);
        out_s[q * k + j] = sc;
        out_i[q * k + j] = row;
      }
    }
    __syncthreads();
  }
}


// ---------------------------------------------------------------- host side

// Workgroups of the score kernels' persistent grid: one per CU, a multiple of 8.
int persistent_grid() {
  static int cache[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
  if (!cache[dev]) {
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        cus <= 0)
      cus = 256;
    cus &= ~7;
    cache[dev] = cus < 8 ? 8 : cus;
  }
  return cache[dev] < kGridMax ? cache[dev] : kGridMax;
}

size_t mfma_qtile_offset(int64_t cap, int64_t N, int k, int grid_max);
size_t qtile_bytes(int64_t cap, int64_t row_bytes);
size_t mfma_part_offset(int64_t cap, int64_t N, int k, int grid_max);
void mfma_split_params(int *mq, int *nc, int64_t *smax, int k);
size_t f32_score_bytes(int64_t cap, int64_t N, int64_t d, int k, size_t limit);
void f32_split_params(int64_t cap, int64_t N, int64_t d, int k, size_t limit, const void *ws,
                      const uint32_t **thr, int *mq, int *nc, int64_t *smax, uint32_t *room,
                      int *grid);
hipError_t launch_score_f32(const void *q, const void *corpus, int64_t N, int64_t d, int k,
                            int64_t n_unique, const int64_t *nu_dev, int64_t cap, size_t limit,
                            void *ws, hipStream_t st);
hipError_t launch_score_mfma(const void *q, const void *corpus, const float *scale, int64_t N,
                             int64_t d, int k, int64_t n_unique, const int64_t *nu_dev,
                             int64_t cap, bool fp8, bool tiled, void *ws, hipStream_t st);

// `limit`: bytes that the workspace should stay within where it can (0: none).  It
// is part of the layout, so the three calls of a score step take the same.
size_t score_workspace_bytes(int64_t cap, int64_t N, int64_t d, int k, int corpus_dtype,
                             size_t limit) {
  if (corpus_dtype == HS_F32) return f32_score_bytes(cap, N, d, k, limit);
  return mfma_qtile_offset(cap, N, k, kGridMax) + qtile_bytes(cap, d * 2);
}

hipError_t launch_score_partial(const void *q, const void *corpus, const float *scale, int64_t N,
                                int64_t d, int k, int64_t n_unique, const int64_t *nu_dev,
                                int64_t cap, int corpus_dtype, bool tiled, size_t limit,
                                void *part, hipStream_t st) {
  if (corpus_dtype != HS_F32)
    return launch_score_mfma(q, corpus, scale, N, d, k, n_unique, nu_dev, cap,
                             corpus_dtype == HS_FP8_E4M3, tiled, part, st);
  return launch_score_f32(q, corpus, N, d, k, n_unique, nu_dev, cap, limit, part, st);
}

hipError_t launch_topk_merge(const void *part, int64_t n_unique, const int64_t *nu_dev,
                             int64_t cap, int64_t N, int64_t d, int k, int corpus_dtype,
                             size_t limit, float *out_s, int32_t *out_i, hipStream_t st) {
  int64_t blocks = n_unique >= 0 ? n_unique : cap;
  if (blocks <= 0) return hipSuccess;
  int mq, nc, grid;
  int64_t smax;
  uint32_t room = 0;   // (bf16 / fp8: the lists hold the worst n_u x S)
  const uint32_t *thr;
  if (corpus_dtype == HS_F32) {
    f32_split_params(cap, N, d, k, limit, part, &thr, &mq, &nc, &smax, &room, &grid);
  } else {
    grid = persistent_grid();
    mfma_split_params(&mq, &nc, &smax, k);
    // the workspace starts with the shared thresholds; the partial lists
    // follow the other scratch
    thr = (const uint32_t *)part;
    part = (const unsigned char *)part + mfma_part_offset(cap, N, k, kGridMax);
  }
  // a persistent grid of at most two workgroups per CU loops over queries
  if (blocks > 2 * (int64_t)grid) blocks = 2 * (int64_t)grid;
  hipLaunchKernelGGL(room ? topk_merge_kernel<true> : topk_merge_kernel<false>,
                     dim3((unsigned)blocks), dim3(kMergeThreads), 0, st,
                     (const uint64_t *)part, thr, n_unique, nu_dev, cap, N, k, mq, nc, smax, room,
                     grid, out_s, out_i);
  return hipGetLastError();
}

}  // namespace hs
