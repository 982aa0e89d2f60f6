// Cross-request selection (scores, ranking, budget choice, keep depths) and packing.
//
// Sec. 3.2 Eq. dcut-prefix-score, Sec. 3.3 Eq. dcut-objective, Alg. 1 and the
// packing of App. C; for rejection-sampling verification (App. B) the same
// kernel ranks the shifted scores of Eq. dcut-shifted-score and chooses the
// budget causally: by the early-stopping scan, or as a budget fixed beforehand.
// At most 8192 positions take part, so nothing here is bound by bytes or
// operations but by serial chains and launches.  A position's place in the
// ranking is the number of positions ahead of it, counted directly against every
// other one: scores are read four at a time as LDS broadcasts and compared in 32
// bits, which needs no sort network and no barrier, and splits over any number of
// workgroups.  Positions that score 1 by definition come first and are left out.
// With up to 512 others one 1024-thread workgroup does everything, 32 positions a
// wave.  Above, a first kernel ranks 16 positions per workgroup over the whole chip and
// the second, one workgroup, does the rest (prefix sums, budget choice, keep depths,
// packing).  The second launch costs the host 3 us, the comparisons of one workgroup
// 4 us at 512 positions (and four times that at 1024): calls in a row with nothing else
// to do, at 512 positions of 32 requests, take 12.1 us in one launch and 15.5 in two
// (on the GPU 11.8 and 9.7), at 384 12.1 and 14.1 (10.0 and 9.6).
// Against sorting 64-key runs and merging them in one workgroup, on the GPU: 64
// positions (batch 4) 9.2 -> 7.3 us, 256 11.6 -> 8.6, 512 13.0 -> 11.8 (8 requests of 64:
// 16.6 -> 15.7), 1024 (batch 64) 15.9 -> 10.2; 4096 (batch 256) 50.2 -> 15.6.
//
// Bit-exactness: each request's scores are one sequential float32 product per
// depth (denormals kept, no contraction); the rank order (score descending, then
// depth, then request) is total, so any correct count gives the same ranks;
// benefits are integer sums of trunc(s * 2^40); the budget objective is one
// float64 division.  The outputs are therefore identical on any hardware.
#include <type_traits>

#include "dcut_internal.h"
#include "scan.h"

namespace dcut {

enum SelectMode { SEL_BUCKETS = 0, SEL_SCAN = 1, SEL_FIXED = 2, SEL_HISTORY = 3 };

struct SelectParams {
  int B, D, R;
  int shift;      // 1: rank the shifted scores s~_{i,k} = s_{i,k-1} (s~_{i,1} = 1)
  int mode;       // SelectMode
  int budgets[DCUT_MAX_CANDIDATES];
  double costs[DCUT_MAX_CANDIDATES];
};

// trunc(s * 2^40) for a score's bits
__device__ __forceinline__ unsigned long long score_units(uint32_t bits) {
  return (unsigned long long)((double)__uint_as_float(bits) * 1099511627776.0);
}

__device__ __forceinline__ bool conf_bad(float c) { return !(c >= 0.0f && c <= 1.0f) || signbit(c); }

#pragma clang fp contract(off)
// Step cost at an arbitrary verification size K for the causal scan: linear
// between consecutive budgets (K_r, C_r), the end costs outside them, and the
// last of several equal budgets at that K.  Same float64 operations, in the
// same order, on every platform.  The candidates sit in LDS (bud, cst); r is
// found by binary search over the non-decreasing budgets.
__device__ double cost_at(const int *bud, const double *cst, int R, int K) {
  int lo = 0, hi = R;                 // r = (number of budgets <= K) - 1
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (bud[mid] <= K) lo = mid + 1;
    else hi = mid;
  }
  const int r = lo - 1;
  if (r < 0) return cst[0];
  if (r == R - 1) return cst[R - 1];
  const int ka = bud[r], kb = bud[r + 1];
  const double ca = cst[r], cb = cst[r + 1];
  return ca + ((cb - ca) * (double)(K - ka)) / (double)(kb - ka);
}

// objective of Eq. dcut-objective for the exact fixed-point benefit P
__device__ __forceinline__ double objective(unsigned long long P, double cost) {
  return ((double)P * 0x1p-40) / cost;
}

constexpr int SEL_FUSED_MAX = 512;     // positions counted by the one-workgroup kernel: 32 a wave
constexpr int RANK_THREADS = 512;

__host__ __device__ constexpr int pad64(int n) { return (n + 63) & ~63; }

// Scores, as bits, of the positions k * B + i (depth, then request: the order of ties) of
// the depths k from `skip` on, into sc[(k - skip) * B + i], one thread per request,
// sequential in depth; zeros up to a multiple of 64.  s_conf: B * D floats of LDS.
// Returns whether a confidence was bad.
__device__ __forceinline__ bool fill_scores(int B, int D, int shift, int skip, const float *__restrict__ conf,
                                            float *s_conf, int *sc) {
  const int n = B * max(D + 1 - skip, 0);
  for (int j = threadIdx.x; j < B * D; j += blockDim.x) s_conf[j] = conf[j];
  __syncthreads();
  bool bad = false;
  for (int i = threadIdx.x; i < B; i += blockDim.x) {
    float s = 1.0f;
    if (skip == 0) sc[i] = __float_as_int(s);
    const float *cf = s_conf + i * D;
    int *at = sc + i - skip * B;
    for (int k0 = 1; k0 <= D; k0 += 8) {
      float c[8];                    // eight confidences at a time: their reads overlap
#pragma unroll
      for (int u = 0; u < 8; ++u) c[u] = cf[min(k0 + u, D) - 1];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int k = k0 + u;
        if (k > D) break;
        const bool no = conf_bad(c[u]);
        bad |= no;
        const float prev = s;        // the shifted score of depth k: the product up to k - 1
        s = s * (no ? 0.0f : c[u]);
        if (k >= skip) at[k * B] = __float_as_int(shift ? prev : s);
      }
    }
  }
  for (int j = n + threadIdx.x; j < pad64(n); j += blockDim.x) sc[j] = 0;
  __syncthreads();
  return bad;
}

// This lane group's part of the counts of positions ahead of P positions, one in each of
// the 16-position units mu .. mu + P - 1 (lane l16 of its unit): a larger score, or an
// equal one earlier in the order of ties (bits of scores are below 2^31, so "at least s"
// is "more than s - 1").  Group seg of those that share the positions takes the units
// [lo, hi) and, if it is one of the first four, four places of their own units.  The zeros
// that pad the last units come after every position and are ahead of none.
template <int P>
__device__ __forceinline__ void count_ahead(const int *sc, int mu, int l16, int seg, int lo, int hi, int (&cnt)[P]) {
  int s[P];
#pragma unroll
  for (int p = 0; p < P; ++p) {
    s[p] = sc[16 * (mu + p) + l16];
    const int4 v = *(const int4 *)(sc + 16 * (mu + p) + 4 * (seg & 3));    // its own unit's equal scores before it
    const int d = l16 - 4 * seg;
    cnt[p] = (v.x == s[p] && d > 0) + (v.y == s[p] && d > 1) + (v.z == s[p] && d > 2) + (v.w == s[p] && d > 3);
  }
  for (int u = lo; u < hi; ++u) {
    const int4 *q = (const int4 *)(sc + 16 * u);
    int thr[P];
    uint32_t ahead[P];               // the signs of thr - score, shifted in: two operations a score
#pragma unroll
    for (int p = 0; p < P; ++p) {
      thr[p] = s[p] - (u < mu + p ? 1 : 0);
      ahead[p] = 0;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int4 v = q[j];
#pragma unroll
      for (int p = 0; p < P; ++p) {
        ahead[p] = __builtin_amdgcn_alignbit(ahead[p], (uint32_t)(thr[p] - v.x), 31);
        ahead[p] = __builtin_amdgcn_alignbit(ahead[p], (uint32_t)(thr[p] - v.y), 31);
        ahead[p] = __builtin_amdgcn_alignbit(ahead[p], (uint32_t)(thr[p] - v.z), 31);
        ahead[p] = __builtin_amdgcn_alignbit(ahead[p], (uint32_t)(thr[p] - v.w), 31);
      }
    }
#pragma unroll
    for (int p = 0; p < P; ++p) cnt[p] += __popc(ahead[p]);
  }
}

// Ranks of 16 positions per workgroup (enough workgroups for the whole chip from
// 4096 positions on): sixteen lanes hold the positions, the four lane groups of each
// wave count against different shares of the list.  Leaves the rank of position
// k * B + i in `rank` and the score bits in rank order in `sorted` (both [N], packed
// arrays of the call until the second kernel overwrites them).
__global__ void __launch_bounds__(RANK_THREADS)
k_select_rank(int B, int D, int shift, const float *__restrict__ conf, int32_t *__restrict__ rank,
              int32_t *__restrict__ sorted, int32_t *__restrict__ dev_err) {
  extern __shared__ __align__(16) int s_rank_mem[];
  constexpr int NW = RANK_THREADS / 64;
  __shared__ int s_cnt[NW][16];
  const int N = B * (D + 1), NU = pad64(N) / 16;
  int *sc = s_rank_mem;                                      // [pad64(N)], then the confidences
  const bool bad = fill_scores(B, D, shift, 0, conf, (float *)(sc + pad64(N)), sc);
  if (bad && blockIdx.x == 0 && dev_err) atomicOr(dev_err, DCUT_DERR_CONF);
  const int l16 = threadIdx.x & 15, seg = threadIdx.x >> 4, wv = threadIdx.x >> 6;
  const int m = 16 * blockIdx.x + l16;
  int c[1];
  count_ahead(sc, blockIdx.x, l16, seg, NU * seg / (4 * NW), NU * (seg + 1) / (4 * NW), c);
  c[0] += __shfl_xor(c[0], 16, 64);
  c[0] += __shfl_xor(c[0], 32, 64);
  if ((threadIdx.x & 63) < 16) s_cnt[wv][l16] = c[0];
  __syncthreads();
  if (threadIdx.x < 16 && m < N) {
    int r = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) r += s_cnt[w][l16];
    rank[m] = r;
    sorted[r] = sc[m];
  }
}

// Everything after the ranking; with FUSED (N <= SEL_FUSED_MAX) the ranking too,
// else ranks and sorted scores come from k_select_rank through ppos and ptok.
template <bool FUSED>
__global__ void __launch_bounds__(1024)
k_select(SelectParams p, const float *__restrict__ conf, const int32_t *__restrict__ draft,
         const int32_t *__restrict__ ctx_len, int32_t *__restrict__ keep_len, int32_t *__restrict__ cu,
         int32_t *ptok, int32_t *ppos, int32_t *__restrict__ preq,
         int32_t *__restrict__ choice, unsigned long long *__restrict__ benefit,
         int32_t *__restrict__ dev_err, int32_t *__restrict__ k_state) {
  extern __shared__ __align__(16) uint32_t s_mem[];
  __shared__ unsigned long long s_wave[17], s_pre[1024];
  __shared__ double s_cost[DCUT_MAX_CANDIDATES];
  __shared__ int s_bud[DCUT_MAX_CANDIDATES];
  __shared__ int s_stop, s_K;
  constexpr int EM = FUSED ? 1 : DCUT_MAX_ROWS / 1024;    // positions per thread, at most

  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int D1 = p.D + 1, B = p.B;
  const int N = B * D1;
  int *s_rank = (int *)s_mem;               // [N]: rank of position k * B + i
  uint32_t *s_sort = s_mem + pad64(N);      // [N]: score bits in rank order
  int *s_kl = (int *)(s_sort + pad64(N));   // [B], then s_cu [B + 1]
  int *s_cu = s_kl + B;
  if (tid == 0) s_stop = N;
  if (tid < p.R) {
    s_bud[tid] = p.budgets[tid];
    s_cost[tid] = p.costs[tid];
  }
  // what the packing needs, fetched before the serial part
  int zt[EM], zl[EM];
#pragma unroll
  for (int e = 0; e < EM; ++e) {
    const int idx = tid + 1024 * e;
    zt[e] = idx < N ? draft[idx] : 0;
    zl[e] = idx < N ? ctx_len[idx / D1] : 0;
  }
  if constexpr (FUSED) {
    // 1.-2. scores, and ranks.  The positions of depth 0 (and 1, shifted) score 1 and come
    // first, in their order; of the others a wave takes 32, its lane groups sharing the list.
    int *sc = (int *)s_mem + ((2 * pad64(N) + 2 * B + 1 + 3) & ~3);   // 16-byte aligned
    const int first = B * min(D1, p.shift + 1);
    const bool bad = fill_scores(B, p.D, p.shift, p.shift + 1, conf, (float *)(sc + pad64(N)), sc);
    if (bad && dev_err) atomicOr(dev_err, DCUT_DERR_CONF);
    if (tid < first) {
      s_rank[tid] = tid;
      s_sort[tid] = __float_as_uint(1.0f);
    }
    const int NU = pad64(N - first) / 16, seg = lane >> 4, l16 = lane & 15;
    auto rank_units = [&](auto pc) {
      constexpr int P = decltype(pc)::value;
      if (P * wv >= NU) return;
      int cnt[P];
      count_ahead(sc, P * wv, l16, seg, NU * seg / 4, NU * (seg + 1) / 4, cnt);
#pragma unroll
      for (int q = 0; q < P; ++q) {
        cnt[q] += __shfl_xor(cnt[q], 16, 64);
        cnt[q] += __shfl_xor(cnt[q], 32, 64);
        const int m = 16 * (P * wv + q) + l16, r = first + cnt[q];
        if (lane < 16 && first + m < N) {
          s_rank[first + m] = r;
          s_sort[r] = (uint32_t)sc[m];
        }
      }
    };
    if (NU <= 16) rank_units(std::integral_constant<int, 1>{});
    else rank_units(std::integral_constant<int, 2>{});
  } else {
#pragma unroll
    for (int e = 0; e < EM; ++e) {
      const int j = tid + 1024 * e;
      if (j < N) {
        s_rank[j] = ppos[j];
        s_sort[j] = (uint32_t)ptok[j];
      }
    }
  }
  __syncthreads();

  // 3. exact prefix sums of the fixed-point scores in rank order
  const int E = (N + 1023) / 1024;          // ranks per thread
  unsigned long long local = 0;
  for (int m = tid * E; m < tid * E + E; ++m)
    if (m < N) local += score_units(s_sort[m]);
  unsigned long long total;
  const unsigned long long pre = block_exclusive_scan(local, s_wave, &total);
  s_pre[tid] = pre;
  __syncthreads();
  double obj = -1.0;                        // candidate tid's objective (first wave)
  if (tid < p.R) {
    const int K = s_bud[tid];
    const int t = K / E, rem = K - t * E;
    unsigned long long P = t < 1024 ? s_pre[t] : total;
    for (int m = t * E; m < t * E + rem; ++m) P += score_units(s_sort[m]);
    obj = objective(P, s_cost[tid]);
    if (benefit) benefit[tid] = P;
  }

  // 4a. causal scan (App. B): the positions enter in rank order from K = B on,
  // and the scan stops at the first K whose next position does not strictly
  // raise the objective.  Every thread tests the sizes of its own ranks.
  if (p.mode == SEL_SCAN) {
    unsigned long long P = pre;             // benefit of the first tid * E ranks
    int stop = N;
    for (int m = tid * E; m < tid * E + E && m < N; ++m) {
      const unsigned long long P1 = P + score_units(s_sort[m]);
      if (m >= B && !(objective(P1, cost_at(s_bud, s_cost, p.R, m + 1)) >
                      objective(P, cost_at(s_bud, s_cost, p.R, m)))) {
        stop = m;
        break;
      }
      P = P1;
    }
    if (stop < N) atomicMin(&s_stop, stop);
    __syncthreads();
  }

  // 4b. budget choice: the first strict maximum of benefit * 2^-40 / cost over
  // the candidates, the fixed budget, the scan's stop, or the budget carried
  // over from the previous block (which then carries this block's choice on)
  if (wv == 0) {
    static_assert(DCUT_MAX_CANDIDATES <= 64, "one candidate per lane");
    double best_obj = obj;
    int bucket = lane;                      // the largest objective, the smaller index among equals
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const double o = __shfl_xor(best_obj, off, 64);
      const int q = __shfl_xor(bucket, off, 64);
      if (o > best_obj || (o == best_obj && q < bucket)) {
        best_obj = o;
        bucket = q;
      }
    }
    if (lane == 0) {
      int best = bucket, Kstar;
      if (p.mode == SEL_BUCKETS) {
        Kstar = s_bud[best];
      } else if (p.mode == SEL_FIXED) {
        best = 0;
        Kstar = s_bud[0];
      } else {
        if (p.mode == SEL_SCAN) {
          Kstar = s_stop;
        } else {
          const int k = k_state[0];
          Kstar = k < B ? B : (k > N ? N : k);
          k_state[0] = s_bud[bucket];
        }
        best = -1;                          // the last candidate budget not above K*
        for (int r = 0; r < p.R; ++r)
          if (s_bud[r] <= Kstar) best = r;
      }
      choice[0] = Kstar;
      choice[1] = best;
      s_K = Kstar;
    }
  }
  __syncthreads();

  // 5. keep depths: request i keeps the depths ranked within the top K* (a prefix;
  // its bonus position always is), so its last one sets the count
  const int K = s_K;
#pragma unroll
  for (int e = 0; e < EM; ++e) {
    const int j = tid + 1024 * e;
    if (j < N && s_rank[j] < K && (j + B >= N || s_rank[j + B] >= K)) {
      const int k = j / B;
      s_kl[j - k * B] = k + 1;
      keep_len[j - k * B] = k + 1;
    }
  }
  __syncthreads();

  // 6. packing (App. C): cu = exclusive scan of keep_len; row t = cu[i] + k
  // gets (z_{i,k}, L_i + k, i), rows past K* zeros
  const int per = (B + 1023) / 1024;        // <= 4
  int v[4];
  int loc = 0;
  for (int j = 0; j < per; ++j) {
    const int i = tid * per + j;
    v[j] = i < B ? s_kl[i] : 0;
    loc += v[j];
  }
  int kept;
  int off = block_exclusive_scan(loc, (int *)s_wave, &kept);
  for (int j = 0; j < per; ++j) {
    const int i = tid * per + j;
    if (i < B) {
      s_cu[i] = off;
      cu[i] = off;
    }
    off += v[j];
  }
  if (tid == 0) {
    s_cu[B] = kept;
    cu[B] = kept;
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < EM; ++e) {
    const int idx = tid + 1024 * e;
    if (idx >= N) break;
    const int i = idx / D1, k = idx - i * D1;
    const int t = s_cu[i] + k;
    if (t < s_cu[i + 1]) {
      ptok[t] = zt[e];
      ppos[t] = zl[e] + k;
      preq[t] = i;
    }
    if (idx >= kept) {
      ptok[idx] = 0;
      ppos[idx] = 0;
      preq[idx] = 0;
    }
  }
}
#pragma clang fp contract(on)

}  // namespace dcut

using namespace dcut;

static int select_run(int B, int D, const float *conf, const int32_t *draft, const int32_t *ctx_len,
                      int shift, int mode, int R, const int32_t *budgets, const double *costs, int32_t *k_state,
                      int32_t *keep_len, int32_t *cu, int32_t *packed_tok, int32_t *packed_pos,
                      int32_t *packed_req, int32_t *choice, uint64_t *benefit, int32_t *dev_err,
                      hipStream_t stream) {
  if (!batch_ok(B, D)) return DCUT_EINVAL;
  if (R < 1 || R > DCUT_MAX_CANDIDATES || !budgets || !costs) return DCUT_EINVAL;
  if (mode == SEL_FIXED && R != 1) return DCUT_EINVAL;
  if (mode == SEL_HISTORY && !k_state) return DCUT_EINVAL;
  if (!conf && D > 0) return DCUT_EINVAL;
  if (!draft || !ctx_len || !keep_len || !cu || !packed_tok || !packed_pos || !packed_req || !choice)
    return DCUT_EINVAL;
  SelectParams p;
  p.B = B;
  p.D = D;
  p.R = R;
  p.shift = shift;
  p.mode = mode;
  for (int r = 0; r < R; ++r) {
    int K = budgets[r];
    double c = costs[r];
    if (K < B || K > B * (D + 1)) return DCUT_EINVAL;
    if (r > 0 && K < budgets[r - 1]) return DCUT_EINVAL;
    if (!(c > 0.0) || !(c < __builtin_inf())) return DCUT_EINVAL;
    p.budgets[r] = K;
    p.costs[r] = c;
  }
  const int N = B * (D + 1);
  const int first = B * (D < shift ? 1 : shift + 1);     // positions of score 1 that come first anyway
  const size_t base = ((size_t)2 * pad64(N) + 2 * B + 1) * sizeof(uint32_t);   // ranks, sorted scores, keep depths, offsets
  const size_t scores = (size_t)pad64(N) * sizeof(uint32_t) + (size_t)B * D * sizeof(float);
  if (N <= 1024 && N - first <= SEL_FUSED_MAX)
    return launch(DCUT_KERNEL_SELECT, k_select<true>, dim3(1), dim3(1024), base + 16 + scores, stream, p, conf, draft,
                  ctx_len, keep_len, cu, packed_tok, packed_pos, packed_req, choice, (unsigned long long *)benefit,
                  dev_err, k_state);
  DCUT_TRY(launch_span(DCUT_KERNEL_SELECT, true, false, k_select_rank, dim3(pad64(N) / 16), dim3(RANK_THREADS), scores,
                       stream, B, D, shift, conf, packed_pos, packed_tok, dev_err));
  return launch_span(DCUT_KERNEL_SELECT, false, true, k_select<false>, dim3(1), dim3(1024), base, stream, p, conf, draft,
                     ctx_len, keep_len, cu, packed_tok, packed_pos, packed_req, choice, (unsigned long long *)benefit,
                     dev_err, k_state);
}

extern "C" int dcut_select(int B, int D, const float *conf, const int32_t *draft,
                           const int32_t *ctx_len, int R, const int32_t *budgets,
                           const double *costs, int32_t *keep_len, int32_t *cu,
                           int32_t *packed_tok, int32_t *packed_pos, int32_t *packed_req,
                           int32_t *choice, uint64_t *benefit, int32_t *dev_err,
                           hipStream_t stream) {
  return select_run(B, D, conf, draft, ctx_len, 0, SEL_BUCKETS, R, budgets, costs, nullptr, keep_len, cu,
                    packed_tok, packed_pos, packed_req, choice, benefit, dev_err, stream);
}

extern "C" int dcut_select_rs(int B, int D, const float *conf, const int32_t *draft,
                              const int32_t *ctx_len, int mode, int R, const int32_t *budgets,
                              const double *costs, int32_t *k_state, int32_t *keep_len, int32_t *cu,
                              int32_t *packed_tok, int32_t *packed_pos, int32_t *packed_req,
                              int32_t *choice, uint64_t *benefit, int32_t *dev_err,
                              hipStream_t stream) {
  int m;
  if (mode == DCUT_RS_SCAN) m = SEL_SCAN;
  else if (mode == DCUT_RS_FIXED) m = SEL_FIXED;
  else if (mode == DCUT_RS_HISTORY) m = SEL_HISTORY;
  else return DCUT_EINVAL;
  return select_run(B, D, conf, draft, ctx_len, 1, m, R, budgets, costs, k_state, keep_len, cu, packed_tok,
                    packed_pos, packed_req, choice, benefit, dev_err, stream);
}
