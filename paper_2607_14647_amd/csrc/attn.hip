// Ragged causal GQA attention over per-request KV slabs, split over key chunks.
//
// App. C: every kept position is scored against its request's accepted prefix
// (cache slots 0..L_i-1) and, causally, against the kept block positions before
// it (slots L_i..L_i+k, appended by the QKV epilogue).
//
// Work item = (request i, kv head g, chunk c).  Chunk c covers cache keys
// [c*CH, min((c+1)*CH, L_i)); the last chunk also covers the block keys
// [L_i, L_i + d_i).  The chunking depends on L_i only, never on d_i, so a row's
// partial results are the same whichever later rows are kept.  All G = n_q/n_kv
// query heads of the group and all d_i kept rows (G*d_i <= 256 rows, 16 per
// wave) share each 32-key tile, so the cache is read from HBM exactly once.
//
// Per tile and wave (v_mfma_f32_16x16x32_bf16):
//   S^T[key][row] = K[key][:] . Q[row][:]   -> lane (row = lane%16) owns keys
//                                              4*(lane/16)+j of each 16-key block
//   online softmax per row (exp2 domain), row statistics stay lane-local
//   O^T[d][row]  += V^T[d][key] . P^T[key][row], with P taken straight from the
//                   S^T accumulators (the same key permutation is applied to the
//                   V^T operand), V staged transposed in LDS.
// Partial (o, m, l) per (row, head, chunk) are merged in chunk order by
// k_attn_combine; a request with a single chunk is finished in place.
//
// What bounds it: the cache stream.  A copy without the compute takes 139 us where
// the kernel takes 145 (batch 64, 0.8 GB), with or without the tile barrier and with
// a deeper ring, so the inner loop is kept short enough to hide: fragment addresses
// are one per-lane constant with the k-step or column tile flipped in, tiles whose
// keys every row sees take no masks, and weights use the hardware exp2.  Batch 16 at
// 128 rows 33 -> 28 us, batch 64 at 1024 rows 173 -> 165; groups of 8 heads (up to 128
// rows, two row blocks per wave in three workgroups per CU instead of 8 waves in two)
// 163 -> 152 us at batch 128.
//
// Workgroup b takes item b of the longest-first work order (attn_plan.h),
// which the layer's first norm kernel builds in one extra workgroup; batches
// too large to plan and grids of one round of slots number the items
// arithmetically, chunk index slowest.
#include "attn_plan.h"
#include "dcut_internal.h"

namespace dcut {

namespace {

constexpr int KT = 32;     // keys per tile

typedef short short4v __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(3))) const bf16x8 lds_frag;

// Barrier of the LDS ring: each wave has waited (s_waitcnt vmcnt) for its own
// loads of the stage it reads next, so only the hardware barrier is needed; a
// memory fence here would drain every stage still in flight.  The empty asm
// statements keep the compiler from moving LDS accesses across it.
__device__ __forceinline__ void ring_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Transposing LDS reads (ds_read_b64_tr_b16), four columns x two key halves per
// call, the second half HALF bytes after the first.  They are issued from one
// asm statement that also waits for them (lgkmcnt(0)), so the compiler only
// ever sees completed results; it cannot model these reads itself without also
// draining every LDS-DMA stage still in flight (vmcnt(0)).  The ring protocol
// (vmcnt wait + barrier) orders them after the DMA writes of the stage they
// read.
template <int HALF>
__device__ __forceinline__ void lds_read_tr16_x8(short4v (&r)[8], uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3) {
  asm volatile(
      "ds_read_b64_tr_b16 %0, %8\n\t"
      "ds_read_b64_tr_b16 %1, %8 offset:%12\n\t"
      "ds_read_b64_tr_b16 %2, %9\n\t"
      "ds_read_b64_tr_b16 %3, %9 offset:%12\n\t"
      "ds_read_b64_tr_b16 %4, %10\n\t"
      "ds_read_b64_tr_b16 %5, %10 offset:%12\n\t"
      "ds_read_b64_tr_b16 %6, %11\n\t"
      "ds_read_b64_tr_b16 %7, %11 offset:%12\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(r[4]), "=&v"(r[5]), "=&v"(r[6]), "=&v"(r[7])
      : "v"(a0), "v"(a1), "v"(a2), "v"(a3), "n"(HALF)
      : "memory");
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t uniform_rsrc(const void *base, int bytes) {
  const uintptr_t b = (uintptr_t)base;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
  const int n = __builtin_amdgcn_readfirstlane(bytes);
  return __builtin_amdgcn_make_buffer_rsrc((void *)(((uintptr_t)hi << 32) | lo), (short)0, n, 0x00020000);
}

// NSTAGE LDS ring stages: NSTAGE - 1 tiles in flight while one is used.  At
// most 168 registers (three waves per SIMD), so three 4-wave workgroups with
// 3-stage rings (48 KB of LDS each) share a CU.  A wave owns RB blocks of 16
// query rows, 16 * NW rows apart; blocks past an item's rows are skipped.
template <int HD, int NW, int NSTAGE, int RB>
__global__ void __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(3)))
k_attn(AttnArgs a) {
  constexpr int ROWB = HD * 2;              // bytes per key row
  constexpr int CPR = ROWB / 16;            // 16-byte chunks per key row (8 or 16)
  constexpr int TILEB = KT * ROWB;          // bytes of one K (or V) tile
  constexpr int STAGEB = 2 * TILEB;         // K tile then V tile
  constexpr int RPI = 1024 / ROWB;          // key rows per 1 KB wave load
  constexpr int LPK = (TILEB / 1024 + NW - 1) / NW;      // wave loads per stage for K (and for V)
  constexpr int LPW = 2 * LPK;
  constexpr int NS = HD / 32;               // k-steps of the QK product
  constexpr int NT = HD / 16;               // 16-row tiles of O^T
  __shared__ __align__(ROWB) unsigned char ring[NSTAGE * STAGEB];   // fragment addresses flip bits within a row

  const int MC = a.max_chunks;
  const int tid = threadIdx.x, lane = tid & 63;
  int g, c, t0, d, L, cap;
  int64_t base;                       // first element of the request's slab
  if (a.plan) {
    const int idx = blockIdx.x;
    const int n = a.plan[0];
    const int4 *it = (const int4 *)((const char *)a.plan + PLAN_HEAD) + 2 * idx;
    const int4 e0 = it[0], e1 = it[1];
    if (idx >= n) return;
    g = e0.y; c = e0.z; t0 = e0.w;
    d = e1.x; L = e1.y; cap = e1.z;
    base = (int64_t)(((uint64_t)(uint32_t)e1.w << 32) | (uint32_t)e0.x);
  } else {
    // Chunk index slowest: the work items that exist for every request (the
    // first chunks) come first, so workgroups of chunks a request does not
    // have are dispatched last and exit without holding a slot among live ones.
    const int idx = blockIdx.x;
    c = idx / (a.B * a.n_kv);
    g = idx % a.n_kv;
    const int i = (idx / a.n_kv) % a.B;
    if (c >= MC) return;
    t0 = a.cu[i];
    d = a.cu[i + 1] - t0;
    const int L0 = a.ctx_len[i];
    cap = a.kv_cap[i];
    if (d <= 0) return;
    if (L0 < 0 || L0 + a.D + 1 > cap) {
      if (c == 0 && g == 0 && threadIdx.x == 0 && a.dev_err) atomicOr(a.dev_err, DCUT_DERR_CAPACITY);
    }
    L = usable_ctx(L0, cap, a.D);
    if (c >= n_chunks(L, a.chunk, MC)) return;
    base = a.kv_base[i];
  }
  const int nc = n_chunks(L, a.chunk, MC);
  const int kstart = c * a.chunk;
  int kend = (c == nc - 1) ? L + d : min((c + 1) * a.chunk, L);
  if (kend > cap) kend = cap;

  const int G = a.n_q / a.n_kv;
  const int R = G * d;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, grp4 = lane >> 4;

  // this lane's query rows, one per block
  bool row_ok[RB];
  int trow[RB], head[RB], kmax[RB];   // packed row, query head, last visible key position
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const int rr = (rb * NW + wave) * 16 + l16;
    row_ok[rb] = rr < R;
    const int hl = row_ok[rb] ? rr / d : 0;
    const int krow = row_ok[rb] ? rr - hl * d : 0;
    head[rb] = g * G + hl;
    trow[rb] = t0 + krow;
    kmax[rb] = L + krow;
  }

  bf16x8 qf[RB][NS];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const uint16_t *qp = a.q + ((size_t)trow[rb] * a.n_q + head[rb]) * HD + 8 * grp4;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      if (row_ok[rb]) qf[rb][s] = *(const bf16x8 *)(qp + 32 * s);
      else {
        uint4 z = make_uint4(0, 0, 0, 0);
        qf[rb][s] = *(bf16x8 *)&z;
      }
    }
  }

  floatx4 o[RB][NT];
  float m_run[RB], l_run[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
    for (int n = 0; n < NT; ++n) o[rb][n] = {0.f, 0.f, 0.f, 0.f};
    m_run[rb] = -__builtin_inff();
    l_run[rb] = 0.0f;
  }
  constexpr float sl2 = 1.4426950408889634f / (HD == 128 ? 11.313708498984761f : 8.0f);   // log2(e) / sqrt(hd)
  static_assert(HD == 64 || HD == 128, "sqrt of the head dimension");

  // K and V of the request's kv head g as buffers: out-of-range keys read as zeros
  const size_t slab = (size_t)base + (size_t)g * cap * HD;
  const int slab_bytes = cap * ROWB;
  const __amdgpu_buffer_rsrc_t rK = uniform_rsrc(a.kv_k + slab, slab_bytes);
  const __amdgpu_buffer_rsrc_t rV = uniform_rsrc(a.kv_v + slab, slab_bytes);
  // Tile layout in LDS: key row r at r * ROWB; its 16-byte chunk c holds the
  // row's global chunk c ^ (r % CPR), so 16 consecutive rows read at one column
  // land in different banks.  A wave load fills RPI rows (1 KB): lane l writes
  // row l / CPR, chunk l % CPR.
  const int lrow = lane / CPR, lchk = lane % CPR;
  auto issue = [&](int tile, int slot) {
    const int p0 = kstart + tile * KT;
    unsigned char *st = ring + slot * STAGEB;
#pragma unroll
    for (int j = 0; j < LPK; ++j) {
      const int q = wave + NW * j;                 // 1 KB block of the K (and V) tile
      if (q >= TILEB / 1024) continue;
      const int r = q * RPI + lrow;                // key row within the tile
      const int p = p0 + r;
      const unsigned off = p < kend ? (unsigned)(p * ROWB + 16 * (lchk ^ (r % CPR))) : 0x80000000u;
      // each key is read once: non-temporal loads (cache policy nt) keep the
      // stream from displacing reused lines in L2
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rK, (lds_void *)(st + q * 1024), 16, off, 0, 0, CPOL_NT);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rV, (lds_void *)(st + TILEB + q * 1024), 16, off, 0, 0, CPOL_NT);
    }
  };

  // Fragment addresses within a tile.  K: key row l16 (16-key blocks 16 rows
  // apart), chunk grp4 ^ (row % CPR), k-step s flips chunk bits 2-3.  V: source
  // lane s of a 16-lane group reads key row k0 + s/4, columns 16n + 4(s%4)..+3,
  // and lane d receives keys k0..k0+3 of column 16n + d; the column tile n flips
  // chunk bits 1-3, the second 16 keys lie 16 rows on.
  const int vrow = 4 * grp4 + (l16 >> 2);
  const uint32_t ring0 = (uint32_t)(uintptr_t)(lds_void *)ring;
  const uint32_t kfrag = ring0 + l16 * ROWB + 16 * (grp4 ^ (l16 % CPR));
  const uint32_t vfrag = ring0 + TILEB + vrow * ROWB + 16 * (((l16 & 3) >> 1) ^ (vrow % CPR)) + 8 * (l16 & 1);

  const int ntiles = (kend - kstart + KT - 1) / KT;
#pragma unroll
  for (int s = 0; s < NSTAGE - 1; ++s)
    if (s < ntiles) issue(s, s);
  constexpr int W0 = 0 | (7 << 4) | (15 << 8);
  constexpr int W1 = (LPW & 15) | ((LPW >> 4) << 14) | (7 << 4) | (15 << 8);
  constexpr int W2 = ((2 * LPW) & 15) | (((2 * LPW) >> 4) << 14) | (7 << 4) | (15 << 8);
  for (int tile = 0; tile < ntiles; ++tile) {
    const int pending = min(NSTAGE - 2, ntiles - 1 - tile);
    if (pending >= 2) __builtin_amdgcn_s_waitcnt(W2);
    else if (pending == 1) __builtin_amdgcn_s_waitcnt(W1);
    else __builtin_amdgcn_s_waitcnt(W0);
    ring_barrier();
    if (tile + NSTAGE - 1 < ntiles) issue(tile + NSTAGE - 1, (tile + NSTAGE - 1) % NSTAGE);
    const int p0 = kstart + tile * KT;
    const uint32_t ks = kfrag + (tile % NSTAGE) * STAGEB, vs = vfrag + (tile % NSTAGE) * STAGEB;
    // every key of the tile is visible to every row (block key 0 is the bonus token
    // itself): no masks.  Depends on L and the chunk only, like all of a row's steps.
    const bool full = p0 + KT <= min(kend, L + 1);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
#pragma clang fp contract(off)     // the scaled scores' subtraction stays one (see below)
      if ((rb * NW + wave) * 16 >= R) break;   // uniform: no rows in this block or any later one
      // S^T: two blocks of 16 keys; lane owns keys 4 grp4 + j of each
      floatx4 s4[KT / 16];
#pragma unroll
      for (int kb = 0; kb < KT / 16; ++kb) {
        s4[kb] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          const bf16x8 kf = *(lds_frag *)(uintptr_t)((ks ^ (64 * s)) + kb * 16 * ROWB);
          s4[kb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qf[rb][s], s4[kb], 0, 0, 0);
        }
      }
      if (!full) {
#pragma unroll
        for (int kb = 0; kb < KT / 16; ++kb)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int p = p0 + kb * 16 + 4 * grp4 + j;
            if (p >= kend || p > kmax[rb]) s4[kb][j] = -__builtin_inff();
          }
      }
      // Weights in the exp2 domain.  A score is scaled first and the maximum of the scaled
      // scores subtracted, so the largest weight is exactly 1: scaled inside the
      // subtraction's fma, a score past 2^31 keeps a rounding error of 2^7 and more, whose
      // exp2 overflows.  Costs nothing (batch 64 at 1024 rows 638 us a layer both ways).
#pragma unroll
      for (int kb = 0; kb < KT / 16; ++kb) s4[kb] *= sl2;
      float tmax = fmaxf(fmaxf(s4[0][0], s4[0][1]), fmaxf(s4[0][2], s4[0][3]));
      tmax = fmaxf(tmax, fmaxf(fmaxf(s4[1][0], s4[1][1]), fmaxf(s4[1][2], s4[1][3])));
      tmax = fmaxf(tmax, __shfl_xor(tmax, 16, 64));
      tmax = fmaxf(tmax, __shfl_xor(tmax, 32, 64));
      const float m_new = fmaxf(m_run[rb], tmax);
      // a row that has seen no key yet keeps m = -inf; subtracting 0 then keeps its weights at 0
      const float sub = m_new == -__builtin_inff() ? 0.0f : m_new;
      const float alpha = __builtin_amdgcn_exp2f(m_run[rb] - sub);
      float psum = 0.0f;
#pragma unroll
      for (int kb = 0; kb < KT / 16; ++kb)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float pv = __builtin_amdgcn_exp2f(s4[kb][j] - sub);
          s4[kb][j] = pv;
          psum += pv;
        }
      psum += __shfl_xor(psum, 16, 64);
      psum += __shfl_xor(psum, 32, 64);
      l_run[rb] = __builtin_fmaf(l_run[rb], alpha, psum);
      m_run[rb] = m_new;
#pragma unroll
      for (int n = 0; n < NT; ++n) o[rb][n] *= alpha;

      // O^T += V^T P^T.  P^T slots of this lane: keys 4*grp4+j of the two 16-key
      // blocks; the V^T fragment with the same keys comes from two transposing reads.
      bf16x8 pf;
      uint32_t *pw = (uint32_t *)&pf;
      pw[0] = pack_bf2(s4[0][0], s4[0][1]);
      pw[1] = pack_bf2(s4[0][2], s4[0][3]);
      pw[2] = pack_bf2(s4[1][0], s4[1][1]);
      pw[3] = pack_bf2(s4[1][2], s4[1][3]);
      static_assert(NT % 4 == 0 && KT == 32, "transposing reads come in groups of four columns, one 32-key step");
#pragma unroll
      for (int n0 = 0; n0 < NT; n0 += 4) {
        short4v vr[8];
        lds_read_tr16_x8<16 * ROWB>(vr, vs ^ (32 * n0), vs ^ (32 * (n0 + 1)), vs ^ (32 * (n0 + 2)), vs ^ (32 * (n0 + 3)));
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          bf16x8 vf;
          short4v *vw = (short4v *)&vf;
          vw[0] = vr[2 * u];
          vw[1] = vr[2 * u + 1];
          o[rb][n0 + u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pf, o[rb][n0 + u], 0, 0, 0);
        }
      }
    }
  }
  // lane holds O^T[16n + 4*grp4 + j][row]
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    if (!row_ok[rb]) continue;
    if (nc == 1) {
      const float inv = l_run[rb] > 0.0f ? 1.0f / l_run[rb] : 0.0f;
      uint16_t *op = a.out + ((size_t)trow[rb] * a.n_q + head[rb]) * HD;
#pragma unroll
      for (int n = 0; n < NT; ++n)
        *(uint2 *)(op + 16 * n + 4 * grp4) = make_uint2(pack_bf2(o[rb][n][0] * inv, o[rb][n][1] * inv),
                                                        pack_bf2(o[rb][n][2] * inv, o[rb][n][3] * inv));
    } else {
      float *pp = a.part + (((size_t)trow[rb] * a.n_q + head[rb]) * MC + c) * ATTN_PITCH(HD);
#pragma unroll
      for (int n = 0; n < NT; ++n)
        *(float4 *)(pp + 16 * n + 4 * grp4) = make_float4(o[rb][n][0], o[rb][n][1], o[rb][n][2], o[rb][n][3]);
      if (grp4 == 0) {
        pp[HD] = m_run[rb];
        pp[HD + 1] = l_run[rb];
      }
    }
  }
}

// Merge of a (row, head)'s chunk partials, one half wave each: lane c reads chunk
// c's (max, sum), so the weights of up to 32 chunks cost one memory round trip,
// taken together with the first eight chunks' values.  Values add up in chunk
// order.  Latency-bound (three dependent loads: row and count, context, partials),
// so a wave carries two pairs and reads its row's index beside the live row count.
template <int HD>
__global__ void __launch_bounds__(256)
k_attn_combine(AttnArgs a, const int32_t *__restrict__ packed_req, int rows_max) {
  constexpr int PER = HD / 32, CG = 8;
  const int lane = threadIdx.x & 31;
  const int pair = blockIdx.x * 8 + (threadIdx.x >> 5);
  const int t = pair / a.n_q, head = pair - t * a.n_q;
  const int req0 = packed_req[min(t, rows_max - 1)];
  const int M = a.cu[a.B];
  if (t >= M || t >= rows_max) return;
  if (req0 < 0 || req0 >= a.B) return;
  const int MC = a.max_chunks;
  const int L = usable_ctx(a.ctx_len[req0], a.kv_cap[req0], a.D);
  const int nc = n_chunks(L, a.chunk, MC);
  if (nc == 1) return;
  const float *pp = a.part + (size_t)pair * MC * ATTN_PITCH(HD);
  float acc[PER];
#pragma unroll
  for (int e = 0; e < PER; ++e) acc[e] = 0.0f;
  float mx = -__builtin_inff(), lsum = 0.0f;
  for (int c0 = 0; c0 < nc; c0 += 32) {
    const int cnt = min(32, nc - c0);
    const float *p0 = pp + (size_t)c0 * ATTN_PITCH(HD);
    float xv[CG][PER];
    auto load = [&](int cc) {
#pragma unroll
      for (int u = 0; u < CG; ++u)
#pragma unroll
        for (int e = 0; e < PER; ++e) xv[u][e] = cc + u < cnt ? p0[(cc + u) * ATTN_PITCH(HD) + lane * PER + e] : 0.0f;
    };
    load(0);
    const float mv = lane < cnt ? p0[lane * ATTN_PITCH(HD) + HD] : -__builtin_inff();
    const float lv = lane < cnt ? p0[lane * ATTN_PITCH(HD) + HD + 1] : 0.0f;
    float gm = mv;
#pragma unroll
    for (int off = 16; off > 0; off >>= 1) gm = fmaxf(gm, __shfl_xor(gm, off, 32));
    const float mn = fmaxf(mx, gm), sub = mn == -__builtin_inff() ? 0.0f : mn;
    const float w = __builtin_amdgcn_exp2f(mv - sub);         // 0 for an empty chunk
    float ls = lv * w;
#pragma unroll
    for (int off = 16; off > 0; off >>= 1) ls += __shfl_xor(ls, off, 32);
    const float old = __builtin_amdgcn_exp2f(mx - sub);
    lsum = lsum * old + ls;
    mx = mn;
#pragma unroll
    for (int e = 0; e < PER; ++e) acc[e] *= old;
    for (int cc = 0;; cc += CG) {
#pragma unroll
      for (int u = 0; u < CG; ++u) {
        const float wc = __shfl(w, cc + u, 32);
#pragma unroll
        for (int e = 0; e < PER; ++e) acc[e] += xv[u][e] * wc;
      }
      if (cc + CG >= cnt) break;
      load(cc + CG);
    }
  }
  const float inv = lsum > 0.0f ? 1.0f / lsum : 0.0f;
  uint16_t *op = a.out + (size_t)pair * HD + lane * PER;
#pragma unroll
  for (int e = 0; e < PER; e += 2) *(uint32_t *)(op + e) = pack_bf2(acc[e] * inv, acc[e + 1] * inv);
}

template <int HD>
int launch_hd(const AttnArgs &a, int rows_max, const int32_t *packed_req, int waves, hipStream_t s) {
  // Up to 128 rows per item: 4 waves and a 3-stage ring, three workgroups per
  // CU, so one streams on while another starts or finishes an item; above 64
  // rows a wave owns two row blocks.  Up to 256 rows: 16 waves and a 4-stage
  // ring, one workgroup per CU.
  const dim3 grid(a.B * a.n_kv * a.max_chunks);
  if (waves <= 4) {
    DCUT_TRY(launch(DCUT_KERNEL_ATTN, k_attn<HD, 4, 3, 1>, grid, dim3(256), 0, s, a));
  } else if (waves <= 8) {
    DCUT_TRY(launch(DCUT_KERNEL_ATTN, k_attn<HD, 4, 3, 2>, grid, dim3(256), 0, s, a));
  } else {
    DCUT_TRY(launch(DCUT_KERNEL_ATTN, k_attn<HD, 16, 4, 1>, grid, dim3(1024), 0, s, a));
  }
  if (a.max_chunks == 1) return DCUT_OK;      // every request is finished in place
  return launch(DCUT_KERNEL_ATTN_COMBINE, k_attn_combine<HD>, dim3((rows_max * a.n_q + 7) / 8), dim3(256), 0, s, a,
                packed_req, rows_max);
}

}  // namespace

size_t attn_plan_bytes(int B, int n_kv, int max_chunks) {
  // a grid that fits in one round of workgroup slots gains nothing from an order
  if (B > PLAN_MAX_B || (long long)B * n_kv * max_chunks <= PLAN_MIN_ITEMS) return 0;
  return PLAN_HEAD + (size_t)B * n_kv * max_chunks * 8 * sizeof(int32_t);
}

int attention_launch(const AttnArgs &a, int rows_max, const int32_t *packed_req, int waves, hipStream_t s) {
  if (a.plan && a.B > PLAN_MAX_B) return DCUT_EINVAL;
  if (a.head_dim == 128) return launch_hd<128>(a, rows_max, packed_req, waves, s);
  if (a.head_dim == 64) return launch_hd<64>(a, rows_max, packed_req, waves, s);
  return DCUT_EUNSUPPORTED;
}

}  // namespace dcut
