// bf16 NT GEMM on gfx950 MFMA with fused epilogues: C = A W^T, A [M][K], W [N][K].
//
// Tile shapes of one kernel template (32x32x16 bf16 MFMA, float32
// accumulators, k-slices of 64), with the A and W ring stages of each:
//   Big      256 x 256, eight waves in a 4 x 2 grid, each wave 64 x 128, 2 + 3 stages:
//            160 KB of LDS, one workgroup per CU (many live rows);
//   Mid      128 x 256, eight waves, 2 + 3 stages; MidDeep 2 + 4 (LM head);
//   Deep     128 x 128, eight waves, 3 + 5 stages, one workgroup per CU (few live
//            rows); DeepPair the same for epilogues that pair column groups;
//   Small    128 x 128, four waves in a 2 x 2 grid, each wave 64 x 64, 2 + 3 stages:
//            80 KB of LDS, two workgroups per CU (grouped MoE GEMMs, small LM heads).
// Operands stream from memory straight into LDS (buffer loads with the LDS
// destination, 128-byte rows of 64 k split in XOR-swizzled 16-byte chunks,
// hardware zeros for rows and k beyond the operands).  A and W have rings of
// their own: of A (activations, mostly L2-resident) one or two slices are in flight,
// of W (weights, streamed from HBM) two to four, so a W slice is requested that many
// k-steps before it is multiplied.  Fragment reads of the next 16-k step are issued
// before the MFMAs of the current one.
//
// What bounds it and what the k loop does about it (measured with loads-only and
// compute-only copies): a CU takes 45-60 GB/s out of L2 whatever the source, so at
// up to 256 live rows the loads alone take as long as the kernel, and the MFMAs
// have to hide under them.
//   - A slice's loads are spread evenly over its MFMAs instead of issued in one
//     burst after the barrier: a wave waits in the load queue for less time, and
//     its MFMAs go out meanwhile.  Slices past the end are loaded too (from beyond
//     the buffer: no memory traffic), so the count of loads in flight is a constant.
//   - The k loop starts at a slice that depends on the column (rot): 28672 rows of
//     8 KB read at the same k put their lines in the same few memory channels.  A
//     stream of 235 MB in that order runs at 4.8 TB/s, and at 6.4 TB/s with the
//     start shifted over the column eighths (the range of one XCD, whose CUs keep
//     sharing the activations in L2).
//   Batch 64, 4096 x 128256 LM head: 940 -> 866 us at 1024 rows; SwiGLU 4096 x 28672:
//   229 -> 210 us at 1024 rows, 63 -> 57 us at 128; 128 experts of 2048 x 1536 at 768
//   rows: 198 -> 174 us (one card, both sides in turn).
//
// Scheduling: the grid is persistent (at most one wave of workgroups); every
// workgroup reads the live row count M (K*) on the device and walks only the
// tiles that exist, so rows beyond K* cost nothing.  Tasks (row tile, column
// tile, k split) are numbered with the row tile fastest and the split slowest
// (grouped: expert by expert, an expert's row tiles fastest) and cut into eight contiguous ranges, one per XCD (the hardware deals
// workgroups round-robin over the eight XCDs): row tiles sharing a W slice run
// at the same time on the same L2, and an XCD reads the A columns of one or
// two splits only, not all of A.
//
// Determinism and causality: every output element is the same sequence of
// MFMA k-steps whatever the tile shape (from the slice `rot` upwards, then from
// k = 0; rot depends on the column's 256-column block, the expert and the
// shapes only); split-K partials are added in split order, and the split factor
// depends on M_max (the grid's row bound), never on M.  The tile may follow M,
// since it changes no bit.  A row's bits therefore do not depend on which or how
// many other rows are present.
//
// Column groups: each 32-column MFMA tile loads a 32-row group of W chosen by
// the epilogue, so that values an epilogue combines sit in the same lane:
//   SWIGLU    groups (2p, 2p+1) = (gate rows, up rows) of the same 32 outputs;
//   QKV_ROPE  groups (2p, 2p+1) = the two halves (j, j + hd/2) of RoPE pairs.

#include <atomic>
#include <type_traits>

#include "dcut_internal.h"
#include "rng.h"

namespace dcut {

namespace {

// Two waves a SIMD is what the LDS of every tile allows, which the compiler cannot see
// (dynamic LDS): told so, it keeps the k loop's order of loads, reads and MFMAs instead of
// trading it for registers it does not need.  Batch-1 layer 115.7 -> 113.7 us, smallest
// step 72.1 -> 71.0, long kernels alike.
#define TWO_WAVES __attribute__((amdgpu_waves_per_eu(2, 2)))

constexpr int TK = 64;       // k per LDS stage: one 128-byte row per operand row
constexpr int CPR = TK / 8;  // 16-byte chunks per row
constexpr int RPI = 64 / CPR;  // rows per 1 KB wave load

template <int GM_, int GN_, int WM_, int WN_, int NA_ = 2, int NB_ = 3, bool SKEW_ = false>
struct Tile {
  static constexpr int GM = GM_, GN = GN_, WM = WM_, WN = WN_;
  static constexpr bool SKEW = SKEW_;   // second half of the waves two sub-steps behind (8-wave tiles)
  static constexpr int NWV = GM * GN, THREADS = 64 * NWV;
  static constexpr int TM = GM * WM * 32, TN = GN * WN * 32;
  // ring stages of A and W: slice it + NA - 1 of A and it + NB - 1 of W are
  // requested while slice it is multiplied
  static constexpr int NA = NA_, NB = NB_;
  static_assert(NA >= 2 && NB >= 2, "double buffering at least");
  static constexpr size_t LDS = (size_t)(NA * TM + NB * TN) * TK * sizeof(uint16_t);
  static_assert(LDS <= 163840, "the LDS of one CU");
  static constexpr int PER_CU = LDS > 81920 ? 1 : 2;
};
using Big = Tile<4, 2, 2, 4, 2, 3, true>;
using Mid = Tile<2, 4, 2, 2, 2, 3, true>;     // 128 x 256, eight waves in a 2 x 4 grid, 128 KB
using Small = Tile<2, 2, 2, 2>;
using Deep = Tile<2, 4, 2, 1, 3, 5>;          // 128 x 128, eight waves, three A and five W slices: 128 KB, one per CU
using DeepPair = Tile<4, 2, 1, 2, 3, 5>;      // the same with two column groups per wave, for the paired epilogues
using MidDeep = Tile<2, 4, 2, 2, 2, 4, true>;   // 128 x 256 with four W slices: the LM head at few live rows
using BigFlat = Tile<4, 2, 2, 4>;   // Big without the skew: the sampling epilogue needs its registers

__device__ __forceinline__ float silu(float g) { return g / (1.0f + __expf(-g)); }

// LDS chunk swizzle of row r: 16 consecutive rows of one chunk column land in
// 16 different 16-byte bank groups, and so do any 8 consecutive rows.  Rows 32
// apart share it, so a wave's fragment addresses differ by constants only.
__device__ __forceinline__ int swz(int r) { return (r ^ ((r >> 3) & 3)) & (CPR - 1); }

// Workgroup barrier for the LDS rings: each wave has already waited (s_waitcnt
// vmcnt) for its own loads of the stage it is about to read, so no memory fence
// (which would drain every stage still in flight) is needed, only the hardware
// barrier; the empty asm statements keep the compiler from moving LDS accesses
// across it.
__device__ __forceinline__ void ring_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// s_waitcnt immediate: at most N vector-memory operations outstanding
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt is six bits");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// W row feeding logical tile column group `grp` (global, 32 columns each);
// -1 when the group is past N.
template <int EPI>
__device__ __forceinline__ int group_wrow(const GemmArgs &a, int grp) {
  if (EPI == EPI_SWIGLU) {
    int p = grp >> 1;                       // output block of 32 columns
    if (p * 32 >= a.swiglu_inter) return -1;
    return (grp & 1) ? a.swiglu_inter + p * 32 : p * 32;
  } else if (EPI == EPI_QKV_ROPE) {
    int hd = a.head_dim;
    int gph = hd / 32;                      // groups per head (2 or 4)
    int head = grp / gph, wg = grp - head * gph;
    int base;
    if (gph == 4) {
      const int perm[4] = {0, 64, 32, 96};
      base = perm[wg];
    } else {
      base = wg * 32;
    }
    int row = head * hd + base;
    return row < a.N ? row : -1;
  } else {
    int row = grp * 32;
    return row < a.N ? row : -1;
  }
}

template <int EPI>
__host__ __device__ __forceinline__ int n_col_tiles(const GemmArgs &a, int TN) {
  return EPI == EPI_SWIGLU ? (a.swiglu_inter + TN / 2 - 1) / (TN / 2) : (a.N + TN - 1) / TN;
}

// QKV epilogue for one RoPE pair of one row: x1, x2 = projections at head
// dimensions j and j + hd/2.  q and k heads are rotated; q goes to out_bf16, k
// and v to the request's cache slot (slots outside the cache are skipped; the
// norm kernel reports them).
__device__ __forceinline__ void qkv_emit(const GemmArgs &a, int gm, int head, int j, float x1, float x2) {
  const int hd = a.head_dim, half = hd >> 1;
  float o1 = x1, o2 = x2;
  if (head < a.n_q + a.n_kv) {
    const float2 r = rope_pair(x1, x2, a.rope_cs[(size_t)gm * half + j]);
    o1 = r.x;
    o2 = r.y;
  }
  if (head < a.n_q) {
    uint16_t *q = a.out_bf16 + (size_t)gm * a.ldo + head * hd;
    q[j] = f2bf(o1);
    q[j + half] = f2bf(o2);
  } else {
    const int req = a.packed_req[gm];
    if ((unsigned)req >= (unsigned)a.n_req) return;   // not a row of this batch
    const int slot = a.packed_pos[gm];
    const int cap = a.kv_cap[req];
    if (slot < 0 || slot >= cap) return;
    const int g = (head < a.n_q + a.n_kv) ? head - a.n_q : head - a.n_q - a.n_kv;
    uint16_t *dst = (head < a.n_q + a.n_kv ? a.kv_k : a.kv_v) + a.kv_base[req] + ((size_t)g * cap + slot) * hd;
    dst[j] = f2bf(o1);
    dst[j + half] = f2bf(o2);
  }
}

// First k of the slice after the one at k0, going round over the task's slices kt0 .. kt0 + nk - 1.
constexpr __host__ __device__ int next_slice(int k0, int kt0, int nk) {
  return k0 + TK == (kt0 + nk) * TK ? kt0 * TK : k0 + TK;
}
constexpr bool slices_in_range() {       // short and long loops, some turns past the last slice
  for (int nk = 1; nk <= 6; ++nk)
    for (int rot = 0; rot < nk; ++rot)
      for (int it = 0, k0 = (3 + rot) * TK; it < 3 * nk + 6; ++it, k0 = next_slice(k0, 3, nk))
        if (k0 != (3 + (rot + it) % nk) * TK) return false;
  return true;
}
static_assert(slices_in_range(), "the slices in turn, none past the task's last");

typedef __attribute__((address_space(3))) const bf16x8 lds_frag;
typedef __attribute__((address_space(3))) void lds_void;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *base, long long bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void *)base, (short)0,
                                           (int)(bytes < 0x7fffffffLL ? bytes : 0x7fffffffLL), 0x00020000);
}

template <int EPI, class T, int WPOL, bool GROUPED = false>
__device__ __forceinline__ void gemm_tasks(const GemmArgs &a) {
  constexpr int GN = T::GN, WM = T::WM, WN = T::WN, NWV = T::NWV;
  constexpr int TM = T::TM, TN = T::TN, NA = T::NA, NB = T::NB;
  constexpr int AJ = TM / (NWV * RPI), BJ = TN / (NWV * RPI);   // load instructions per wave per stage
  static_assert(AJ * NWV * RPI == TM && BJ * NWV * RPI == TN, "tile rows must fill whole wave loads");
  static_assert(NWV % 4 == 0, "the swizzle of a lane's rows is the same in every load");
  extern __shared__ __align__(16) uint16_t lds[];   // [NA][TM*TK] (A), then [NB][TN*TK] (W)
  constexpr int ASTAGE = TM * TK * 2, WSTAGE = TN * TK * 2;     // bytes
  constexpr unsigned OOB = 0x80000000u;

  // the wave index is uniform: kept in a scalar register, so LDS destinations
  // of the operand loads are scalar arithmetic
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / GN, wn = wave % GN;
  const int l32 = lane & 31, kh = lane >> 5;
  const int lr = lane / CPR, lc = lane % CPR;

  // live tasks: (row tile, column tile, split), row tile fastest, split slowest
  const int M = min(__builtin_amdgcn_readfirstlane(*a.m_count), a.M_max);
  const unsigned nMT = GROUPED ? __builtin_amdgcn_readfirstlane(*a.n_tiles) : (M + TM - 1) / TM;
  const unsigned nNT = n_col_tiles<EPI>(a, TN);
  constexpr bool SPLIT = !GROUPED && (EPI == EPI_RESID_F32 || EPI == EPI_STORE_F32 || EPI == EPI_QKV_ROPE);
  const int splits = SPLIT && a.splits > 1 ? a.splits : 1;
  const unsigned ntask = nMT * nNT * splits;
  const unsigned xcd = blockIdx.x & 7, per_xcd = gridDim.x >> 3;
  const unsigned lo = (unsigned)(((unsigned long long)ntask * xcd) >> 3);
  const unsigned hi = (unsigned)(((unsigned long long)ntask * (xcd + 1)) >> 3);

  const int nk_all = (a.K + TK - 1) / TK;
  const int per_split = (nk_all + splits - 1) / splits;
  // Buffer resources take 32-bit offsets: each task addresses A from its first
  // row (or, for gathered rows, from the start of A) and W from the first
  // weight row of its column tile, so the offsets stay below 2^31 for any
  // operand size the host checks admit (gemm_span_ok).
  const int w_rows_ext = (EPI == EPI_SWIGLU) ? 2 * a.swiglu_inter : a.N;
  // Each wave load instruction fills one 1 KB block = 8 rows x 64 k; row r's
  // 16-byte chunk c holds global chunk c ^ swz(r), swz being the same for this
  // lane's row in every load (rows 8 * NWV apart).
  const int kchunk = 8 * (lc ^ swz(RPI * wave + lr));   // first k of this lane's chunk within a slice
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_void *)lds;
  // fragment read addresses: row l32 of the wave's first row (column) block,
  // chunk kh; the 16-k sub-step ks flips chunk bits 1-2, blocks are 4 KB apart
  const uint32_t frow = (uint32_t)(l32 * TK * 2 + 16 * (kh ^ swz(l32)));
  const uint32_t fragA = lds0 + wm * WM * 4096 + frow;
  const uint32_t fragW = lds0 + NA * ASTAGE + wn * WN * 4096 + frow;

  // One task's position and operand addresses; setup() fills them and starts the
  // task's first loads.
  int m0, Mlim, grp0, kt0, nk, rot;
  int kA, kW;             // first k of the next A and W slices to load
  unsigned sp, nt;
  __amdgpu_buffer_rsrc_t rsA, rsW;
  unsigned aoff[AJ], boff[BJ];
  // The k offset of a slice goes in the scalar offset; the per-lane offsets
  // stay fixed over the k loop.  `kill` is zero, or OOB for a slice past the
  // task's last (issued all the same, so that the count of loads in flight
  // stays constant) and for chunks beyond K in a slice that reaches past it.
  // The slices go round (next_slice), also past the last one, so that no scalar
  // offset ever passes the operand's end.
  auto kill = [&](int it, int k0) { return ((unsigned)(it >= nk) | (unsigned)(kchunk >= a.K - k0)) << 31; };
  auto step = [&](int k0) { return next_slice(k0, kt0, nk); };
  auto issueA = [&](int j, int koff, unsigned kill, uint32_t stage) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsA, (lds_void *)(uintptr_t)(lds0 + stage + (wave + NWV * j) * 1024), 16,
                                             aoff[j] | kill, koff, 0, 0);
  };
  auto issueW = [&](int j, int koff, unsigned kill, uint32_t stage) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsW, (lds_void *)(uintptr_t)(lds0 + NA * ASTAGE + stage + (wave + NWV * j) * 1024),
                                             16, boff[j] | kill, koff, 0, WPOL);
  };
  constexpr int PA = NA - 1, PW = NB - 1;   // slices in flight ahead of the one multiplied
  constexpr int PMAX = PA > PW ? PA : PW;
  static_assert(PW >= PA, "W runs at least as far ahead as A");
  constexpr int NL = AJ + BJ, NM = TK / 16 * WM * WN;   // loads and MFMAs per slice
  // loads issued after A[it] and W[it] were, when iteration `it` needs them:
  // the W loads of A[it]'s own iteration (when W runs further ahead) and the
  // iterations in between
  constexpr int PEND = (PW > PA ? BJ : 0) + (PA - 1) * NL;
  static_assert(PMAX * NL <= 63, "outstanding loads within the vmcnt range");

  auto setup = [&](unsigned task) {
    const uint16_t *Wb = a.W;
    int e = 0;
    if constexpr (GROUPED) {
      // experts slowest, an expert's row tiles fastest: the row tiles that multiply one
      // slice of its weights run at the same time, and its rows are read by its column
      // tiles in a row.  Task numbers of an expert start at its first tile's share.
      // (uniform, but loaded through the vector path: kept scalar)
      const int32_t *t = a.tiles + 3 * (task / nNT);
      const int id = __builtin_amdgcn_readfirstlane(t[0]), first = __builtin_amdgcn_readfirstlane(t[1]);
      Mlim = __builtin_amdgcn_readfirstlane(t[2]);
      e = id & 255;
      const unsigned q = task - (unsigned)(id >> 8) * nNT, nr = (Mlim - first + TM - 1) / TM;
      nt = q / nr;
      m0 = first + (q - nt * nr) * TM;
      sp = 0;
      Wb += (size_t)e * a.w_stride;
    } else {
      const unsigned rest = task / nMT;
      sp = splits > 1 ? rest / nNT : 0;
      nt = rest - sp * nNT;
      m0 = (task - rest * nMT) * TM;
      Mlim = M;
    }
    kt0 = sp * per_split;
    nk = max(0, min(nk_all, kt0 + per_split) - kt0);
    grp0 = nt * (TN / 32);
    // First slice of the k loop: spread over the column eighths, or, for grouped
    // tasks (each reads weights of its own), over experts and column tiles.  With
    // split-K the splits start apart already (a shift on top measured no faster).
    // Logits all start at k = 0: equal weight rows have to give equal logits.
    rot = 0;
    if constexpr (GROUPED) {
      rot = nk > 0 ? (int)((e * nNT + nt) * 5u % (unsigned)nk) : 0;
    } else if (splits == 1 && EPI != EPI_ARGMAX && EPI != EPI_SAMPLE) {
      const unsigned n256 = (nNT * (TN / 32) + 7) / 8;
      rot = (int)((grp0 / 8) * 8u / n256) * nk / 8;
    }
    // the lowest W row of the tile: its first column group (gate rows precede
    // up rows; a head's first group is its first 32 dimensions)
    const int wrow0 = max(group_wrow<EPI>(a, grp0), 0);
    rsW = make_rsrc(Wb + (size_t)wrow0 * a.ldw, (long long)(w_rows_ext - wrow0) * a.ldw * 2);
    const bool gather = GROUPED && a.a_rows != nullptr;
    rsA = gather ? make_rsrc(a.A, (long long)a.a_extent * a.lda * 2)
               : make_rsrc(a.A + (size_t)m0 * a.lda, (long long)(Mlim - m0) * a.lda * 2);

    // Byte offsets of this lane's loads at k = 0.  Rows past the operand lie
    // beyond the buffer (A: Mlim ends it; W: the last row does, and the last
    // gate rows of an odd tile read up rows that no output uses) and read as
    // zeros; gathered rows past Mlim get an offset beyond it.
    if (gather) {
      int src[AJ];
#pragma unroll
      for (int j = 0; j < AJ; ++j) src[j] = a.a_rows[min(m0 + RPI * (wave + NWV * j) + lr, Mlim - 1)];
#pragma unroll
      for (int j = 0; j < AJ; ++j)
        aoff[j] = m0 + RPI * (wave + NWV * j) + lr < Mlim ? (unsigned)(src[j] * a.lda + kchunk) * 2 : OOB;
    } else {
#pragma unroll
      for (int j = 0; j < AJ; ++j) aoff[j] = (unsigned)((RPI * (wave + NWV * j) + lr) * a.lda + kchunk) * 2;
    }
#pragma unroll
    for (int j = 0; j < BJ; ++j) {
      const int blk = wave + NWV * j;                   // 8-row block of the tile: all in one 32-row group
      const int wr = group_wrow<EPI>(a, grp0 + (blk >> 2));
      boff[j] = wr < 0 ? OOB : (unsigned)((wr - wrow0 + RPI * (blk & 3) + lr) * a.ldw + kchunk) * 2;
    }
    // prologue: A[0 .. PA-1] and W[0 .. PW-1], interleaved by slice
    int k0 = (kt0 + rot) * TK;
#pragma unroll
    for (int q = 0; q < PMAX; ++q) {
      const unsigned dead = kill(q, k0);
      if (q == PA) kA = k0;
      if (q < PA) {
#pragma unroll
        for (int j = 0; j < AJ; ++j) issueA(j, k0 * 2, dead, q * ASTAGE);
      }
      if (q < PW) {
#pragma unroll
        for (int j = 0; j < BJ; ++j) issueW(j, k0 * 2, dead, q * WSTAGE);
      }
      k0 = step(k0);
    }
    kW = k0;
    if (PA == PMAX) kA = k0;
  };

  // The argmax LM head requests the next task's first slices before this one's
  // epilogue, which hides their latency (768 rows of 2048 x 151936, seven tasks per
  // CU: 397 -> 388 us; 1024 rows of 4096 x 128256: 833 -> 820).  They go to the stages
  // 0 .. PA-1 and 0 .. PW-1; the epilogue uses the last stage of W, which the next task
  // fills only after its first barrier.  The other GEMMs have one or two tasks per CU
  // and lost up to 0.9 % to the registers it holds (sampling LM head 320 -> 323).
  constexpr bool EARLY = EPI == EPI_ARGMAX;
  unsigned task = lo + (blockIdx.x >> 3);
  if (EARLY && task < hi) setup(task);
  while (task < hi) {
    if (!EARLY) setup(task);
    floatx16 acc[WM][WN];
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
      for (int j = 0; j < WN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

    // One slice's loads are spread over its MFMAs: A[it + PA] first, then
    // W[it + PW].  State of the iteration: read and write stages, load operands.
    uint32_t raS = 0, rwS = 0, waS = PA * ASTAGE, wwS = PW * WSTAGE;
    int ka, kw;
    unsigned killA, killW;
    auto begin = [&](int it) {
      if constexpr (EPI == EPI_SAMPLE) {
        // the same slices from the iteration (this loop starts at k = 0 and is whole): two
        // scalars less to carry through the largest epilogue, 4096 x 16000 at 128 rows
        // 63.2 -> 61.4 us
        kA = (it + PA < nk ? it + PA : 0) * TK;
        kW = (it + PW < nk ? it + PW : 0) * TK;
      }
      ka = kA * 2;
      kw = kW * 2;
      killA = kill(it + PA, kA);
      killW = kill(it + PW, kW);
      kA = step(kA);
      kW = step(kW);
    };
    auto advance = [&]() {
      raS = raS == (NA - 1) * ASTAGE ? 0 : raS + ASTAGE;
      rwS = rwS == (NB - 1) * WSTAGE ? 0 : rwS + WSTAGE;
      waS = waS == (NA - 1) * ASTAGE ? 0 : waS + ASTAGE;
      wwS = wwS == (NB - 1) * WSTAGE ? 0 : wwS + WSTAGE;
    };
    auto load_at = [&](int m) {               // the loads issued right after MFMA m of the slice
#pragma unroll
      for (int l = 0; l < NL; ++l) {
        if (l * NM / NL != m) continue;
        if (l < AJ) issueA(l, ka, killA, waS);
        else issueW(l - AJ, kw, killW, wwS);
        __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
      }
    };
    // One 16-k sub-step: the WM x WN MFMAs on the fragments in (fa, fb), each
    // fragment register refilled with sub-step nks of the stage at (pa, pw)
    // right after its last use (A fragment i after MFMA (i, WN-1), W fragment
    // j after MFMA (WM-1, j)), so one set of fragment registers serves the
    // pipeline; nks < 0 refills nothing.  q: the sub-step's place among the
    // slice's loads (negative: none).
    auto substep = [&](bf16x8 (&fa)[WM], bf16x8 (&fb)[WN], uint32_t pa, uint32_t pw, int nks, int q) {
      const uint32_t xa = pa ^ (nks * 32), xw = pw ^ (nks * 32);
#pragma unroll
      for (int i = 0; i < WM; ++i) {
#pragma unroll
        for (int j = 0; j < WN; ++j) {
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          if (nks >= 0 && i == WM - 1) {
            fb[j] = *(lds_frag *)(uintptr_t)(xw + j * 4096);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
          }
          if (q >= 0) load_at(q * WM * WN + i * WN + j);
        }
        if (nks >= 0) {
          fa[i] = *(lds_frag *)(uintptr_t)(xa + i * 4096);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
      }
    };
    auto first_frags = [&](uint32_t pa, uint32_t pw, bf16x8 (&fa)[WM], bf16x8 (&fb)[WN]) {
#pragma unroll
      for (int i = 0; i < WM; ++i) fa[i] = *(lds_frag *)(uintptr_t)(pa + i * 4096);
#pragma unroll
      for (int j = 0; j < WN; ++j) fb[j] = *(lds_frag *)(uintptr_t)(pw + j * 4096);
    };
    bf16x8 fa[WM], fb[WN];
    if (T::SKEW && wave >= NWV / 2) {
      // The second half of the waves runs one 16-k sub-step behind the first:
      // at each barrier it holds the last sub-step of the previous slice in
      // registers, so on every SIMD one wave has MFMAs ready while the other
      // waits for its first fragments.  Each accumulator still takes the k
      // sub-steps in order.
      for (int it = 0; it < nk; ++it) {
        begin(it);
        wait_vm<PEND>();
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the previous slice is out of LDS
        ring_barrier();
        const uint32_t pa = fragA + raS, pw = fragW + rwS;
        if (it == 0) {
          first_frags(pa, pw, fa, fb);
#pragma unroll
          for (int m = 0; m < WM * WN; ++m) load_at(m);
        } else {
          substep(fa, fb, pa, pw, 0, 0);              // last sub-step of the previous slice
        }
#pragma unroll
        for (int ks = 0; ks < TK / 16 - 1; ++ks) substep(fa, fb, pa, pw, ks + 1, ks + 1);
        advance();
      }
      if (nk > 0) substep(fa, fb, 0, 0, -1, -1);
    } else {
      for (int it = 0; it < nk; ++it) {
        begin(it);
        wait_vm<PEND>();
        ring_barrier();
        const uint32_t pa = fragA + raS, pw = fragW + rwS;
        first_frags(pa, pw, fa, fb);
#pragma unroll
        for (int ks = 0; ks < TK / 16; ++ks) substep(fa, fb, pa, pw, ks + 1 < TK / 16 ? ks + 1 : -1, ks);
        advance();
      }
    }
    // every wave is done with the rings, and no load is left in flight, before
    // the epilogue or the next task's prologue writes them
    wait_vm<0>();
    ring_barrier();

    // this task's place, for its epilogue
    const int em0 = m0, eMlim = Mlim, egrp0 = grp0;
    const unsigned esp = sp, ent = nt;
    task += per_xcd;
    if (EARLY && task < hi) setup(task);

    // accumulator element r of a 32x32 tile: row 8*(r/4) + 4*(lane/32) + r%4, column lane%32
    if (splits > 1 || EPI == EPI_STORE_F32 || EPI == EPI_RESID_F32) {
      // float32 rows at the true output columns: split-K partials (the reduce
      // pass adds the splits in order and applies the epilogue), plain stores or
      // residual adds.  The buffer ends at row eMlim, so rows past it are dropped; each
      // block of 32 rows has a buffer of its own, whose offsets stay below 2^31 at any width.
      const bool part = splits > 1;
      const int ld = part ? a.N : a.ldo;
      static_assert(32 * 4 * MAX_QKV_COLS < 0x80000000LL, "a block's rows lie within 32-bit offsets");
      float *base = part ? a.split_part + (size_t)esp * a.M_max * a.N : a.out_f32;
#pragma unroll
      for (int j = 0; j < WN; ++j) {
        const int wr = group_wrow<EPI>(a, egrp0 + wn * WN + j);
        if (wr < 0) continue;
        const unsigned v0 = wr + l32 < a.N ? (unsigned)(4 * kh * ld + wr + l32) * 4 : OOB;
#pragma unroll
        for (int i = 0; i < WM; ++i) {
          const int rw = em0 + (wm * WM + i) * 32;         // the block's first row
          const __amdgpu_buffer_rsrc_t rs = make_rsrc(base + (size_t)rw * ld, (long long)max(eMlim - rw, 0) * ld * 4);
          if (EPI == EPI_RESID_F32 && !part) {
            float old[16];
#pragma unroll
            for (int r = 0; r < 16; ++r)
              old[r] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, v0 + (8 * (r >> 2) + (r & 3)) * ld * 4, 0, 0));
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = old[r] + acc[i][j][r];
          }
#pragma unroll
          for (int r = 0; r < 16; ++r)
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[i][j][r]), rs,
                                                  v0 + (8 * (r >> 2) + (r & 3)) * ld * 4, 0, 0);
        }
      }
      continue;
    }

    // ------------------------------------------------------------ epilogues
    const int rbase = em0 + wm * WM * 32 + 4 * (lane >> 5);
    if constexpr (EPI == EPI_SWIGLU) {
      const int rw = em0 + wm * WM * 32;
      const __amdgpu_buffer_rsrc_t rs = make_rsrc(a.out_bf16 + (size_t)rw * a.ldo, (long long)max(eMlim - rw, 0) * a.ldo * 2);
#pragma unroll
      for (int p = 0; p < WN / 2; ++p) {
        const int col = (egrp0 + wn * WN + 2 * p) / 2 * 32 + l32;
        const unsigned v0 = col < a.swiglu_inter ? (unsigned)(4 * kh * a.ldo + col) * 2 : OOB;
#pragma unroll
        for (int i = 0; i < WM; ++i)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const float v = silu(acc[i][2 * p][r]) * acc[i][2 * p + 1][r];
            __builtin_amdgcn_raw_buffer_store_b16(f2bf(v), rs, v0 + (i * 32 + 8 * (r >> 2) + (r & 3)) * a.ldo * 2, 0, 0);
          }
      }
    } else if constexpr (EPI == EPI_QKV_ROPE && WN % 2 == 0) {
      const int hd = a.head_dim, gph = hd / 32;
#pragma unroll
      for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int p = 0; p < WN / 2; ++p) {
          int grp = egrp0 + wn * WN + 2 * p;
          int head = grp / gph;
          if (head >= a.n_q + 2 * a.n_kv) continue;
          int wr = group_wrow<EPI>(a, grp);
          int j = wr - head * hd + l32;       // dimension in the first half, < hd/2
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            int gm = rbase + i * 32 + 8 * (r >> 2) + (r & 3);
            if (gm < eMlim) qkv_emit(a, gm, head, j, acc[i][2 * p][r], acc[i][2 * p + 1][r]);
          }
        }
    } else if constexpr (EPI == EPI_ARGMAX || EPI == EPI_SAMPLE) {
      // One key per row and wave column range (WN * 32 columns), stored and
      // merged by a later pass.  Each lane first takes the maximum over its WN
      // columns; the 32 column keys of each of 16 rows then go through LDS (the last
      // W stage) and four lanes per row take their maximum, which avoids
      // a chain of dependent cross-lane shuffles per row.
      static_assert((size_t)NWV * 16 * 32 * 8 <= WSTAGE, "key transpose fits one W stage");
      unsigned long long *kl = (unsigned long long *)(lds + (NA * ASTAGE + PW * WSTAGE) / 2) + (size_t)wave * 16 * 32;
      // key of (row, column lane), rows XORed apart over the banks
      auto at = [](int row, int c) { return row * 32 + (c ^ row); };
      const int mrow = lane & 15, mq = lane >> 4;    // this lane's row and quarter in the merges
      const int slot = ent * GN + wn;
      const int col0 = (egrp0 + wn * WN) * 32 + l32;   // this lane's column in group j: col0 + 32 j
      if (a.logits) {
#pragma unroll
        for (int i = 0; i < WM; ++i)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int gm = rbase + i * 32 + 8 * (r >> 2) + (r & 3);
            if (gm < eMlim)
#pragma unroll
              for (int j = 0; j < WN; ++j)
                if (col0 + 32 * j < a.N) a.logits[(size_t)gm * a.ld_logits + col0 + 32 * j] = acc[i][j][r];
          }
      }
      // the row blocks go through a compile-time index: a plain loop over them
      // is too large to unroll once sampling is fused in, and a run-time index
      // into acc would move the accumulators to scratch memory
      auto row_block = [&](auto ic) {
        constexpr int i = decltype(ic)::value;
        // A block without live rows draws nothing (uniform): noise is most of this epilogue.
        // Sampling 4096 x 128256 at 16 rows 252 -> 225 us, 4096 x 16000 57.9 -> 49.9.
        if (EPI == EPI_SAMPLE && em0 + wm * WM * 32 + i * 32 >= eMlim) return;
        // branch-free per-lane maximum over the WN columns (increasing with j):
        // a strictly larger order key replaces, so the lowest column wins ties
#pragma unroll
        for (int half = 0; half < 2; ++half) {
#pragma unroll
        for (int r = 8 * half; r < 8 * half + 8; ++r) {
          float noise[WN];
          if constexpr (EPI == EPI_SAMPLE) {
            // one Philox call per row and lane covers this lane's WN columns:
            // counter (32 (c >> 7) + (c & 31), pos, req, 0), word (c >> 5) & 3
            const int gm = min(rbase + i * 32 + 8 * (r >> 2) + (r & 3), a.M_max - 1);
            const uint4 w = philox4x32_10(make_uint4((uint32_t)(32 * (col0 >> 7) + l32), (uint32_t)a.row_pos[gm],
                                                     (uint32_t)a.row_req[gm], 0u), a.seed_lo, a.seed_hi);
            const int w0 = (col0 >> 5) & 3;
#pragma unroll
            for (int j = 0; j < WN; ++j) {
              const int k = (w0 + j) & 3;     // selects, not an indexed array (which would live in scratch)
              const uint32_t wk = k == 0 ? w.x : k == 1 ? w.y : k == 2 ? w.z : w.w;
              noise[j] = gumbel_of(wk);
            }
          }
          uint32_t bo = 0u, bc = 0xffffffffu;
#pragma unroll
          for (int j = 0; j < WN; ++j) {
            const uint32_t c = (uint32_t)(col0 + 32 * j);
            float v = acc[i][j][r];
            if constexpr (EPI == EPI_SAMPLE) v = v * a.inv_temp + noise[j];
            const uint32_t o = c < (uint32_t)a.N ? order_key(v) : 0u;
            const bool up = o > bo;
            bo = up ? o : bo;
            bc = up ? c : bc;
          }
          const int q = 8 * ((r >> 2) & 1) + 4 * kh + (r & 3);   // row within these 16
          kl[at(q, l32)] = ((unsigned long long)bo << 32) | (0xffffffffu - bc);
        }
        __builtin_amdgcn_wave_barrier();
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        {
          unsigned long long best = 0ull;
#pragma unroll
          for (int c = 0; c < 8; ++c) {
            const unsigned long long v = kl[at(mrow, 8 * mq + c)];
            best = v > best ? v : best;
          }
#pragma unroll
          for (int off = 16; off < 64; off <<= 1) {
            const unsigned long long v = __shfl_xor(best, off, 64);
            best = v > best ? v : best;
          }
          const int gm = em0 + wm * WM * 32 + i * 32 + 16 * half + mrow;
          if (lane < 16 && gm < eMlim) a.amax_keys[(size_t)gm * a.amax_slots + slot] = best;
        }
        __builtin_amdgcn_wave_barrier();
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        }
        if constexpr (EPI == EPI_SAMPLE) {
          // the row's log-partition partials over the same column range: each
          // lane's (max, rescaled sum) over its WN columns, merged per row
          // through the same LDS transpose
          if (a.lse_part) {
            float2 *kf = (float2 *)kl;
#pragma unroll
            for (int half = 0; half < 2; ++half) {
#pragma unroll
              for (int r = 8 * half; r < 8 * half + 8; ++r) {
                float x[WN];
                float m = -__builtin_inff();
#pragma unroll
                for (int j = 0; j < WN; ++j) {
                  x[j] = col0 + 32 * j < a.N ? acc[i][j][r] * a.inv_temp : -__builtin_inff();
                  m = fmaxf(m, x[j]);
                }
                float sum = 0.0f;
#pragma unroll
                for (int j = 0; j < WN; ++j) sum += __expf(x[j] - m);
                if (m == -__builtin_inff()) sum = 0.0f;
                kf[at(8 * ((r >> 2) & 1) + 4 * kh + (r & 3), l32)] = make_float2(m, sum);
              }
              __builtin_amdgcn_wave_barrier();
              asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
              float2 v[8];
              float m = -__builtin_inff();
#pragma unroll
              for (int c = 0; c < 8; ++c) {
                v[c] = kf[at(mrow, 8 * mq + c)];
                m = fmaxf(m, v[c].x);
              }
              m = fmaxf(m, __shfl_xor(m, 16, 64));
              m = fmaxf(m, __shfl_xor(m, 32, 64));
              float sum = 0.0f;
              if (m != -__builtin_inff()) {
#pragma unroll
                for (int c = 0; c < 8; ++c) sum += v[c].y * __expf(v[c].x - m);
              }
              sum += __shfl_xor(sum, 16, 64);
              sum += __shfl_xor(sum, 32, 64);
              const int gm = em0 + wm * WM * 32 + i * 32 + 16 * half + mrow;
              if (lane < 16 && gm < eMlim) a.lse_part[(size_t)gm * a.amax_slots + slot] = make_float2(m, sum);
              __builtin_amdgcn_wave_barrier();
              asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            }
          }
        }
      };
      static_assert(WM >= 1 && WM <= 4, "row blocks per wave");
      row_block(std::integral_constant<int, 0>{});
      if constexpr (WM > 1) row_block(std::integral_constant<int, 1>{});
      if constexpr (WM > 2) row_block(std::integral_constant<int, 2>{});
      if constexpr (WM > 3) row_block(std::integral_constant<int, 3>{});
    }
  }
}

template <int EPI, class T, int WPOL>
__global__ void __launch_bounds__(T::THREADS) TWO_WAVES
k_gemm(GemmArgs a) {
  gemm_tasks<EPI, T, WPOL>(a);
}

// Argmax LM head, its tile following the live row count M (read on the device):
// 128 x 256 tiles with four W slices when the last 256-row tile would be at most half
// full, else 256 x 256.  Every element is the same sequence of MFMA k-steps in both
// shapes, so the choice never changes a result bit.
template <int EPI, int WPOL>
__global__ void __launch_bounds__(Big::THREADS) TWO_WAVES
k_gemm_dual(GemmArgs a) {
  static_assert(MidDeep::THREADS == Big::THREADS && MidDeep::LDS <= Big::LDS, "one launch shape for both tiles");
  if (lm_head_mid_tile(min(*a.m_count, a.M_max))) gemm_tasks<EPI, MidDeep, WPOL>(a);
  else gemm_tasks<EPI, Big, WPOL>(a);
}

// LM head in 128 x 128 tiles.  Weights worth streaming (`stream_tasks` not zero) are streamed
// up to that many tasks, one per CU; with more, a second row tile reads the same slices
// later and the default policy keeps them for it.  Ten weight matrices in turn, us,
// streamed and default: argmax 4096 x 16000 (125 column tiles) 256 rows 54.1 and 56.0, 384
// rows 84.3 and 74.1, 1024 rows 164.9 and 143.7; sampling 4096 x 8192 (64) 512 rows 61.1
// and 62.5, 768 rows 92.1 and 84.5.
// Of the two waves a SIMD that LDS allows the compiler is asked for one only: it then
// keeps the accumulators in AGPRs (sampling 3072 x 12000 at 1024 rows 112.9 -> 107.4 us)
// and stays within 256 registers all the same.
template <int EPI>
__global__ void __launch_bounds__(Small::THREADS) __attribute__((amdgpu_waves_per_eu(1, 2)))
k_gemm_head(GemmArgs a, unsigned stream_tasks) {
  const unsigned M = min(*a.m_count, a.M_max);
  if ((M + Small::TM - 1) / Small::TM * n_col_tiles<EPI>(a, Small::TN) <= stream_tasks) gemm_tasks<EPI, Small, CPOL_NT>(a);
  else gemm_tasks<EPI, Small, 0>(a);
}

// Grouped (MoE expert) GEMM.  An expert's weights are read by its row tiles alone.  With
// one row tile they are read once and streamed past the caches (non-temporal loads); with
// more, the row tiles that run at the same time share each slice in L2, which the default
// policy keeps.  The line lies where a third of the experts has a second row tile (E
// experts, live tiles counted on the device).  Gate-up and down, us, streamed and default:
// 128 experts of 2048 x 768, top-8: 768 rows 143 + 87 and 168 + 90, 1792 rows (112 an
// expert) 183 + 109 and 200 + 109, 2048 rows 255 + 148 and 215 + 120; 8 experts of
// 4096 x 14336, top-2: 400 rows 357 + 168 and 380 + 208, 480 rows 454 + 299 and 449 + 302,
// 1024 rows 873 + 473 and 669 + 436.
template <int EPI, class T>
__global__ void __launch_bounds__(T::THREADS) TWO_WAVES
k_gemm_grouped(GemmArgs a) {
  if (3 * *a.n_tiles <= 4 * a.n_groups) gemm_tasks<EPI, T, CPOL_NT, true>(a);
  else gemm_tasks<EPI, T, 0, true>(a);
}

// out[m][n] (+)= sum over splits of part[s][m][n], in split order (rows m < K*).
__global__ void __launch_bounds__(256)
k_splitk_reduce(const float *__restrict__ part, int splits, int M_max, int N,
                const int32_t *__restrict__ m_count, float *__restrict__ out, int ldo, int accumulate) {
  const int m = blockIdx.y;
  if (m >= *m_count) return;
  const int n = (blockIdx.x * 256 + threadIdx.x) * 4;
  if (n >= N) return;
  float4 *o = (float4 *)(out + (size_t)m * ldo + n);
  const float4 x = accumulate ? *o : make_float4(0.f, 0.f, 0.f, 0.f);
  float4 acc = sum_splits<float4>(splits, [&](int s) {
    return *(const float4 *)(part + ((size_t)s * M_max + m) * N + n);
  });
  if (accumulate) {
    acc.x += x.x; acc.y += x.y; acc.z += x.z; acc.w += x.w;
  }
  *o = acc;
}

// QKV split-K epilogue: one thread per (row, head, four consecutive RoPE pairs);
// the partials of dimensions j..j+3 and j+hd/2..j+hd/2+3 added in split order,
// then the QKV epilogue on each pair (the element-wise operations of qkv_emit),
// stored four bf16 at a time.
__global__ void __launch_bounds__(256)
k_qkv_reduce(GemmArgs a) {
  const int m = blockIdx.y;
  if (m >= *a.m_count) return;
  const int hd = a.head_dim, half = hd >> 1, nh = a.n_q + 2 * a.n_kv;
  const int idx = blockIdx.x * 256 + threadIdx.x;
  if (idx >= nh * (half / 4)) return;
  const int head = idx / (half / 4), j = 4 * (idx - head * (half / 4));
  const size_t c1 = (size_t)head * hd + j, c2 = c1 + half;
  const f4x2 x = sum_splits<f4x2>(a.splits, [&](int s) {
    const float *q = a.split_part + ((size_t)s * a.M_max + m) * a.N;
    return f4x2{*(const float4 *)(q + c1), *(const float4 *)(q + c2)};
  });
  float o1[4] = {x.a.x, x.a.y, x.a.z, x.a.w}, o2[4] = {x.b.x, x.b.y, x.b.z, x.b.w};
  if (head < a.n_q + a.n_kv) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float2 r = rope_pair(o1[e], o2[e], a.rope_cs[(size_t)m * half + j + e]);
      o1[e] = r.x;
      o2[e] = r.y;
    }
  }
  uint16_t *dst;
  if (head < a.n_q) {
    dst = a.out_bf16 + (size_t)m * a.ldo + head * hd;
  } else {
    const int req = a.packed_req[m];
    if ((unsigned)req >= (unsigned)a.n_req) return;   // not a row of this batch
    const int slot = a.packed_pos[m];
    const int cap = a.kv_cap[req];
    if (slot < 0 || slot >= cap) return;
    const int g = (head < a.n_q + a.n_kv) ? head - a.n_q : head - a.n_q - a.n_kv;
    dst = (head < a.n_q + a.n_kv ? a.kv_k : a.kv_v) + a.kv_base[req] + ((size_t)g * cap + slot) * hd;
  }
  if (((uintptr_t)(dst + j) & 7) == 0) {
    *(uint2 *)(dst + j) = make_uint2(pack_bf2(o1[0], o1[1]), pack_bf2(o1[2], o1[3]));
    *(uint2 *)(dst + j + half) = make_uint2(pack_bf2(o2[0], o2[1]), pack_bf2(o2[2], o2[3]));
  } else {   // a cache slab base that is not a multiple of four elements
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      dst[j + e] = f2bf(o1[e]);
      dst[j + half + e] = f2bf(o2[e]);
    }
  }
}

// Compute units of the current device, cached per device (atomic: calls from
// several host threads may fill the cache at once, all with the same value).
int cu_count() {
  static std::atomic<int> cached[64];
  int dev = 0, c = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 256;
  if (dev >= 0 && dev < 64) {
    const int n = cached[dev].load(std::memory_order_relaxed);
    if (n > 0) return n;
  }
  if (hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || c <= 0) return 256;
  if (dev >= 0 && dev < 64) cached[dev].store(c, std::memory_order_relaxed);
  return c;
}

// Layer GEMMs (QKV, O, gate-up, down, router), split over k or not: the tile
// whose rounds of the persistent grid take least, at 0.64, 0.9 and 1.15 us per 64-k
// slice (measured) for 128 x 128, 128 x 256 and 256 x 256 tiles: 32, 48 and 64 KB out
// of L2 at 50-57 GB/s per CU.  So the large tile takes over where the rounds of the
// small ones add up.  Batch 64 at 1024 rows: down 4096 x 14336 133 -> 104 us, O
// 50 -> 41, QKV 63 -> 58, against 128 x 128 tiles in two workgroups per CU.  The deep
// rings of the 128 x 128 tile cover the HBM latency where a slice brings few bytes: at
// 16 rows QKV 17.2 -> 14.4 us and O 15.1 -> 13.5 against a two-slice lead; from 128
// rows on both leads measured the same.  Every element is the same sequence of MFMA
// k-steps in all of them.
//
// The SwiGLU GEMM takes the same choice (4096 x 28672 with room for 256 rows: 200 live
// rows 87 -> 71 us; 16 rows with room for 16 44 -> 40.6).
template <int EPI, int WPOL>
__device__ __forceinline__ void gemm_by_rows(const GemmArgs &a) {
  using Flat = std::conditional_t<EPI == EPI_SWIGLU, DeepPair, Deep>;
  static_assert(Flat::THREADS == Big::THREADS && Flat::LDS <= Big::LDS, "one launch shape for all tiles");
  static_assert(Mid::THREADS == Big::THREADS && Mid::LDS <= Big::LDS, "one launch shape for all tiles");
  const unsigned M = min(*a.m_count, a.M_max), G = gridDim.x, sp = a.splits > 1 ? a.splits : 1;
  auto cost = [&](unsigned tm, unsigned tn, unsigned w) {
    return ((M + tm - 1) / tm * (unsigned)n_col_tiles<EPI>(a, tn) * sp + G - 1) / G * w;
  };
  const unsigned flat = cost(Flat::TM, Flat::TN, 64), mid = cost(Mid::TM, Mid::TN, 90), big = cost(Big::TM, Big::TN, 115);
  if (flat <= mid && flat <= big) {
    // without split-K the RoPE epilogue needs both halves of a pair in one wave
    if (EPI == EPI_QKV_ROPE && sp == 1) gemm_tasks<EPI, DeepPair, WPOL>(a);
    else gemm_tasks<EPI, Flat, WPOL>(a);
  }
  else if (mid <= big) gemm_tasks<EPI, Mid, WPOL>(a);
  else gemm_tasks<EPI, Big, WPOL>(a);
}

template <int EPI, int WPOL>
__global__ void __launch_bounds__(Big::THREADS) TWO_WAVES
k_gemm_rows(GemmArgs a) {
  gemm_by_rows<EPI, WPOL>(a);
}

template <int EPI, class T, int WPOL, bool GROUPED = false>
int launch_tile(int kid, const GemmArgs &a, hipStream_t s) {
  const int nMT = GROUPED ? a.m_tiles : (a.M_max + T::TM - 1) / T::TM;
  const int nNT = n_col_tiles<EPI>(a, T::TN);
  if (a.splits > 1) return DCUT_EINVAL;
  if ((EPI == EPI_ARGMAX || EPI == EPI_SAMPLE) && (!a.amax_keys || a.amax_slots < nNT * T::GN))
    return DCUT_EINVAL;
  if (EPI == EPI_SAMPLE && (!a.row_req || !a.row_pos || !(a.inv_temp >= 0.0f))) return DCUT_EINVAL;
  // persistent grid: one wave of workgroups, a multiple of 8 (one share per XCD)
  const long long tasks = (long long)nMT * nNT;
  long long g = (long long)cu_count() * T::PER_CU;
  if (tasks < g) g = tasks;
  g = (g + 7) / 8 * 8;
  if (g < 8) g = 8;
  const dim3 grid((unsigned)g), block(T::THREADS);
  if constexpr (GROUPED) return launch(kid, k_gemm_grouped<EPI, T>, grid, block, T::LDS, s, a);
  else if constexpr (std::is_same_v<T, Small>)
    return launch(kid, k_gemm_head<EPI>, grid, block, T::LDS, s, a, WPOL == CPOL_NT ? (unsigned)cu_count() : 0u);
  else return launch(kid, k_gemm<EPI, T, WPOL>, grid, block, T::LDS, s, a);
}

// k_gemm_rows and, with split-K, the pass that adds the partials (unless the
// caller does).  One workgroup per CU, fewer when the 128 x 128 tasks are fewer.
template <int EPI, int WPOL>
int launch_rows(int kid, const GemmArgs &a, hipStream_t s) {
  const int splits = a.splits > 1 ? a.splits : 1;
  if (splits > 1 && (!a.split_part || a.N % 4 || (EPI != EPI_QKV_ROPE && a.ldo % 4))) return DCUT_EINVAL;
  const long long tasks = (long long)((a.M_max + Deep::TM - 1) / Deep::TM) * n_col_tiles<EPI>(a, Deep::TN) * splits;
  long long g = cu_count();
  if (tasks < g) g = tasks;
  g = (g + 7) / 8 * 8;
  DCUT_TRY(launch(kid, k_gemm_rows<EPI, WPOL>, dim3((unsigned)g), dim3(Big::THREADS), Big::LDS, s, a));
  if (splits == 1 || a.defer_reduce) return DCUT_OK;
  if (EPI == EPI_QKV_ROPE) {
    const int quads = (a.n_q + 2 * a.n_kv) * (a.head_dim / 8);
    return launch(DCUT_KERNEL_NONE, k_qkv_reduce, dim3((quads + 255) / 256, a.M_max), dim3(256), 0, s, a);
  }
  return launch(DCUT_KERNEL_NONE, k_splitk_reduce, dim3((a.N + 1023) / 1024, a.M_max), dim3(256), 0, s,
                (const float *)a.split_part, splits, a.M_max, a.N, a.m_count, a.out_f32, a.ldo,
                EPI == EPI_RESID_F32 ? 1 : 0);
}

// The layer GEMMs choose their tile on the device (k_gemm_rows).  The LM heads: Big
// tiles with at least one Big tile per CU at M_max rows (the argmax one picks Big or a
// 128-row tile on the device from the live rows), Small tiles below that.
template <int EPI, int WPOL>
int launch_policy(int kid, const GemmArgs &a, hipStream_t s) {
  if constexpr (EPI == EPI_RESID_F32 || EPI == EPI_STORE_F32 || EPI == EPI_QKV_ROPE || EPI == EPI_SWIGLU) {
    return launch_rows<EPI, WPOL>(kid, a, s);
  } else {
    const long long big_tasks = (long long)((a.M_max + Big::TM - 1) / Big::TM) * ((a.N + Big::TN - 1) / Big::TN);
    if (big_tasks < cu_count()) return launch_tile<EPI, Small, WPOL>(kid, a, s);
    if constexpr (EPI == EPI_ARGMAX) {
      // tile shape chosen on the device from the live row count (one workgroup per CU);
      // the sampling epilogue keeps the 256-row tile (both paths in one kernel would spill)
      if (!a.amax_keys || a.amax_slots < (a.N + MidDeep::TN - 1) / MidDeep::TN * MidDeep::GN)
        return DCUT_EINVAL;
      const int g = (cu_count() + 7) / 8 * 8;
      return launch(kid, k_gemm_dual<EPI, WPOL>, dim3((unsigned)g), dim3(Big::THREADS), Big::LDS, s, a);
    } else {
      return launch_tile<EPI, BigFlat, WPOL>(kid, a, s);
    }
  }
}

// Cache policy of the weight loads.  A matrix of 64 MB or more is streamed
// (non-temporal), so that it does not take the activations, partials and caches of the
// layer out of the 256 MB memory-side cache.  Measured over ten layers with weights of
// their own (no weight survives to its next use), us a layer, nothing streamed / this
// rule / everything streamed: 4096 x 14336 layer at 16 rows 127.8 / 121.8 / 117.6, 128 rows
// 166.6 / 158.3 / 159.7, 256 rows 211.3 / 208.6 / 207.3, 1024 rows 505.6 / 505.6 / 502.1,
// 4096 rows 1866 / 1866 / 1863, 8192 rows 3885 / 3997 / 4009; 3072 x 8200 layer, whose down
// matrix of 50 MB loses by it, at 128 rows 131.3 / 130.9 / 131.3, 512 rows 225.9 / 225.5 /
// 234.5, 4096 rows 1147 / 1157 / 1191; attention matrices of the 2048-wide MoE layer
// (20 MB) at 64 rows 287.5 / 287.6 / 284.5, 768 rows 392.1 / 391.6 / 395.9.  So below 64 MB
// streaming gains 3 % at the fewest rows and loses up to 4 % above; from 64 MB on it gains
// 5 % up to 128 rows and costs 3 % at 8192.  LM head 4096 x 128256 at 64 rows 201 -> 187.
// Expert weights have a rule of their own (k_gemm_grouped).
template <int EPI>
int launch_epi(int kid, const GemmArgs &a, hipStream_t s) {
  const long long w_rows = EPI == EPI_SWIGLU ? 2LL * a.swiglu_inter : a.N;
  if (a.tiles) {
    if constexpr (EPI == EPI_SWIGLU || EPI == EPI_STORE_F32) return launch_tile<EPI, Small, 0, true>(kid, a, s);
    else return DCUT_EINVAL;
  }
  if (w_rows * a.ldw * 2 >= (64LL << 20)) return launch_policy<EPI, CPOL_NT>(kid, a, s);
  return launch_policy<EPI, 0>(kid, a, s);
}

}  // namespace

int gemm_splits(int M_max, int N, int K) {
  // Split-K tasks are 128 x 128 tiles over a k range (256 x 256 at many live rows), and a
  // split-K GEMM at few live rows runs at the per-CU load rate: its time is that of the busiest
  // CU.  The factor minimises a model of that time summed over a quarter, a half, three quarters
  // and all of M_ref = min(M_max, 1024) live rows (a large batch verifies far fewer than its
  // B(D+1) rows at the budgets a cost row picks): the busiest CU's task count (tasks over CUs,
  // rounded up) times a task's operand bytes, its float32 partial tile and a fixed cost per task
  // (prologue and drain) worth about 150 KB of operand loads.  At least 16 k-slices per split;
  // ties go to fewer splits.  The shapes and the CU count decide it, never the live rows.
  const long long M_ref = M_max < 1024 ? M_max : 1024;
  const long long nNT = (N + Small::TN - 1) / Small::TN, nk = (K + TK - 1) / TK;
  long long cap = nk / 16;
  if (cap > 16) cap = 16;
  if (cap < 1) cap = 1;
  const long long cus = cu_count();
  int best = 1;
  double best_cost = 0.0;
  for (int sp = 1; sp <= cap; ++sp) {
    const long long per = (nk + sp - 1) / sp;
    const double bytes = (double)(Small::TM + Small::TN) * per * TK * 2 +
                         (sp > 1 ? (double)Small::TM * Small::TN * 4 : 0.0) + 150e3;
    double cost = 0.0;
    for (int q = 1; q <= 4; ++q) {
      const long long M = M_ref * q / 4 > 0 ? M_ref * q / 4 : 1;
      const long long tasks = (M + Small::TM - 1) / Small::TM * nNT * sp;
      cost += (double)((tasks + cus - 1) / cus) * bytes;
    }
    if (sp == 1 || cost < best_cost) {
      best = sp;
      best_cost = cost;
    }
  }
  return best;
}

void gemm_argmax_slots(const GemmArgs &a, EpiKind epi, int *big, int *mid) {
  const bool big_tiles = !a.tiles && a.splits <= 1 &&
                         (long long)((a.M_max + Big::TM - 1) / Big::TM) * ((a.N + Big::TN - 1) / Big::TN) >= cu_count();
  if (big_tiles) {
    *big = (a.N + Big::TN - 1) / Big::TN * Big::GN;
    *mid = epi == EPI_ARGMAX ? (a.N + MidDeep::TN - 1) / MidDeep::TN * MidDeep::GN : *big;
  } else {
    *big = *mid = (a.N + Small::TN - 1) / Small::TN * Small::GN;
  }
}

int gemm_launch(int kid, EpiKind epi, const GemmArgs &a, hipStream_t s) {
  switch (epi) {
    case EPI_RESID_F32: return launch_epi<EPI_RESID_F32>(kid, a, s);
    case EPI_SWIGLU: return launch_epi<EPI_SWIGLU>(kid, a, s);
    case EPI_QKV_ROPE: return launch_epi<EPI_QKV_ROPE>(kid, a, s);
    case EPI_ARGMAX: return launch_epi<EPI_ARGMAX>(kid, a, s);
    case EPI_SAMPLE: return launch_epi<EPI_SAMPLE>(kid, a, s);
    case EPI_STORE_F32: return launch_epi<EPI_STORE_F32>(kid, a, s);
  }
  return DCUT_EINVAL;
}

}  // namespace dcut
