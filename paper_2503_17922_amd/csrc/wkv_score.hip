// Observation-window token scores (WindowKV Eq. 1-2) for one or more layer groups.
//
//   t[b,h,j] = sum_{g<G} sum_{i<w_obs} softmax_j( q_{g,i} . k_j * scale )      j < L - w_obs
//
// The G*w_obs query rows that share a KV head are stacked into one M-row operand, so the
// logits of a KV head are one [M x d] x [d x L] contraction.  The softmax normaliser of a row
// needs every key of the prefix before any column sum can be finished, hence two passes over
// the keys of the scored layer:
//
//   pass 1 (stats)  per (row, key chunk): running maximum m and sum z = sum 2^(v - m) of the
//                   base-2 logits v = (q.k) * scale * log2(e), with the causal mask of the
//                   observation block applied.  Partials go to the workspace.
//   fold            the partials of every row become lse2_i = m_i + log2(z_i) (in pass 2's prologue; a launch
//                   of its own when a row has very many chunks).
//   pass 2 (score)  each workgroup recomputes its logits and writes t_j = sum_i 2^(v_ij - lse2_i).
//
// A caller whose prefill attention kept the normalisers of the observation rows hands them
// over; pass 1 and the fold are then skipped and the keys are read once.
//
// Both passes run on the matrix pipe: v_mfma_f32_16x16x32_bf16 / _f16 for 16-bit inputs, v_mfma_f32_16x16x4_f32
// for fp32 inputs.  Every wave holds the query fragments of its row tiles in registers for the whole launch and
// reads 16-key tiles from a ring in LDS that it fills itself, by DMA from global memory several tiles
// ahead: the waves of a workgroup do not synchronise in the loop, and nothing but the keys crosses LDS.
#include "wkv_device.h"
#include "wkv_pool.h"

namespace wkv {

// =========================================================================================
// fold: per-chunk (m, z) partials of pass 1 -> one lse2 per row, once per (group, sequence, KV head)
// =========================================================================================
// Partials lie [chunk][row]: the threads of a workgroup take consecutive rows and every so many chunks, so the
// reads are coalesced and, sixteen at a time, independent of each other.
__device__ __forceinline__ void fold_rows(const float2 *__restrict__ part, int n_chunks, int m_pad, int r, int first, int step,
                                          float &m, float &z) {
  m = -INFINITY;
  z = 0.0f;
  constexpr int N = 16;                                 // (64 partials by two threads: two round trips)
  for (int c = first; c < n_chunks; c += N * step) {
    float2 p[N];
#pragma unroll
    for (int i = 0; i < N; ++i) p[i] = part[(int64_t)min(c + i * step, n_chunks - 1) * m_pad + r];
    float mn = m;
#pragma unroll
    for (int i = 0; i < N; ++i) mn = c + i * step < n_chunks ? fmaxf(mn, p[i].x) : mn;
    if (mn == -INFINITY) continue;
    z *= fast_exp2(m - mn);
#pragma unroll
    for (int i = 0; i < N; ++i) z += c + i * step < n_chunks ? p[i].y * fast_exp2(p[i].x - mn) : 0.0f;
    m = mn;
  }
}

// lse2 of the rows of one (group, sequence, KV head) into lse[0 .. rows-1] by NT threads; padded rows get +inf
// (2^-inf = 0: they contribute nothing).  part_s: NT entries of scratch.  Synchronises before it returns.
template <int NT>
__device__ __forceinline__ void fold_all(const Shape &s, int n_chunks, int m_pad, const float2 *__restrict__ part, int rows,
                                         float2 *part_s, float *lse) {
  const int tpr = max(NT / rows, 1);                    // threads per row
  for (int r0 = 0; r0 < rows; r0 += NT / tpr) {
    const int r = r0 + threadIdx.x % (NT / tpr), which = threadIdx.x / (NT / tpr);
    float m = -INFINITY, z = 0.0f;
    if (r < s.M) fold_rows(part, n_chunks, m_pad, r, which, tpr, m, z);
    part_s[threadIdx.x] = make_float2(m, z);
    __syncthreads();
    if (which == 0 && r < rows) {
      for (int i = 1; i < tpr; ++i) {
        const float2 p = part_s[threadIdx.x + i * (NT / tpr)];
        merge_stats(m, z, p.x, p.y);
      }
      lse[r] = r < s.M ? m + fast_log2(z) : INFINITY;
    }
    __syncthreads();
  }
}

constexpr int FOLD_THREADS = 256;

__global__ __launch_bounds__(FOLD_THREADS) void fold_kernel(Shape s, ScorePlan pl, const float2 *__restrict__ partials,
                                                            float *__restrict__ lse, const uint32_t *__restrict__ only_if) {
  __shared__ float2 part_s[FOLD_THREADS];
  if (only_if && *only_if == 0u) return;
  const int64_t row = (int64_t)blockIdx.y * s.B * s.Hkv + blockIdx.x;
  const int b = blockIdx.x / s.Hkv;
  fold_all<FOLD_THREADS>(s, pl.pass[0].first[b + 1] - pl.pass[0].first[b], pl.m_pad, partials + row * pl.n_chunks1 * pl.m_pad, pl.m_pad, part_s,
                         lse + row * pl.m_pad);
}

// The base-2 log-sum-exp of softmax row r of (group g, sequence b, KV head h): converted from the
// caller's natural-log normalisers [B, Hq, w_obs] when they were handed over (the rows of a KV
// head are contiguous there), else what the fold left in the workspace.  Padded rows get +inf.
__device__ __forceinline__ float row_lse2(const Shape &s, const ScorePlan &pl, const GroupPtrs &gp,
                                          const float *__restrict__ lse_ws, int g, int b, int h, int64_t row, int r) {
  if (r >= s.M) return INFINITY;
  const float *given = gp.lse[g];
  if (given) return given[((int64_t)b * s.Hq + (int64_t)h * s.G) * s.w_obs + r] * 1.4426950408889634f;
  return lse_ws[row * pl.m_pad + r];
}

// =========================================================================================
// the two passes
// =========================================================================================
// A 16x16 tile of logits takes 16 rows of each operand, 64 bytes of a row per step: lane l holds row l%16, the
// 16-byte piece l/16.  Both operands have this layout, so which of them is A is a free choice per pass:
//   PASS 1 (stats)   keys as A: a lane gets 4 consecutive keys of ONE query row per row tile, so the row
//                    statistics are in-lane accumulations (RT of them), merged once per chunk.
//   PASS 2 (scores)  queries as A: a lane gets 4 query rows of ONE key, so a key's column sum is in-lane adds
//                    over all row tiles plus two permlane swaps.
//
// Waves.  HV waves share a key tile slot and take RT row tiles each (128 rows a wave at most, 64 for fp32 with 128
// channels: the queries take RT * D * esize / 16 registers); the KW slots of a workgroup take the chunk's key
// tiles in turn.  Two waves fit a SIMD.
//
// The ring.  A slot has NS places of 16 key rows each.  A DMA instruction (global_load_lds_dwordx4) writes 64 pieces
// of 16 bytes in lane order; which piece of its row a lane fetches is permuted (swizzle) so that the 16 lanes
// that later read the same piece of 16 rows find them in different banks.  Global reads stay whole rows.
// Tile i is in registers (the next one being read from LDS) while tiles i+2 .. i+NS are on their way; the loads are
// counted by hand (s_waitcnt vmcnt), which holds because the loop has no other global access.  With one row group
// a wave fills its own slot and the waves never synchronise in the loop.  With several, the waves of a slot fetch a part
// of each tile and the workgroup meets at a barrier per tile, or (OWN_RINGS, two groups of 16-bit inputs) every wave
// fetches whole tiles for itself: half the bytes in flight, no barriers, and the second of a slot's waves finds the
// tile in the L2, as long as the two do not drift too far apart (see plan_score).
//
// What bounds it.  Per 64 logits a SIMD issues one 16x16x32 MFMA (8.6 ns on random data at the clocks the chip then
// holds) and one multiply-add, exponential and add (7.8 ns); they hardly overlap: 13 ns together in a loop of
// nothing else, in whatever order they are written.  The 32K-token model (8 groups, 128 rows): 103 + 100 us for the two
// passes (shortest launches 92 + 90), 70-76 us without the loads; with plain loads 108 + 107 us, of which the loads alone 91-95
// (5.9 TB/s; a reading kernel reaches 7.0 by nontemporal loads, 6.1 without).  The kernels before this
// one kept the queries in LDS, read the keys in operand layout straight from global memory and took 111 + 107 us there;
// 12.0 + 11.6 us for a group of 4096 tokens (now 9.0 + 10.1, fold included: half the code to fetch, one round of loads in the
// prologue), 15.9 + 9.3 (fold) + 14.7 us for 16384 tokens (13.8 + 15.7), 28.3 + 27.7 us for 4096 tokens in fp32 (19.5 + 20.2),
// 54 + 50 us for 48 rows of ragged sequences with 224 softmax rows (31 + 31).
// With two row groups a pass takes the sum of the two, not the longer: 16381 tokens, 8 groups, 256 rows 53 us of arithmetic by these
// figures and 38 us of keys at 7.0 TB/s, measured 97-99; the ragged sequences 12 us of arithmetic, measured 31.  One workgroup a
// compute unit, two waves a SIMD, and with shared rings a barrier per tile: while these wait there is nothing else to run.
constexpr int score_slots(int row_groups) { return row_groups == 4 ? 2 : 4; }         // key tile slots of a workgroup
constexpr int score_threads(int row_groups) { return 64 * row_groups * score_slots(row_groups); }

template <int D, int DT, int RT, int HV, bool OWN_RINGS>
struct ScoreConfig {
  static constexpr int ES = DT == DT_F32 ? 4 : 2;       // bytes per element
  static constexpr int ROWB = D * ES;                   // bytes per key row
  static constexpr int KS = ROWB / 64;                  // steps of a contraction
  static constexpr int TILE = 16 * ROWB;
  static constexpr int PPR = ROWB / 16;                 // 16-byte pieces per row: 8, 16 or 32
  static constexpr int RPI = 64 / PPR;                  // rows per DMA instruction
  static constexpr bool SHARED = HV > 1 && !OWN_RINGS;
  static constexpr int PARTS = SHARED ? HV : 1;         // waves that fetch a tile together
  static constexpr int LPT = TILE / 1024 / PARTS;       // DMA instructions per tile and wave
  static constexpr int KW = score_slots(HV), NT = score_threads(HV), WAVES = NT / 64;
  static constexpr int RINGS = SHARED ? KW : WAVES;
  static constexpr int FIT = (HV == 1 ? 65536 : 131072) / (RINGS * TILE);
  static constexpr int NS = FIT < 8 * PARTS ? FIT : 8 * PARTS;
  static constexpr int RING = RINGS * NS * TILE;
  // the queries pass through the part of the ring that is filled last
  static constexpr int QBYTES = HV * RT * 16 * ROWB;
  static constexpr int FIRST = NS - (QBYTES + RINGS * TILE - 1) / (RINGS * TILE);
  static_assert(FIRST >= 0, "the queries fit the ring");
  static_assert(NS >= 2, "a tile being read and one under way");
  // Read the next tile's fragments while this one is computed.  fp32: a tile takes thousands of cycles on the matrix
  // pipe, and its fragments twice the registers.
  static constexpr bool AHEAD = DT != DT_F32;
  static constexpr int SEG = HV == 4 ? SCORE_SEG / 2 : SCORE_SEG;
  // where piece p of row r lies within its row's slot
  static __device__ __forceinline__ int swizzle(int r, int p) { return p ^ (PPR == 8 ? (r >> 1) & 7 : r & 15); }
};

__device__ __forceinline__ uint32_t lds_address(const void *p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char *)p;
}
// At most N loads outstanding, every LDS read returned.
template <int N>
__device__ __forceinline__ void wait_vmcnt() { asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory"); }

// A DMA instruction of the ring: 64 lanes fetch 16 bytes each, to lds, lds + 16, ... in lane order.  From base + off bytes, or from
// an address per lane.  m0 holds the LDS address; naming it as overwritten keeps the compiler's own uses of it, should there be any,
// clear of this one (it is a reserved register, which clang warns of: nothing relies on its being preserved).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <bool NT_LOADS>
__device__ __forceinline__ void dma_to_lds(uint32_t lds, const char *base, uint32_t off) {
  if constexpr (NT_LOADS)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(lds), "v"(off), "s"(base) : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(off), "s"(base) : "memory", "m0");
}
__device__ __forceinline__ void dma_to_lds(uint32_t lds, const char *p) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds), "v"(p) : "memory", "m0");
}
#pragma clang diagnostic pop

// NT_LOADS: the keys are not put into the memory-side cache (see plan_score).  Kernels of their own, as a branch at every fetch
// costs small calls 1 %.
template <int D, int DT, int RT, int HV, int PASS, bool NT_LOADS, bool OWN_RINGS>
__global__ __launch_bounds__(score_threads(HV), 2) void score_kernel(Shape s, BatchParams bp, GroupPtrs gp, ScorePlan pl,
                                                                                 float2 *__restrict__ partials,
                                                                                 const float *__restrict__ lse_g,
                                                                                 float *__restrict__ t_out,
                                                                                 float *__restrict__ s_pool,
                                                                                 const uint32_t *__restrict__ only_if) {
  using C = ScoreConfig<D, DT, RT, HV, OWN_RINGS>;
  constexpr int KS = C::KS, KW = C::KW, NT = C::NT, NS = C::NS, ROWS = HV * RT * 16;
  __shared__ __attribute__((aligned(1024))) char ring[C::RING];
  __shared__ __attribute__((aligned(16))) float t_s[PASS == 2 ? HV * (C::SEG + KW * 16) : 4];     // token scores of a segment
  __shared__ __attribute__((aligned(16))) float lse_s[PASS == 2 ? ROWS : 4];
  __shared__ float2 part_s[PASS == 2 ? NT : KW * ROWS];
  // Launched behind the single-read kernel as its fall-back: nothing to do unless that kernel
  // raised the word (uniform over the grid).
  if (only_if && *only_if == 0u) return;

  // Pass 2 walks the work items in the opposite order of pass 1: the keys pass 1 read last
  // are the ones most likely still held by the memory-side cache.
  const int x = PASS == 1 ? blockIdx.x : gridDim.x - 1 - blockIdx.x;
  const int h = PASS == 1 ? blockIdx.y : gridDim.y - 1 - blockIdx.y;
  const int g = PASS == 1 ? blockIdx.z : gridDim.z - 1 - blockIdx.z;
  const PassPlan &pp = pl.pass[PASS - 1];
  int b = 0;
  while (b + 1 < s.B && x >= pp.first[b + 1]) ++b;
  const int bx = x - pp.first[b];                           // chunk of the sequence
  const int L = bp.seq[b].L;
  const int n_review = L - s.w_obs;
  const int64_t row = ((int64_t)g * s.B + b) * s.Hkv + h;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int half = wave / KW, kw = wave % KW;               // row group, key tile slot of this wave
  const int col = lane & 15, quad = lane >> 4;
  const int my_ring = C::SHARED ? kw : wave, my_part = C::SHARED ? half : 0;

  const int chunk = pp.chunk[b] * CHUNK_UNIT;
  const int limit = PASS == 1 ? L : n_review;               // keys that matter to this pass
  const int c_first = bx * chunk;
  int c0 = c_first, cend = min(c0 + chunk, limit);          // keys c0 .. cend-1 of the row
  int seg_len = PASS == 1 ? 0x40000000 : C::SEG;            // pass 2 writes its scores out a segment at a time
  int win = 1;
  if (PASS == 2 && s_pool) {
    // A window belongs to the chunk that holds its first token: the workgroup scores and pools whole
    // windows, whatever their size, and no token is scored twice.
    win = bp.seq[b].win;
    c0 = (c0 + win - 1) / win * win;
    cend = min((cend + win - 1) / win * win, limit);
    seg_len = C::SEG / win * win;
  }
  float *trow = PASS == 2 ? t_out + row * s.t_stride : nullptr;
  if (PASS == 2 && !s_pool)                                 // the row's padding
    for (int j = n_review + threadIdx.x; j < (x + 1 == pp.first[b + 1] ? s.t_stride : 0); j += NT) trow[j] = 0.0f;
  if (PASS == 2 && c0 >= cend) return;
  float2 *part = partials + row * pl.n_chunks1 * pl.m_pad;

  // ---- the key stream -------------------------------------------------------------------------
  const char *kbase = (const char *)gp.k[g] + ((int64_t)b * s.kv_sb + (int64_t)h * s.kv_sh) * C::ES;
  const int64_t kst = s.kv_st * C::ES;
  const bool wide = kst * 16 >= 0x7fffffff;                 // rows too far apart for 32-bit offsets within a tile
  uint32_t off[C::LPT];                                     // this lane's piece of each of its DMA instructions, from the tile's first row
#pragma unroll
  for (int n = 0; n < C::LPT; ++n) {
    const int r = (my_part * C::LPT + n) * C::RPI + lane / C::PPR;
    off[n] = (uint32_t)((uint32_t)r * (uint32_t)kst + C::swizzle(r, lane % C::PPR) * 16);
  }
  const uint32_t ring_lds = lds_address(ring) + my_ring * (NS * C::TILE) + my_part * (C::LPT * 1024);
  // keys j .. j+15 (this wave's part) into place `slot`; rows from cend on are not read (their lanes fetch row cend-1 again)
  auto fetch = [&](int j, int slot) __attribute__((always_inline)) {
    const uint32_t dst = ring_lds + slot * C::TILE;
    if (j + 16 <= cend && !wide) {
      const char *base = kbase + (int64_t)j * kst;
#pragma unroll
      for (int n = 0; n < C::LPT; ++n) dma_to_lds<NT_LOADS>(dst + n * 1024, base, off[n]);
    } else {
#pragma unroll
      for (int n = 0; n < C::LPT; ++n) {
        const int r = (my_part * C::LPT + n) * C::RPI + lane / C::PPR;
        const char *p = kbase + (int64_t)min(j + r, cend - 1) * kst + C::swizzle(r, lane % C::PPR) * 16;
        dma_to_lds(dst + n * 1024, p);
      }
    }
  };
  // The order of this wave's tiles: KW apart within a segment, segment by segment.
  int jf = c0 + kw * 16, jf_end = min(c0 + seg_len, cend), slot_f = 0;      // the next tile to fetch
  auto fetch_next = [&]() __attribute__((always_inline)) {
    fetch(jf, slot_f);
    slot_f = slot_f == NS - 1 ? 0 : slot_f + 1;
    jf += KW * 16;
    while (PASS == 2 && (C::SHARED ? jf - kw * 16 : jf) >= jf_end && jf_end < cend) {
      jf = jf_end + kw * 16;
      jf_end = min(jf_end + seg_len, cend);
    }
  };
#pragma unroll
  for (int i = 0; i < C::FIRST; ++i) fetch_next();

  // ---- the queries: into the ring's other places as fragments (lane l: row l%16 of a row tile, piece l/16 of a step),
  // from there into registers.  Rows past the last one repeat it: their statistics are never used and their
  // normaliser is +inf.
  constexpr int FRAGS = HV * RT * KS, PER_SLOT = (NS - C::FIRST) * C::TILE / 1024;
  auto frag_at = [&](int f) __attribute__((always_inline)) {
    return f / PER_SLOT * (NS * C::TILE) + C::FIRST * C::TILE + f % PER_SLOT * 1024;
  };
  for (int f = wave; f < FRAGS; f += C::WAVES) {
    const int r = min(f / KS * 16 + col, s.M - 1);
    const int hq = (int)((uint32_t)r * s.w_magic >> 16), io = r - hq * s.w_obs;      // r / w_obs, r % w_obs
    const char *qp = (const char *)gp.q[g] +
                     ((int64_t)b * s.q_sb + (int64_t)(h * s.G + hq) * s.q_sh + (int64_t)io * s.q_st) * C::ES + f % KS * 64 + quad * 16;
    dma_to_lds(lds_address(ring) + frag_at(f), qp);
  }
  if (PASS == 2) {
    if (pl.fold_in_pass2) fold_all<NT>(s, pl.pass[0].first[b + 1] - pl.pass[0].first[b], pl.m_pad, part, ROWS, part_s, lse_s);
    else
      for (int r = threadIdx.x; r < ROWS; r += NT) lse_s[r] = row_lse2(s, pl, gp, lse_g, g, b, h, row, r);
  }
  wait_vmcnt<0>();
  __syncthreads();
  bf16x8 qf[RT][KS];
#pragma unroll
  for (int mt = 0; mt < RT; ++mt)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[mt][ks] = *(const bf16x8 *)(ring + frag_at((half * RT + mt) * KS + ks) + lane * 16);
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __syncthreads();
#pragma unroll
  for (int i = C::FIRST; i < NS; ++i) fetch_next();
  const float sc = s.c1;
  float mref[PASS == 1 ? RT : 1], zsum[PASS == 1 ? RT : 1];  // pass 1: reference and sum of query row (half*RT + mt)*16 + col
  bool settled = false;                                     // (uniform) every sum of this wave is large enough for its reference
  if (PASS == 1) {
#pragma unroll
    for (int mt = 0; mt < RT; ++mt) { mref[mt] = 0.0f; zsum[mt] = 0.0f; }
  }

  // ---- tiles -----------------------------------------------------------------------------------
  // Meeting of the workgroup without the wait for outstanding loads that __syncthreads() brings.
  auto barrier = [&]() __attribute__((always_inline)) { asm volatile("s_barrier" ::: "memory"); };
  struct Frags { bf16x8 f[KS]; };
  const uint32_t lane_row = col * C::ROWB;
  int slot_r = 0;                                           // the slot read next
  auto read_frags = [&](Frags &kf) __attribute__((always_inline)) {
    const char *p = ring + my_ring * (NS * C::TILE) + slot_r * C::TILE + lane_row;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) kf.f[ks] = *(const bf16x8 *)(p + C::swizzle(col, ks * 4 + quad) * 16);
    slot_r = slot_r == NS - 1 ? 0 : slot_r + 1;
  };
  auto logits = [&](const Frags &kf, int mt) __attribute__((always_inline)) {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      acc = PASS == 1 ? mfma_64b<DT>(kf.f[ks], qf[mt][ks], acc) : mfma_64b<DT>(qf[mt][ks], kf.f[ks], acc);
    return acc;
  };

  // Statistics of one tile, with care: the causal mask (key j visible to observation query io iff
  // j <= n_review + io), the end of the sequence, and rows whose reference does not suit their logits.  A
  // reference is good while the sum taken with it stays between MF_LOW (what underflowed is negligible) and
  // MF_BIG; otherwise it moves to the larger of the tile's maximum and the sum so far.
  auto careful = [&](const Frags &kf, int j0) __attribute__((always_inline)) {
#pragma unroll
    for (int mt = 0; mt < RT; ++mt) {
      f32x4 acc = logits(kf, mt);
      const int r = min((half * RT + mt) * 16 + col, s.M - 1);
      const int last = min(n_review + r - (int)((uint32_t)r * s.w_magic >> 16) * s.w_obs, cend - 1);
      float vmax = -INFINITY, a = 0.0f;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        acc[e] = j0 + quad * 4 + e <= last ? acc[e] * sc : -INFINITY;
        vmax = fmaxf(vmax, acc[e]);
        a += fast_exp2(acc[e] - mref[mt]);
      }
      const float z = zsum[mt];
      if (!(a <= MF_BIG) || !(z + a >= MF_LOW)) {
        const float have = z > 0.0f ? mref[mt] + fast_log2(z) : -INFINITY;
        const float nref = fmaxf(vmax, have);
        if (nref != -INFINITY) {                            // else the row has seen no key yet
          a = fast_exp2(have - nref);
#pragma unroll
          for (int e = 0; e < 4; ++e) a += fast_exp2(acc[e] - nref);
          mref[mt] = nref;
          zsum[mt] = a;
        }
      } else {
        zsum[mt] = z + a;
      }
    }
  };

  auto tile = [&](Frags &kf, Frags &kn, int j0, int seg0) __attribute__((always_inline)) {
    if (C::AHEAD) {                                         // tile i+1 out of the ring, tile i+NS into the slot tile i left
      wait_vmcnt<(NS - 2) * C::LPT>();
      if (C::SHARED) barrier();                             // (every part of it; every wave has tile i in registers)
      read_frags(kn);
    } else {
      wait_vmcnt<(NS - 1) * C::LPT>();
      if (C::SHARED) barrier();
      read_frags(kf);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");    // its place is free for the fetch below
      if (C::SHARED) barrier();
    }
    fetch_next();
    if (PASS == 1) {
      bool care = j0 + 16 > min(n_review, cend);            // uniform
      if (!care) {
        f32x4 acc[RT];
        float psum[RT];
#pragma unroll
        for (int mt = 0; mt <= RT; ++mt) {                  // the MFMAs of a row tile beside the exponentials of the one before
          if (mt < RT) acc[mt] = logits(kf, mt);
          if (mt > 0) {
            const int m1 = mt - 1;
            float a = fast_exp2(fmaf(acc[m1][0], sc, -mref[m1]));
#pragma unroll
            for (int e = 1; e < 4; ++e) a += fast_exp2(fmaf(acc[m1][e], sc, -mref[m1]));
            psum[m1] = a;
          }
        }
        float big = psum[0];
#pragma unroll
        for (int mt = 1; mt < RT; ++mt) big = fmaxf(big, psum[mt]);
        bool bad = !(big <= MF_BIG);
        if (!settled) {
          float low = zsum[0] + psum[0];
#pragma unroll
          for (int mt = 1; mt < RT; ++mt) low = fminf(low, zsum[mt] + psum[mt]);
          bad |= !(low >= MF_LOW);
        }
        care = __any(bad);
        if (!care) {
#pragma unroll
          for (int mt = 0; mt < RT; ++mt) zsum[mt] += psum[mt];
          settled = true;
        }
      }
      if (care) {
        careful(kf, j0);
        if (!settled) {
          float low = zsum[0];
#pragma unroll
          for (int mt = 1; mt < RT; ++mt) low = fminf(low, zsum[mt]);
          settled = __all(low >= MF_LOW);
        }
      }
    } else {
      f32x4 acc[RT];
      float ta = 0.0f, tb = 0.0f;
#pragma unroll
      for (int mt = 0; mt <= RT; ++mt) {
        if (mt < RT) acc[mt] = logits(kf, mt);
        if (mt > 0) {
          const int m1 = mt - 1;
          // (from LDS every time: 4 * RT of them would not fit beside the queries)
          const f32x4 lse = *(const f32x4 *)&lse_s[(half * RT + m1) * 16 + quad * 4];
          ta += fast_exp2(fmaf(acc[m1][0], sc, -lse[0]));
          tb += fast_exp2(fmaf(acc[m1][1], sc, -lse[1]));
          ta += fast_exp2(fmaf(acc[m1][2], sc, -lse[2]));
          tb += fast_exp2(fmaf(acc[m1][3], sc, -lse[3]));
        }
      }
      // (the four lanes of a key store the same value to the same place: no branch in the loop)
      t_s[half * (C::SEG + KW * 16) + j0 - seg0 + col] = quads_sum(ta + tb);
    }
  };

  Frags ka, kb;
  if (C::AHEAD) {
    wait_vmcnt<(NS - 1) * C::LPT>();
    if (C::SHARED) barrier();
    read_frags(ka);
  }
  for (int seg0 = c0; seg0 < cend; seg0 += seg_len) {
    const int seg_end = min(seg0 + seg_len, cend);
    // with row groups every slot takes a tile in every round, if need be one past the end (masked in pass 1, past the
    // scores that count in pass 2): the waves meet at barriers
    for (int j = seg0 + kw * 16; (C::SHARED ? j - kw * 16 : j) < seg_end; j += KW * 16) {
      tile(ka, kb, j, seg0);
      if (C::AHEAD) ka = kb;
    }
    if (PASS == 1) break;
    __syncthreads();
    if (HV > 1) {                                           // column sums of the other row groups
      for (int i = threadIdx.x; i < seg_end - seg0; i += NT) {
        float x = t_s[i];
#pragma unroll
        for (int v = 1; v < HV; ++v) x += t_s[v * (C::SEG + KW * 16) + i];
        t_s[i] = x;
      }
      __syncthreads();
    }
    if (s_pool)                                             // Eq. 3-4 while the token scores are in LDS
      pool_windows<NT>(t_s, seg0 / win, (seg_end + win - 1) / win, win, bp.seq[b].p, n_review, s_pool + row * s.nw_max);
    else
      for (int i = threadIdx.x; i < seg_end - seg0; i += NT) trow[seg0 + i] = t_s[i];
    if (seg_end == cend) break;
    __syncthreads();
  }

  if (PASS == 1) {
    // merge the 4 quads of each row, then the KW waves
#pragma unroll
    for (int mt = 0; mt < RT; ++mt) {
      float m = zsum[mt] > 0.0f ? mref[mt] : -INFINITY, z = zsum[mt];
      Pair pm = swap_halves(m, m), pz = swap_halves(z, z);
      merge_stats(pm.a, pz.a, pm.b, pz.b);
      m = pm.a; z = pz.a;
      pm = swap_rows(m, m); pz = swap_rows(z, z);
      merge_stats(pm.a, pz.a, pm.b, pz.b);
      if (quad == 0) part_s[kw * ROWS + (half * RT + mt) * 16 + col] = make_float2(pm.a, pz.a);
    }
    __syncthreads();
    for (int r = threadIdx.x; r < pl.m_pad; r += NT) {           // m_pad <= ROWS
      float m = part_s[r].x, z = part_s[r].y;
      for (int w = 1; w < KW; ++w) merge_stats(m, z, part_s[w * ROWS + r].x, part_s[w * ROWS + r].y);
      part[(int64_t)bx * pl.m_pad + r] = make_float2(m, z);
    }
  }
}

// =========================================================================================
// launch
// =========================================================================================
template <int D, int DT, int RT, int HV, bool NT_LOADS, bool OWN_RINGS = false>
static hipError_t launch_passes(const Shape &s, const BatchParams &bp, const ScorePlan &pl, const GroupPtrs &gp, int32_t n_groups,
                                bool have_lse, float2 *partials, float *lse, float *t_out, float *s_pool, hipStream_t stream,
                                hipEvent_t mid, const uint32_t *only_if) {
  const dim3 block(score_threads(HV));
  hipError_t e;
  if (have_lse) {                                      // no statistics pass: pass 2 reads the caller's normalisers
    if (mid && (e = hipEventRecord(mid, stream)) != hipSuccess) return e;
    if (s.t_stride <= 0) return hipSuccess;
  } else {
    dim3 g1(pl.pass[0].first[s.B], s.Hkv, n_groups);
    hipLaunchKernelGGL((score_kernel<D, DT, RT, HV, 1, NT_LOADS, OWN_RINGS>), g1, block, 0, stream, s, bp, gp, pl, partials, lse, t_out, s_pool, only_if);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (mid && (e = hipEventRecord(mid, stream)) != hipSuccess) return e;
    if (s.t_stride <= 0) return hipSuccess;
    if (!pl.fold_in_pass2) {
      hipLaunchKernelGGL(fold_kernel, dim3(s.B * s.Hkv, n_groups), dim3(FOLD_THREADS), 0, stream, s, pl, partials, lse, only_if);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
  }
  ScorePlan pl2 = pl;
  if (have_lse) pl2.fold_in_pass2 = false;
  dim3 g2(pl.pass[1].first[s.B], s.Hkv, n_groups);
  hipLaunchKernelGGL((score_kernel<D, DT, RT, HV, 2, NT_LOADS, OWN_RINGS>), g2, block, 0, stream, s, bp, gp, pl2, partials, lse, t_out, s_pool, only_if);
  return hipGetLastError();
}

template <int D, int DT>
static hipError_t launch_rows(const Shape &s, const BatchParams &bp, const ScorePlan &pl, const GroupPtrs &gp, int32_t n_groups,
                              bool have_lse, float2 *partials, float *lse, float *t_out, float *s_pool, hipStream_t stream,
                              hipEvent_t mid, const uint32_t *only_if) {
  // Row tiles per wave: the counts of the usual head layouts (w_obs of 8 to 32 with 1 to 8 query heads per KV
  // head) are met exactly, the rest rounds up; a wave holds eight at most, four of fp32 with 128 channels.
  const int mt = pl.m_pad / 16;
#define WKV_PASSES(RR, HH, ...) \
  launch_passes<D, DT, RR, HH, __VA_ARGS__>(s, bp, pl, gp, n_groups, have_lse, partials, lse, t_out, s_pool, stream, mid, only_if)
#define WKV_ROWS(RR, HH) \
  if (mt <= RR * HH) { \
    if constexpr (HH == 2 && DT != DT_F32) if (pl.own_rings) return WKV_PASSES(RR, HH, false, true); \
    return pl.nontemporal ? WKV_PASSES(RR, HH, true) : WKV_PASSES(RR, HH, false); \
  }
  if constexpr (DT == DT_F32 && D == 128) {
    WKV_ROWS(1, 1) WKV_ROWS(2, 1) WKV_ROWS(4, 1) WKV_ROWS(4, 2) WKV_ROWS(4, 4)
  } else {
    WKV_ROWS(1, 1) WKV_ROWS(2, 1) WKV_ROWS(4, 1) WKV_ROWS(6, 1) WKV_ROWS(7, 1) WKV_ROWS(8, 1) WKV_ROWS(6, 2) WKV_ROWS(7, 2) WKV_ROWS(8, 2)
  }
#undef WKV_ROWS
#undef WKV_PASSES
  return hipErrorInvalidValue;
}

hipError_t launch_score(const Shape &s, const BatchParams &bp, const ScorePlan &pl, const GroupPtrs &gp,
                        int32_t n_groups, bool have_lse, float2 *partials, float *lse, float *t_out, float *s_pool,
                        hipStream_t stream, hipEvent_t mid, const uint32_t *only_if) {
#define WKV_TYPE(DD, TT) return launch_rows<DD, TT>(s, bp, pl, gp, n_groups, have_lse, partials, lse, t_out, s_pool, stream, mid, only_if);
  if (s.d == 128) {
    if (s.dtype == WKV_BF16) WKV_TYPE(128, DT_BF16)
    if (s.dtype == WKV_F16) WKV_TYPE(128, DT_F16)
    WKV_TYPE(128, DT_F32)
  }
  if (s.dtype == WKV_BF16) WKV_TYPE(64, DT_BF16)
  if (s.dtype == WKV_F16) WKV_TYPE(64, DT_F16)
  WKV_TYPE(64, DT_F32)
#undef WKV_TYPE
}

}  // namespace wkv
