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
// Both passes run on the matrix pipe: v_mfma_f32_32x32x16_bf16 / _f16 or _16x16x32 for 16-bit inputs, v_mfma_f32_16x16x4_f32
// for fp32 inputs.  Every wave holds the query fragments of its row tiles in registers for the whole launch and
// reads tiles of 32 or 16 keys from a ring in LDS that it fills itself, by DMA from global memory several tiles
// ahead: the waves of a workgroup do not synchronise in the loop, and nothing but the keys crosses LDS.
#include "wkv_device.h"
#include "wkv_pool.h"

namespace wkv {

// =========================================================================================
// fold: per-chunk (m, z) partials of pass 1 -> one lse2 per row, once per (group, sequence, KV head)
// =========================================================================================
// Partials lie [chunk][row]: the threads of a workgroup take consecutive rows and every so many chunks, so the
// reads are coalesced and, sixteen at a time (64 partials by two threads: two round trips), independent of each other.
constexpr int FOLD_AT_ONCE = 16;
// NT threads fold `rows` rows (at most NT): this thread's row, its first chunk and the chunks from one to the next.
template <int NT>
struct FoldShare {
  int tpr, row, first;
  __device__ __forceinline__ FoldShare(int rows) : tpr(max(NT / rows, 1)) { row = threadIdx.x % (NT / tpr); first = threadIdx.x / (NT / tpr); }
};
// The partials of chunks at + first, tpr further on, ...  (Only as many requests as there are chunks for: each costs time before the
// key stream begins.  By offsets of 32 bits: at most 64 chunks of 256 rows here, and in fold_kernel the 2^15 that a sequence can have.)
template <int NT>
__device__ __forceinline__ void fold_load(float2 (&p)[FOLD_AT_ONCE], const float2 *__restrict__ part, int n_chunks, int m_pad, const FoldShare<NT> &me, int at) {
  const uint32_t step = (uint32_t)(me.tpr * m_pad) * 8u, last = ((uint32_t)(n_chunks - 1) * m_pad + me.row) * 8u;
  uint32_t off = ((uint32_t)(at + me.first) * m_pad + me.row) * 8u;
#pragma unroll
  for (int i = 0; i < FOLD_AT_ONCE; ++i) {
    p[i] = make_float2(-INFINITY, 0.0f);
    if (at + i * me.tpr < n_chunks) p[i] = *(const float2 *)((const char *)part + min(off, last));
    off += step;
  }
}

// lse2 of the rows of one (group, sequence, KV head) into lse[0 .. rows-1] by NT threads; padded rows get +inf
// (2^-inf = 0: they contribute nothing).  p: this thread's first partials, requested by the caller.  part_s: NT entries of scratch.
// Synchronises before it returns.
template <int NT>
__device__ __forceinline__ void fold_all(const Shape &s, int n_chunks, int m_pad, const float2 *__restrict__ part, int rows, const FoldShare<NT> &me,
                                         float2 (&p)[FOLD_AT_ONCE], float2 *part_s, float *lse) {
  float m = -INFINITY, z = 0.0f;
  if (me.row < s.M) {
    for (int at = 0;;) {
      const int c = at + me.first;
      float mn = m;
#pragma unroll
      for (int i = 0; i < FOLD_AT_ONCE; ++i) mn = c + i * me.tpr < n_chunks ? fmaxf(mn, p[i].x) : mn;
      if (mn != -INFINITY) {
        z *= fast_exp2(m - mn);
#pragma unroll
        for (int i = 0; i < FOLD_AT_ONCE; ++i) z += c + i * me.tpr < n_chunks ? p[i].y * fast_exp2(p[i].x - mn) : 0.0f;
        m = mn;
      }
      at += FOLD_AT_ONCE * me.tpr;
      if (at >= n_chunks) break;
      fold_load(p, part, n_chunks, m_pad, me, at);
    }
  }
  part_s[threadIdx.x] = make_float2(m, z);
  __syncthreads();
  if (me.first == 0 && me.row < rows) {
    for (int i = 1; i < me.tpr; ++i) {
      const float2 o = part_s[threadIdx.x + i * (NT / me.tpr)];
      merge_stats(m, z, o.x, o.y);
    }
    lse[me.row] = me.row < s.M ? m + fast_log2(z) : INFINITY;
  }
  __syncthreads();
}

constexpr int FOLD_THREADS = 256;

__global__ __launch_bounds__(FOLD_THREADS) void fold_kernel(Shape s, ScoreArgs a, const float2 *__restrict__ partials,
                                                            float *__restrict__ lse, const uint32_t *__restrict__ only_if) {
  __shared__ float2 part_s[FOLD_THREADS];
  if (only_if && *only_if == 0u) return;
  const int64_t row = (int64_t)blockIdx.y * s.B * s.Hkv + blockIdx.x;
  const int b = blockIdx.x / s.Hkv;
  const FoldShare<FOLD_THREADS> me(a.m_pad);
  const int n_chunks = a.seq[b].n_parts;
  const float2 *part = partials + row * a.n_chunks1 * a.m_pad;
  float2 p[FOLD_AT_ONCE];
  if (me.row < s.M) fold_load(p, part, n_chunks, a.m_pad, me, 0);
  fold_all<FOLD_THREADS>(s, n_chunks, a.m_pad, part, a.m_pad, me, p, part_s, lse + row * a.m_pad);
}

// The base-2 log-sum-exp of softmax row r of a (group, sequence b, KV head h): converted from the
// caller's natural-log normalisers [B, Hq, w_obs] when they were handed over (the rows of a KV
// head are contiguous there), else what the fold left in the workspace.  Padded rows get +inf.
__device__ __forceinline__ float row_lse2(const Shape &s, const float *__restrict__ given, const float *__restrict__ lse_ws, int m_pad, int b, int h,
                                          int64_t row, int r) {
  if (r >= s.M) return INFINITY;
  if (given) return given[((int64_t)b * s.Hq + (int64_t)h * s.G) * s.w_obs + r] * 1.4426950408889634f;
  return lse_ws[row * m_pad + r];
}

// =========================================================================================
// the two passes
// =========================================================================================
// A tile of TS x TS logits takes TS rows of each operand, 64 lanes times 16 bytes per step: lane l holds row l % TS, piece l / TS
// of the step.  TS = 32 (v_mfma_f32_32x32x16) or 16 (v_mfma_f32_16x16x32, fp32: _16x16x4_f32; score_tile says which).  In the result lane l
// holds column l % TS, rows tile_row(e).  Both operands have this layout, so which of them is A is a free choice per pass:
//   PASS 1 (stats)   keys as A: a lane gets TS * TS / 64 keys of ONE query row per row tile, so the row
//                    statistics are in-lane accumulations (RT of them), merged once per chunk.
//   PASS 2 (scores)  queries as A: a lane gets as many query rows of ONE key, so a key's column sum is in-lane adds
//                    over all row tiles plus one or two permlane swaps.
//
// Waves.  HV waves share a key tile slot and take RT row tiles each (128 rows a wave at most, 64 for fp32 with 128
// channels: the queries take RT * TS * D * esize / 256 registers); the KW slots of a workgroup take the chunk's key
// tiles in turn.  Two waves fit a SIMD.
//
// The ring.  A slot has NS places of TS key rows each.  A DMA instruction (global_load_lds_dwordx4) writes 64 pieces
// of 16 bytes in lane order; which piece of its row a lane fetches is permuted (swizzle) so that the 16 lanes
// that later read the same piece of 16 rows find them in different banks.  Global reads stay whole rows.
// A tile is read into registers as a whole (16-row tiles of 16-bit inputs: while the one before is computed) and its place refilled at once; the
// loads are counted by hand (s_waitcnt vmcnt), which holds because the loop has no other global access.  With one row group
// a wave fills its own slot and the waves never synchronise in the loop.  With several, the waves of a slot fetch a part
// of each tile and the workgroup meets at a barrier per tile (a place is then refilled one tile later, when all have read it), or
// (OWN_RINGS, two groups of 16-bit inputs) every wave
// fetches whole tiles for itself: half the bytes in flight, no barriers, and the second of a slot's waves finds the
// tile in the L2, as long as the two do not drift too far apart (see plan_score).
//
// What bounds it.  Per 64 logits a SIMD issues a multiply-add, an exponential and an add (16 cycles) and one 16x16x32 MFMA or half a
// 32x32x16 one (16 cycles of the matrix pipe).  In a loop of nothing else, two waves a SIMD: 34 cycles with 16-row tiles, 29 with 32-row
// tiles, 26 where two waves take turns at the two by barriers; 18.1, 14.5 and 13.3 ns, as the clock falls from 2.4 to 1.9-2.0 GHz on random data
// (it does not with zeros).  So a pass that lasts and also streams keys is bound by power: the 32K-token model (8 groups, 128
// rows) takes 90 + 90 us from first wave to last, 84-86 without the arithmetic, 69 without the loads, and with 32-row tiles the clock is
// 1.8-2.0 instead of 2.1-2.2 GHz: the same time, 4 % more for the second pass of the handed-over normalisers where the chip is warm.  Eight
// waves in one workgroup, or paced by a barrier every 1 to 8 tiles so that none runs ahead: 105-125 us.  With two row groups the
// arithmetic is what takes longest, and 32-row tiles pay however long the stream is (score_tile has both sides).
// A workgroup's start, in microseconds for 4096 tokens (second pass of the 32K model): arguments and the first key requests 1.4 (2.4), queries 0.8
// (1.5), partials to normalisers 0.8 (1.2), queries to registers 0.6 (0.7).  Requests are issued at 20 bytes a cycle and compute unit, so the 32 KB of queries cost what as many
// keys cost.  The fold's requests stand before the queries', not behind them: 1.8 (3.6) us for the fold before.  Requested by whole rows instead
// of fragments, the queries of 256 rows take 1.9 instead of 2.6 us.
// The start runs through its code once, at some 7 cycles an instruction (each launch fetches it anew), so its length counts as well: 120 comparisons of
// the unrolled windows, which the compiler had put ahead of the key stream, 50 instructions per query request and 10 per partial, and a third trip
// for arguments of the fold.  Without them 4096 tokens 22.25 -> 21.1 us a call, 16384 with sorted windows 41.2 -> 38.9, 256 rows of 16381 in 8 groups 277 -> 274.
constexpr int score_slots(int row_groups) { return row_groups == 4 ? 2 : 4; }         // key tile slots of a workgroup
constexpr int score_threads(int row_groups) { return 64 * row_groups * score_slots(row_groups); }

template <int D, int DT, int TS_, int RT, int HV, bool OWN_RINGS>
struct ScoreConfig {
  static constexpr int ES = DT == DT_F32 ? 4 : 2;       // bytes per element
  static constexpr int TS = TS_, E = TS * TS / 64;      // rows of a tile, logits of a lane
  static constexpr int PPS = 64 / TS;                   // 16-byte pieces of a row per step of a contraction
  static constexpr int ROWB = D * ES;                   // bytes per key row
  static constexpr int PPR = ROWB / 16;                 // pieces per row: 8, 16 or 32
  static constexpr int KS = PPR / PPS;                  // steps of a contraction
  static constexpr int TILE = TS * ROWB;
  static constexpr int RPI = 64 / PPR;                  // rows per DMA instruction
  static constexpr bool SHARED = HV > 1 && !OWN_RINGS;
  static constexpr int PARTS = SHARED ? HV : 1;         // waves that fetch a tile together
  static constexpr int LPT = TILE / 1024 / PARTS;       // DMA instructions per tile and wave
  static constexpr int OFFS = LPT < 16 / RPI ? LPT : 16 / RPI;     // of them with offsets of their own (rows 16 apart are swizzled alike)
  static constexpr int KW = score_slots(HV), NT = score_threads(HV), WAVES = NT / 64;
  static constexpr int RINGS = SHARED ? KW : WAVES;
  static constexpr int FIT = (HV == 1 ? 65536 : 131072) / (RINGS * TILE);
  static constexpr int NS = FIT < 8 * PARTS ? FIT : 8 * PARTS;
  static constexpr int RING = RINGS * NS * TILE;
  // the queries pass through the part of the ring that is filled last
  static constexpr int QBYTES = HV * RT * TILE;
  static constexpr int FIRST = NS - (QBYTES + RINGS * TILE - 1) / (RINGS * TILE);
  static_assert(FIRST >= 0, "the queries fit the ring");
  static_assert(NS >= 2, "a tile being read and one under way");
  // With 16-row tiles the next tile's fragments are read while this one is computed.  fp32: a tile takes thousands of cycles on the
  // matrix pipe, and its fragments twice the registers.
  static constexpr bool AHEAD = DT != DT_F32 && TS == 16;
  static constexpr int SEG = HV == 4 ? SCORE_SEG / 2 : SCORE_SEG;
  static constexpr int T_S = SEG + KW * TS;             // token scores of a segment, and of the tiles that reach past its end
  // where piece p of row r lies within its row's slot
  static __device__ __forceinline__ int swizzle(int r, int p) { return p ^ (PPR == 8 ? (r >> 1) & 7 : r & 15); }
  // row of a result that element e of a lane belongs to; sub: lane / TS
  static __device__ __forceinline__ int tile_row(int sub, int e) { return e / 4 * (4 * PPS) + sub * 4 + e % 4; }
};

// At most N loads outstanding, every LDS read returned.
template <int N>
__device__ __forceinline__ void wait_vmcnt() { asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory"); }

// A DMA instruction of the ring from base + off bytes (wkv_device.h has the one with an address per lane).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <bool NT_LOADS>
__device__ __forceinline__ void dma_to_lds(uint32_t lds, const char *base, uint32_t off) {
  if constexpr (NT_LOADS)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(lds), "v"(off), "s"(base) : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(off), "s"(base) : "memory", "m0");
}
#pragma clang diagnostic pop

// NT_LOADS: the keys are not put into the memory-side cache (see plan_score).  Kernels of their own, as a branch at every fetch
// costs small calls 1 %.
// TS: rows of a tile (see score_tile in wkv_host.cpp).  WAVE_ROWS: rows a wave takes, in RT tiles.
template <int D, int DT, int WAVE_ROWS, int HV, int PASS, int TS, bool NT_LOADS, bool OWN_RINGS>
__global__ __launch_bounds__(score_threads(HV), 2) void score_kernel(Shape s, ScoreArgs a,
                                                                                 float2 *__restrict__ partials,
                                                                                 const float *__restrict__ lse_g,
                                                                                 float *__restrict__ t_out,
                                                                                 float *__restrict__ s_pool,
                                                                                 const uint32_t *__restrict__ only_if) {
  constexpr int RT = WAVE_ROWS / TS;
  using C = ScoreConfig<D, DT, TS, RT, HV, OWN_RINGS>;
  constexpr int KS = C::KS, KW = C::KW, NT = C::NT, NS = C::NS, E = C::E, ROWS = HV * RT * TS;
  __shared__ __attribute__((aligned(1024))) char ring[C::RING];
  __shared__ __attribute__((aligned(16))) float t_s[PASS == 2 ? HV * C::T_S : 4];     // token scores of a segment
  __shared__ __attribute__((aligned(16))) float lse_s[PASS == 2 ? ROWS : 4];
  __shared__ float2 part_s[PASS == 2 ? NT : KW * ROWS];
  // First trip for arguments: all at fixed places, requested together (see ScoreArgs; left to itself the compiler asks for each where it is used).
  int ends[ENDS_AT_ONCE];
#pragma unroll
  for (int i = 0; i < ENDS_AT_ONCE; ++i) ends[i] = a.ends[i];
  asm volatile("" ::"s"(ends[0]), "s"(ends[1]), "s"(ends[2]), "s"(ends[3]), "s"(ends[4]), "s"(ends[5]), "s"(ends[6]), "s"(ends[7]),
               "s"(s.B), "s"(s.Hkv), "s"(s.w_obs), "s"(s.G), "s"(s.M), "s"(s.kv_st), "s"(s.kv_sh), "s"(s.kv_sb), "s"(s.q_st), "s"(s.q_sh), "s"(s.q_sb),
               "s"(a.hkv_magic), "s"(a.row_bits), "s"(a.last_x), "s"(a.last_y), "s"(a.last_z), "s"(a.items), "s"(only_if));
  asm volatile("" ::"s"(partials), "s"(a.m_pad), "s"(a.n_chunks1), "s"(a.fold), "s"(s.w_magic), "s"(s_pool));
  // Launched behind the single-read kernel as its fall-back: nothing to do unless that kernel
  // raised the word (uniform over the grid).
  if (only_if && *only_if == 0u) return;

  // Pass 2 walks the work items in the opposite order of pass 1: the keys pass 1 read last
  // are the ones most likely still held by the memory-side cache.
  const bool back = PASS == 2;
  const ScoreItem item(back && a.row_bits == 0 ? a.last_x - blockIdx.x : blockIdx.x, back ? a.last_y - blockIdx.y : blockIdx.y,
                       back ? a.last_z - blockIdx.z : blockIdx.z, a.row_bits, s.Hkv, a.hkv_magic);
  const int x = item.item;
  if (x >= a.items) return;
  const int g = item.group, h = item.head;
  int b = 0;
#pragma unroll
  for (int i = 0; i < ENDS_AT_ONCE; ++i) b += x >= ends[i];
  if (b == ENDS_AT_ONCE)
    while (b + 1 < s.B && x >= a.ends[b]) ++b;
  // Second trip: the sequence and the group.
  const ScoreSeq seq = a.seq[b];
  const char *k_layer = (const char *)a.gp.k[g], *q_layer = (const char *)a.gp.q[g];
  const float *given = a.gp.lse[g];
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::"s"(seq.L), "s"(seq.first), "s"(seq.n_parts), "s"(seq.packed), "s"(seq.win_magic), "s"(seq.last), "s"(k_layer), "s"(q_layer), "s"(given));
  const int bx = x - seq.first;                             // chunk of the sequence
  const int L = seq.L;
  const int n_review = L - s.w_obs;
  const int64_t row = ((int64_t)g * s.B + b) * s.Hkv + h;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int half = wave / KW, kw = wave % KW;               // row group, key tile slot of this wave
  const int col = lane % TS, sub = lane / TS;
  const int my_ring = C::SHARED ? kw : wave, my_part = C::SHARED ? half : 0;

  const int chunk = (seq.packed & 0xff) * CHUNK_UNIT;
  const int limit = PASS == 1 ? L : n_review;               // keys that matter to this pass
  const int c_first = bx * chunk;
  int c0 = c_first, cend = min(c0 + chunk, limit);          // keys c0 .. cend-1 of the row
  int seg_len = PASS == 1 ? 0x40000000 : C::SEG;            // pass 2 writes its scores out a segment at a time
  int win = 1;
  uint32_t win_magic = 0u;
  if (PASS == 2 && s_pool) {
    // A window belongs to the chunk that holds its first token: the workgroup scores and pools whole
    // windows, whatever their size, and no token is scored twice.
    win = seq.packed >> 8 & 0xff;
    win_magic = seq.win_magic;
    c0 = divide(c0 + win - 1, win_magic) * win;
    cend = min(divide(cend + win - 1, win_magic) * win, limit);
    seg_len = divide(C::SEG, win_magic) * win;
  }
  float *trow = PASS == 2 ? t_out + row * s.t_stride : nullptr;
  if (PASS == 2 && !s_pool)                                 // the row's padding
    for (int j = n_review + threadIdx.x; j < (x == seq.last ? s.t_stride : 0); j += NT) trow[j] = 0.0f;
  if (PASS == 2 && c0 >= cend) return;
  float2 *part = partials + row * a.n_chunks1 * a.m_pad;

  // ---- the key stream -------------------------------------------------------------------------
  const char *kbase = k_layer + ((int64_t)b * s.kv_sb + (int64_t)h * s.kv_sh) * C::ES;
  const int64_t kst = s.kv_st * C::ES;
  // rows too far apart for 32-bit offsets within a tile: below that 16 rows span less than 2 GiB, and the 31 that the offsets of a shared
  // 32-row tile's second part reach over less than 4
  const bool wide = kst * 16 >= 0x7fffffff;
  const int row_in_part = my_part * (C::LPT * C::RPI) + lane / C::PPR;      // of this lane's first DMA instruction
  uint32_t off[C::OFFS];                                    // this lane's pieces, from the first row of its 16
#pragma unroll
  for (int n = 0; n < C::OFFS; ++n) {
    const int r = row_in_part + n * C::RPI;
    off[n] = (uint32_t)r * (uint32_t)kst + C::swizzle(r, lane % C::PPR) * 16;
  }
  const uint32_t ring_lds = lds_address(ring) + my_ring * (NS * C::TILE) + my_part * (C::LPT * 1024);
  // keys j .. j+TS-1 (this wave's part) into place `slot`; rows from cend on are not read (their lanes fetch row cend-1 again)
  auto fetch = [&](int j, int slot) __attribute__((always_inline)) {
    const uint32_t dst = ring_lds + slot * C::TILE;
    if (j + TS <= cend && !wide) {
#pragma unroll
      for (int n = 0; n < C::LPT; ++n)
        dma_to_lds<NT_LOADS>(dst + n * 1024, kbase + (int64_t)(j + n / C::OFFS * 16) * kst, off[n % C::OFFS]);
    } else {
      int first = row_in_part;
      asm volatile("" : "+v"(first));                       // what follows from it is not kept in registers between tiles
#pragma unroll
      for (int n = 0; n < C::LPT; ++n) {
        const int r = first + n * C::RPI;
        const char *p = kbase + (int64_t)min(j + r, cend - 1) * kst + C::swizzle(r, lane % C::PPR) * 16;
        dma_to_lds(dst + n * 1024, p);
      }
    }
  };
  // The order of this wave's tiles: KW apart within a segment, segment by segment.
  int jf = c0 + kw * TS, jf_end = min(c0 + seg_len, cend), slot_f = 0;      // the next tile to fetch
  auto fetch_next = [&]() __attribute__((always_inline)) {
    fetch(jf, slot_f);
    slot_f = slot_f == NS - 1 ? 0 : slot_f + 1;
    jf += KW * TS;
    while (PASS == 2 && (C::SHARED ? jf - kw * TS : jf) >= jf_end && jf_end < cend) {
      jf = jf_end + kw * TS;
      jf_end = min(jf_end + seg_len, cend);
    }
  };
#pragma unroll
  for (int i = 0; i < C::FIRST; ++i) fetch_next();

  // ---- the partials that this thread folds: requested here, they arrive together with the keys and the queries
  const FoldShare<NT> share(ROWS);
  const int n_parts = seq.n_parts;
  float2 parts[PASS == 2 ? FOLD_AT_ONCE : 1];
  if constexpr (PASS == 2)
    if (a.fold && share.row < s.M) fold_load(parts, part, n_parts, a.m_pad, share, 0);

  // ---- the queries: into the ring's other places, tiles of rows as the keys', from there into registers as fragments.  Rows past the
  // last one repeat it: their statistics are never used and their normaliser is +inf.
  constexpr int PIECES = HV * RT * KS, PER_RING = (NS - C::FIRST) * KS;          // DMA instructions: all, what a ring takes
  auto query_at = [&](int f) __attribute__((always_inline)) { return f / PER_RING * (NS * C::TILE) + C::FIRST * C::TILE + f % PER_RING * 1024; };
  const char *qbase = q_layer + ((int64_t)b * s.q_sb + (int64_t)(h * s.G) * s.q_sh) * C::ES;
  // rows one after the other at equal distances, as in a contiguous tensor: one offset per lane serves them all
  const bool even = s.q_sh == (int64_t)s.w_obs * s.q_st && s.q_st < 0x1000000;
  const uint32_t q_lane = (uint32_t)(lane / C::PPR) * (uint32_t)s.q_st * C::ES;
  // (whole groups of such rows without a loop: one would compute its addresses anew for every instruction, 0.3 to 0.5 us of a workgroup's start.
  // The rows of a wave are STEP apart, a power of two, so that the swizzle of the later ones differs from the first one's by constants.)
  constexpr int STEP = C::WAVES * C::RPI;
  const int whole = even ? s.M / C::RPI : 0;                  // DMA instructions
  const int row0 = wave * C::RPI + lane / C::PPR;
  const uint32_t piece0 = C::swizzle(row0, lane % C::PPR) * 16;
  const char *qp = qbase + (int64_t)(wave * C::RPI) * s.q_st * C::ES;
#pragma unroll
  for (int i = 0; i * C::WAVES < PIECES; ++i) {
    const int f = wave + i * C::WAVES;
    const uint32_t turned = (C::PPR == 8 ? (i * STEP >> 1) & 7 : (i * STEP) & 15) * 16;
    if (f < (PIECES < whole ? PIECES : whole))
      dma_to_lds<false>(lds_address(ring) + (PER_RING % C::WAVES == 0 ? query_at(i * C::WAVES) + wave * 1024 : query_at(f)), qp, q_lane + (piece0 ^ turned));
    qp += (int64_t)STEP * s.q_st * C::ES;
  }
  for (int f = wave + (whole + C::WAVES - 1 - wave) / C::WAVES * C::WAVES; f < PIECES; f += C::WAVES) {
    const int row = f * C::RPI + lane / C::PPR, r = min(row, s.M - 1);
    const int hq = (int)((uint32_t)r * s.w_magic >> 16), io = r - hq * s.w_obs;      // r / w_obs, r % w_obs
    dma_to_lds(lds_address(ring) + query_at(f), qbase + ((int64_t)hq * s.q_sh + (int64_t)io * s.q_st) * C::ES + C::swizzle(row, lane % C::PPR) * 16);
  }
  if (PASS == 2) {
    if (a.fold) {
      if constexpr (PASS == 2) fold_all<NT>(s, n_parts, a.m_pad, part, ROWS, share, parts, part_s, lse_s);
    } else
      for (int r = threadIdx.x; r < ROWS; r += NT) lse_s[r] = row_lse2(s, given, lse_g, a.m_pad, b, h, row, r);
  }
  wait_vmcnt<0>();
  __syncthreads();
  bf16x8 qf[RT][KS];
#pragma unroll
  for (int mt = 0; mt < RT; ++mt)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      qf[mt][ks] = *(const bf16x8 *)(ring + query_at((half * RT + mt) * KS) + ((col * C::ROWB + C::swizzle(col, sub) * 16) ^ (ks * C::PPS * 16)));
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __syncthreads();
  // a place of shared rings stays empty until the first tile has been read by all, unless a tile is read ahead
  constexpr bool LATE = C::SHARED && !C::AHEAD;
#pragma unroll
  for (int i = C::FIRST; i < NS - (LATE ? 1 : 0); ++i) fetch_next();
  const float sc = s.c1;
  float mref[PASS == 1 ? RT : 1], zsum[PASS == 1 ? RT : 1];  // pass 1: reference and sum of query row (half*RT + mt)*TS + col
  bool settled = false;                                     // (uniform) every sum of this wave is large enough for its reference
  if (PASS == 1) {
#pragma unroll
    for (int mt = 0; mt < RT; ++mt) { mref[mt] = 0.0f; zsum[mt] = 0.0f; }
  }

  // ---- tiles -----------------------------------------------------------------------------------
  // Meeting of the workgroup without the wait for outstanding loads that __syncthreads() brings.
  auto barrier = [&]() __attribute__((always_inline)) { asm volatile("s_barrier" ::: "memory"); };
  typedef typename TileOf<TS>::acc acc_t;
  struct Frags { bf16x8 f[KS]; } kf, kn;                    // this tile's keys, the next one's
  uint32_t read_at = my_ring * (NS * C::TILE) + col * C::ROWB + C::swizzle(col, sub) * 16;     // of the place read next
  const uint32_t ring_end = (my_ring + 1) * (NS * C::TILE);
  auto read_keys = [&](Frags &k) __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) k.f[ks] = *(const bf16x8 *)(ring + (read_at ^ (ks * C::PPS * 16)));       // swizzle(col, ks * PPS + sub)
    read_at += C::TILE;
    if (read_at >= ring_end) read_at -= NS * C::TILE;
  };
  auto logits = [&](int mt) __attribute__((always_inline)) {
    acc_t acc = {};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      acc = PASS == 1 ? mfma_step<DT, TS>(kf.f[ks], qf[mt][ks], acc) : mfma_step<DT, TS>(qf[mt][ks], kf.f[ks], acc);
    return acc;
  };

  // Statistics of one tile, with care: the causal mask (key j visible to observation query io iff
  // j <= n_review + io), the end of the sequence, and rows whose reference does not suit their logits.  A
  // reference is good while the sum taken with it stays between MF_LOW (what underflowed is negligible) and
  // MF_BIG; otherwise it moves to the larger of the tile's maximum and the sum so far.
  auto careful = [&](int j0) __attribute__((always_inline)) {
#pragma unroll
    for (int mt = 0; mt < RT; ++mt) {
      acc_t acc = logits(mt);
      const int r = min((half * RT + mt) * TS + col, s.M - 1);
      const int last = min(n_review + r - (int)((uint32_t)r * s.w_magic >> 16) * s.w_obs, cend - 1);
      float vmax = -INFINITY, a = 0.0f;
#pragma unroll
      for (int e = 0; e < E; ++e) {
        acc[e] = j0 + C::tile_row(sub, e) <= last ? acc[e] * sc : -INFINITY;
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
          for (int e = 0; e < E; ++e) a += fast_exp2(acc[e] - nref);
          mref[mt] = nref;
          zsum[mt] = a;
        }
      } else {
        zsum[mt] = z + a;
      }
    }
  };

  // The row tiles of one key tile: the MFMAs of a row tile beside the exponentials of the one before.  A row tile past the
  // last row is left out (of the last row group, where the counts do not divide).
  const bool one_less = HV > 1 && (half * RT + RT - 1) * TS >= s.M;                    // uniform
  auto left_out = [&](int mt) __attribute__((always_inline)) { return HV > 1 && mt == RT - 1 && one_less; };
  auto statistics = [&](int j0) __attribute__((always_inline)) {
    bool care = j0 + TS > min(n_review, cend);              // uniform
    if (!care) {
      acc_t acc[RT];
      float psum[RT];
#pragma unroll
      for (int mt = 0; mt <= RT; ++mt) {
        if (mt < RT && !left_out(mt)) acc[mt] = logits(mt);
        if (mt > 0 && !left_out(mt - 1)) {
          const int m1 = mt - 1;
          float a[4];                                       // (four sums: half the additions one after the other, and less rounding)
#pragma unroll
          for (int e = 0; e < E; ++e) {
            const float x = fast_exp2(fmaf(acc[m1][e], sc, -mref[m1]));
            a[e % 4] = e < 4 ? x : a[e % 4] + x;
          }
          psum[m1] = (a[0] + a[1]) + (a[2] + a[3]);
        }
      }
      if (left_out(RT - 1)) psum[RT - 1] = psum[0];         // (any sum that does not ask for care)
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
      careful(j0);
      if (!settled) {
        float low = zsum[0];
#pragma unroll
        for (int mt = 1; mt < RT; ++mt) low = fminf(low, zsum[mt]);
        settled = __all(low >= MF_LOW);
      }
    }
  };
  auto scores = [&](int j0, int seg0) __attribute__((always_inline)) {
    // 32-row tiles: a tile's MFMAs, then its exponentials, as two tiles' results would not fit; the SIMD's other wave fills the gaps
    constexpr int LAG = TS == 16 ? 1 : 0;
    float t[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    acc_t acc[RT];
#pragma unroll
    for (int mt = 0; mt < RT + LAG; ++mt) {
      if (mt < RT && !left_out(mt)) acc[mt] = logits(mt);
      if (mt >= LAG && !left_out(mt - LAG)) {
        const int m1 = mt - LAG;
#pragma unroll
        for (int e = 0; e < E; e += 4) {
          // (from LDS every time: E * RT of them would not fit beside the queries)
          const f32x4 lse = *(const f32x4 *)&lse_s[(half * RT + m1) * TS + C::tile_row(sub, e)];
          t[e / 4 % 2 * 2] += fast_exp2(fmaf(acc[m1][e], sc, -lse[0]));
          t[e / 4 % 2 * 2 + 1] += fast_exp2(fmaf(acc[m1][e + 1], sc, -lse[1]));
          t[e / 4 % 2 * 2] += fast_exp2(fmaf(acc[m1][e + 2], sc, -lse[2]));
          t[e / 4 % 2 * 2 + 1] += fast_exp2(fmaf(acc[m1][e + 3], sc, -lse[3]));
        }
        if (TS == 32) asm volatile("" ::: "memory");        // the normalisers of the next tile are not loaded yet, for want of registers
      }
    }
    // (the lanes of a key store the same value to the same place: no branch in the loop)
    const float sum = TS == 16 ? t[0] + t[1] : (t[0] + t[1]) + (t[2] + t[3]);
    t_s[half * C::T_S + j0 - seg0 + col] = TS == 16 ? quads_sum(sum) : add_halves(sum, sum);
  };

  if constexpr (C::AHEAD) {
    wait_vmcnt<(NS - 1) * C::LPT>();
    if (C::SHARED) barrier();
    read_keys(kf);
  }
  for (int seg0 = c0; seg0 < cend; seg0 += seg_len) {
    const int seg_end = min(seg0 + seg_len, cend);
    // with row groups every slot takes a tile in every round, if need be one past the end (masked in pass 1, past the
    // scores that count in pass 2): the waves meet at barriers
    for (int j = seg0 + kw * TS; (C::SHARED ? j - kw * TS : j) < seg_end; j += KW * TS) {
      if constexpr (C::AHEAD) {                             // the next tile out of the ring, a later one into the place this one left
        wait_vmcnt<(NS - 2) * C::LPT>();
        if (C::SHARED) barrier();                           // (every part of it; every wave has this tile in registers)
        read_keys(kn);
      } else {                                              // this tile out of the ring, a later one into its place or (LATE) that of the one before
        wait_vmcnt<(NS - (LATE ? 2 : 1)) * C::LPT>();
        if (C::SHARED) barrier();
        read_keys(kf);
        if (!LATE) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      }
      fetch_next();
      if (PASS == 1) statistics(j); else scores(j, seg0);
      if (C::AHEAD) kf = kn;
    }
    if (PASS == 1) break;
    __syncthreads();
    if (HV > 1) {                                           // column sums of the other row groups
      for (int i = threadIdx.x; i < seg_end - seg0; i += NT) {
        float x = t_s[i];
#pragma unroll
        for (int v = 1; v < HV; ++v) x += t_s[v * C::T_S + i];
        t_s[i] = x;
      }
      __syncthreads();
    }
    if (s_pool) {                                           // Eq. 3-4 while the token scores are in LDS
      // (what the compiler knows nothing of before: else the hundred comparisons of the unrolled windows stand ahead of the key stream)
      int w_here = win, p_here = (int)(seq.packed >> 16);
      asm volatile("" : "+s"(w_here), "+s"(p_here));
      pool_windows<NT>(t_s, divide(seg0, win_magic), divide(seg_end + win - 1, win_magic), w_here, p_here, n_review, s_pool + row * s.nw_max);
    } else
      for (int i = threadIdx.x; i < seg_end - seg0; i += NT) trow[seg0 + i] = t_s[i];
    if (seg_end == cend) break;
    __syncthreads();
  }

  if (PASS == 1) {
    // merge the lanes of each row, then the KW waves
#pragma unroll
    for (int mt = 0; mt < RT; ++mt) {
      float m = zsum[mt] > 0.0f ? mref[mt] : -INFINITY, z = zsum[mt];
      Pair pm = swap_halves(m, m), pz = swap_halves(z, z);
      merge_stats(pm.a, pz.a, pm.b, pz.b);
      if constexpr (TS == 16) {
        m = pm.a; z = pz.a;
        pm = swap_rows(m, m); pz = swap_rows(z, z);
        merge_stats(pm.a, pz.a, pm.b, pz.b);
      }
      if (sub == 0) part_s[kw * ROWS + (half * RT + mt) * TS + col] = make_float2(pm.a, pz.a);
    }
    __syncthreads();
    for (int r = threadIdx.x; r < a.m_pad; r += NT) {           // m_pad <= ROWS
      float m = part_s[r].x, z = part_s[r].y;
      for (int w = 1; w < KW; ++w) merge_stats(m, z, part_s[w * ROWS + r].x, part_s[w * ROWS + r].y);
      part[(int64_t)bx * a.m_pad + r] = make_float2(m, z);
    }
  }
}

// =========================================================================================
// launch
// =========================================================================================
template <int D, int DT, int WAVE_ROWS, int HV, int TS, bool NT_LOADS, bool OWN_RINGS = false>
static hipError_t launch_passes(const Shape &s, const BatchParams &bp, const ScorePlan &pl, const GroupPtrs &gp, int32_t n_groups,
                                bool have_lse, float2 *partials, float *lse, float *t_out, float *s_pool, hipStream_t stream,
                                hipEvent_t mid, const uint32_t *only_if) {
  const dim3 block(score_threads(HV));
  ScoreArgs a;
  ScoreGrid grid;
  hipError_t e;
  if (have_lse) {                                      // no statistics pass: pass 2 reads the caller's normalisers
    if (mid && (e = hipEventRecord(mid, stream)) != hipSuccess) return e;
    if (s.t_stride <= 0) return hipSuccess;
  } else {
    fill_score_args(s, bp, pl, gp, n_groups, 0, false, &a, &grid);
    hipLaunchKernelGGL((score_kernel<D, DT, WAVE_ROWS, HV, 1, TS, NT_LOADS, OWN_RINGS>), dim3(grid.x, grid.y, grid.z), block, 0, stream, s, a, partials, lse, t_out, s_pool, only_if);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (mid && (e = hipEventRecord(mid, stream)) != hipSuccess) return e;
    if (s.t_stride <= 0) return hipSuccess;
    if (!pl.fold_in_pass2) {
      hipLaunchKernelGGL(fold_kernel, dim3(s.B * s.Hkv, n_groups), dim3(FOLD_THREADS), 0, stream, s, a, partials, lse, only_if);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
  }
  fill_score_args(s, bp, pl, gp, n_groups, 1, pl.fold_in_pass2 && !have_lse, &a, &grid);
  hipLaunchKernelGGL((score_kernel<D, DT, WAVE_ROWS, HV, 2, TS, NT_LOADS, OWN_RINGS>), dim3(grid.x, grid.y, grid.z), block, 0, stream, s, a, partials, lse, t_out, s_pool, only_if);
  return hipGetLastError();
}

template <int D, int DT>
static hipError_t launch_rows(const Shape &s, const BatchParams &bp, const ScorePlan &pl, const GroupPtrs &gp, int32_t n_groups,
                              bool have_lse, float2 *partials, float *lse, float *t_out, float *s_pool, hipStream_t stream,
                              hipEvent_t mid, const uint32_t *only_if) {
  // Rows per wave: the counts of the usual head layouts (w_obs of 8 to 32 with 1 to 8 query heads per KV head) in steps of 32, those
  // of 16 where it pays (score_tile); a wave holds 128 at most, 64 of fp32 with 128 channels.
#define WKV_PASSES(RR, HH, ...) \
  if (s.M <= RR * HH) return launch_passes<D, DT, RR, HH, __VA_ARGS__>(s, bp, pl, gp, n_groups, have_lse, partials, lse, t_out, s_pool, stream, mid, only_if);
#define WKV_ROWS(RR, HH) if (pl.nontemporal) { WKV_PASSES(RR, HH, 16, true) } else { WKV_PASSES(RR, HH, 16, false) }
  if constexpr (DT == DT_F32 && D == 128) {
    WKV_ROWS(16, 1) WKV_ROWS(32, 1) WKV_ROWS(64, 1) WKV_ROWS(64, 2) WKV_ROWS(64, 4)
  } else if constexpr (DT == DT_F32) {
    WKV_ROWS(16, 1) WKV_ROWS(32, 1) WKV_ROWS(64, 1) WKV_ROWS(96, 1) WKV_ROWS(112, 1) WKV_ROWS(128, 1) WKV_ROWS(96, 2) WKV_ROWS(112, 2) WKV_ROWS(128, 2)
  } else if (pl.tile == 16) {
    if (!pl.nontemporal) { WKV_PASSES(112, 1, 16, false) }
    else if constexpr (D == 64) { WKV_PASSES(112, 1, 16, true) }
    else { WKV_PASSES(16, 1, 16, true) WKV_PASSES(32, 1, 16, true) WKV_PASSES(64, 1, 16, true) WKV_PASSES(96, 1, 16, true) WKV_PASSES(112, 1, 16, true) WKV_PASSES(128, 1, 16, true) }
  } else if (pl.nontemporal) {
    if constexpr (D == 64) { WKV_PASSES(32, 1, 32, true) WKV_PASSES(64, 1, 32, true) WKV_PASSES(96, 1, 32, true) WKV_PASSES(128, 1, 32, true) }
    WKV_PASSES(96, 2, 32, true) WKV_PASSES(128, 2, 32, true)
  } else {
    WKV_PASSES(32, 1, 32, false) WKV_PASSES(64, 1, 32, false) WKV_PASSES(96, 1, 32, false) WKV_PASSES(128, 1, 32, false)
    if (pl.own_rings) { WKV_PASSES(96, 2, 32, false, true) WKV_PASSES(128, 2, 32, false, true) }
    WKV_PASSES(96, 2, 32, false) WKV_PASSES(128, 2, 32, false)
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
