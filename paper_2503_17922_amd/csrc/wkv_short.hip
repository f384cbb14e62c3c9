// A whole call (WindowKV Section 2.2: scores, pooling, selection, gather) in one launch, for short prompts.
//
// Launched one after the other, the passes of such a call wait for launches, arguments and first loads and compute next to nothing: 512
// fp32 tokens of two KV heads 5 + 7 + 4 us from first wave to last, 1 us between.  A row (group, sequence, KV head) of a short prompt is so little
// that every workgroup scores and selects it for itself, from one read of its keys, and copies its share of the kept rows of one
// tensor: nothing passes between workgroups.
//
// A wave takes every eighth tile of 16 keys, whole rows through LDS into registers, then the queries take that place in LDS.  It keeps
// its logits: statistics per row (keys as A: those of a lane belong to one query row per row tile), merged over the waves in LDS, then the
// column sums from the same registers.  So the logits and their exponentials are computed once; what is summed is what the two passes sum, and
// window scores are 1.3 to 2.8e-7 off their 64-bit values (2-norm) where those of the passes are 3.1 to 3.9e-7.
//
// Us a call of four layers by the passes / so: 512 tokens bf16, 128 channels, 16 rows a KV head 15.4 / 7.9, 32 15.4 / 9.5, 64 16.5 / 11.0, 128 18.9 / 14.4; 1000
// tokens, 16 rows 15.6 / 9.7, 32 15.8 / 11.9; fp32, 64 channels, 512 tokens, 16 rows 18.0 / 9.4.  Keys in operand layout straight from memory instead of
// whole rows through LDS: 10.7 for the first, 15.5 for 1000 tokens.  One row tile at a time in a loop, its logits computed once for the statistics
// and again for the scores: 8.9, and 19.2 with 128 rows.
#include "wkv_pool.h"
#include "wkv_select.h"

namespace wkv {

constexpr int SHORT_THREADS = 512, SHORT_WAVES = SHORT_THREADS / 64;
static_assert(SHORT_TOKENS == SHORT_THREADS, "a token a thread");

struct ShortScore {
  const void *q[SMALL_GROUPS];
  const float *lse[SMALL_GROUPS];               // the caller's normalisers, or all null
};

// RT row tiles; KT key tiles a wave.
template <int D, int DT, int RT, int KT>
__global__ __launch_bounds__(SHORT_THREADS, 2) void short_kernel(Shape s, SmallJob job, ShortScore in, float *__restrict__ sc, int32_t *__restrict__ win_idx,
                                                                 int32_t *__restrict__ tok_idx, int32_t *__restrict__ n_keep) {
  constexpr int ES = DT == DT_F32 ? 4 : 2, ROWB = D * ES, PPR = ROWB / 16, KS = PPR / 4, ROWS = RT * 16, KEYS = KT * 16 * SHORT_WAVES, NT = SHORT_THREADS;
  constexpr int TILE = 16 * ROWB, KR = 131072 / (SHORT_WAVES * TILE);      // key tiles of a wave that LDS holds at a time
  constexpr int RING = (KR < KT ? KR : KT) * TILE;                // of a wave
  __shared__ __attribute__((aligned(1024))) char ring[SHORT_WAVES * RING > ROWS * ROWB ? SHORT_WAVES * RING : ROWS * ROWB];      // keys, then queries
  __shared__ __attribute__((aligned(16))) float t_s[KEYS];        // token scores
  __shared__ float win_s[KEYS];                                   // window scores
  __shared__ uint32_t keys[KEYS];                                 // the selection's
  __shared__ float2 part_s[SHORT_WAVES][ROWS];
  __shared__ float lse_s[ROWS];
  // Two trips to memory for the arguments, as in the other kernels of a call.
  const int bh = blockIdx.x, split = blockIdx.y, layer = blockIdx.z >> 1, is_v = blockIdx.z & 1;
  const char *src = (const char *)job.in[layer][is_v];
  char *dst = (char *)job.out[layer][is_v];
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::"s"(src), "s"(dst), "s"(s.B), "s"(s.Hkv), "s"(s.hkv_magic), "s"(s.w_obs), "s"(s.nw_max), "s"(s.k_max), "s"(s.nkeep_max), "s"(s.fill_padding),
               "s"(s.kv_sb), "s"(s.kv_sh), "s"(s.kv_st), "s"(s.o_sb), "s"(s.o_sh), "s"(s.o_st), "s"(s.q_sb), "s"(s.q_sh), "s"(s.q_st), "s"(s.G), "s"(s.Hq), "s"(s.M), "s"(s.w_magic),
               "s"(s.c1), "s"(job.gamma), "s"(job.gamma_magic));
  const int b = divide(bh, s.hkv_magic), h = bh - b * s.Hkv, g = divide(layer, job.gamma_magic);
  SeqParam sp = job.seq[b];
  sp.k = job.k[g * s.B + b];
  const char *k_layer = (const char *)job.in[g * job.gamma][0], *q_layer = (const char *)in.q[g];
  const float *given = in.lse[g];
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::"s"(sp.L), "s"(sp.win), "s"(sp.p), "s"(sp.k), "s"(sp.win_magic), "s"(k_layer), "s"(q_layer), "s"(given));
  const int L = sp.L, n_review = L - s.w_obs;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), col = lane & 15, sub = lane >> 4;

  // ---- queries (past the last row: that row again) and keys of this wave -------------------------------------------------------
  auto swizzle = [](int r, int p) __attribute__((always_inline)) { return p ^ (PPR == 8 ? (r >> 1) & 7 : r & 15); };     // as in the score passes
  const char *qbase = q_layer + ((int64_t)b * s.q_sb + (int64_t)(h * s.G) * s.q_sh) * ES;
  constexpr int QN = (ROWS * PPR + NT - 1) / NT;                  // pieces of a thread
  u32x4 qv[QN];
#pragma unroll
  for (int i = 0; i < QN; ++i) {
    const int at = threadIdx.x + i * NT, r = min(at / PPR, s.M - 1), hq = (int)((uint32_t)r * s.w_magic >> 16), io = r - hq * s.w_obs;
    qv[i] = *(const u32x4 *)(qbase + ((int64_t)hq * s.q_sh + (int64_t)io * s.q_st) * ES + at % PPR * 16);
  }
  float given_lse = 0.0f;
  if (given && (int)threadIdx.x < s.M) given_lse = given[((int64_t)b * s.Hq + (int64_t)h * s.G) * s.w_obs + threadIdx.x];
  // A tile that reaches past the end has the last row again; one that lies past it is whatever LDS held, and counts for nothing.
  const char *kbase = k_layer + ((int64_t)b * s.kv_sb + (int64_t)h * s.kv_sh) * ES;
  constexpr int RPI = 64 / PPR, LPT = 16 / RPI;                   // rows per DMA instruction, instructions per tile
  bf16x8 kf[KT][KS];
#pragma unroll
  for (int k0 = 0; k0 < KT; k0 += KR) {
#pragma unroll
    for (int kt = k0; kt < KT && kt < k0 + KR; ++kt) {
      const int j0 = (kt * SHORT_WAVES + wave) * 16;
      if (j0 < L)                                                 // (uniform)
#pragma unroll
        for (int n = 0; n < LPT; ++n) {
          const int r = n * RPI + lane / PPR;
          dma_to_lds(lds_address(ring) + wave * RING + (kt - k0) * TILE + n * 1024,
                     kbase + (int64_t)min(j0 + r, L - 1) * s.kv_st * ES + swizzle(r, lane % PPR) * 16);
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
    for (int kt = k0; kt < KT && kt < k0 + KR; ++kt)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        kf[kt][ks] = *(const bf16x8 *)(ring + wave * RING + (kt - k0) * TILE + col * ROWB + swizzle(col, ks * 4 + sub) * 16);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < QN; ++i) {
    const int at = threadIdx.x + i * NT, r = at / PPR;
    if (ROWS * PPR % NT == 0 || at < ROWS * PPR) *(u32x4 *)(ring + r * ROWB + swizzle(r, at % PPR) * 16) = qv[i];
  }
  if (given && (int)threadIdx.x < ROWS) lse_s[threadIdx.x] = (int)threadIdx.x < s.M ? given_lse * 1.4426950408889634f : INFINITY;
  __syncthreads();

  // ---- logits: lane (col, sub) has keys tile * 16 + sub * 4 + e of row mt * 16 + col ------------------------------------------
  f32x4 acc[KT][RT];
#pragma unroll
  for (int mt = 0; mt < RT; ++mt) {
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) acc[kt][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const bf16x8 qf = *(const bf16x8 *)(ring + ((mt * 16 + col) * ROWB + swizzle(col, ks * 4 + sub) * 16));
#pragma unroll
      for (int kt = 0; kt < KT; ++kt)
        acc[kt][mt] = mfma_step<DT, 16>(kf[kt][ks], qf, acc[kt][mt]);
    }
  }

  // ---- statistics: the causal mask of the observation rows, then maximum and sum per row; the logits give way to their exponentials
  // with this wave's reference (handed-over normalisers are that reference).
  float ref[RT];                                                  // of row mt * 16 + col; -inf: no key of this wave counts for the row
#pragma unroll
  for (int mt = 0; mt < RT; ++mt) {
    const int r = min(mt * 16 + col, s.M - 1);
    const int last = n_review + r - (int)((uint32_t)r * s.w_magic >> 16) * s.w_obs;        // the last key that the row sees, < L
    float m = -INFINITY, z = 0.0f;
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
      const int j0 = (kt * SHORT_WAVES + wave) * 16;
      if (j0 + 16 > n_review)                                     // (uniform)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[kt][mt][e] = j0 + sub * 4 + e <= last ? acc[kt][mt][e] : -INFINITY;
      m = fmaxf(fmaxf(m, fmaxf(acc[kt][mt][0], acc[kt][mt][1])), fmaxf(acc[kt][mt][2], acc[kt][mt][3]));
    }
    ref[mt] = given ? lse_s[mt * 16 + col] : quads_max(m) * s.c1;
    const float from = !given && ref[mt] == -INFINITY ? 0.0f : ref[mt];
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[kt][mt][e] = fast_exp2(fmaf(acc[kt][mt][e], s.c1, -from));
      z += (acc[kt][mt][0] + acc[kt][mt][1]) + (acc[kt][mt][2] + acc[kt][mt][3]);
    }
    z = quads_sum(z);
    if (sub == 0) part_s[wave][mt * 16 + col] = make_float2(ref[mt], z);
  }
  if (!given) {
    __syncthreads();
    if ((int)threadIdx.x < ROWS) {
      float m = -INFINITY, z = 0.0f;
#pragma unroll
      for (int w = 0; w < SHORT_WAVES; ++w) {
        const float2 o = part_s[w][threadIdx.x];
        merge_stats(m, z, o.x, o.y);
      }
      lse_s[threadIdx.x] = (int)threadIdx.x < s.M ? m + fast_log2(z) : INFINITY;
    }
    __syncthreads();
  }

  // ---- token scores: from the wave's reference to the row's normaliser -------------------------------------------------------------
  float weight[RT];
#pragma unroll
  for (int mt = 0; mt < RT; ++mt) {
    weight[mt] = given ? 1.0f : fast_exp2(ref[mt] - lse_s[mt * 16 + col]);
  }
#pragma unroll
  for (int kt = 0; kt < KT; ++kt) {
    f32x4 t;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float x = 0.0f;
#pragma unroll
      for (int mt = 0; mt < RT; ++mt) x = fmaf(acc[kt][mt][e], weight[mt], x);
      t[e] = row16_sum(x);
    }
    if (col == 0) *(f32x4 *)&t_s[(kt * SHORT_WAVES + wave) * 16 + sub * 4] = t;
  }
  __syncthreads();

  // ---- windows, selection, rows -----------------------------------------------------------------------------------------------
  const int nw = divide(n_review + sp.win - 1, sp.win_magic);
  pool_windows<NT>(t_s, 0, nw, sp.win, sp.p, n_review, win_s);
  __syncthreads();
  const int64_t row = (int64_t)g * s.B * s.Hkv + bh;
  const bool writer = split == 0 && (int)blockIdx.z == 2 * g * job.gamma;       // this row's index outputs are this workgroup's
  int32_t *wrow = writer ? win_idx + row * s.k_max : nullptr;
  if (writer)
    for (int w = threadIdx.x; w < nw; w += NT) sc[row * s.nw_max + w] = win_s[w];
  const FirstScores<NT> first(win_s, nw);
  const int n_rev_kept = select_windows<NT>(sp, s.w_obs, win_s, first, keys, wrow);
  const TokenOf token(sp, s.w_obs, keys, n_rev_kept);
  copy_kept_rows<PPR, NT>(s, ES, b, h, token, split, gridDim.y, src, dst);
  if (writer) write_indices<NT>(s, sp.k, token, wrow, tok_idx + row * s.nkeep_max, n_keep + row);
}

hipError_t launch_short(const Shape &s, const BatchParams &bp, const GroupK &gk, const GroupPtrs &gp, const LayerPtrs &lp, int32_t n_groups, int32_t gamma,
                        float *sc, int32_t *win_idx, int32_t *tok_idx, int32_t *n_keep, hipStream_t stream) {
  const SmallJob job = small_job(s, bp, gk, lp, n_groups, gamma);
  ShortScore in;
  for (int g = 0; g < SMALL_GROUPS; ++g) {
    in.q[g] = g < n_groups ? gp.q[g] : nullptr;
    in.lse[g] = g < n_groups ? gp.lse[g] : nullptr;
  }
  const int pairs = 2 * n_groups * gamma * s.B * s.Hkv, rows = SHORT_THREADS / (int)(s.d * job.esize / 16);
  const int splits = max(min(SHORT_WORKGROUPS / pairs, (s.nkeep_max + rows - 1) / rows), 1);
  // (rows in x: all workgroups of a row on one XCD where the rows are a multiple of eight, so that its keys come into one L2)
  const dim3 grid(s.B * s.Hkv, splits, 2 * n_groups * gamma);
  const int tiles = short_row_tiles(s);
  // (four key tiles a wave where they are enough: what lies past the end is computed like the rest)
#define WKV_SHORT_KEYS(DD, TT, RR, KK) \
  if constexpr (short_key_tiles(DD, TT == DT_F32 ? 4 : 2, RR) >= KK) \
    if (s.d == DD && tiles == RR && s.t_stride + s.w_obs <= KK * 16 * SHORT_WAVES) { \
      hipLaunchKernelGGL((short_kernel<DD, TT, RR, KK>), grid, dim3(SHORT_THREADS), 0, stream, s, job, in, sc, win_idx, tok_idx, n_keep); \
      return hipGetLastError(); \
    }
#define WKV_SHORT(DD, TT, RR) WKV_SHORT_KEYS(DD, TT, RR, 4) WKV_SHORT_KEYS(DD, TT, RR, 8)
#define WKV_SHORT_ROWS(DD, TT) WKV_SHORT(DD, TT, 1) WKV_SHORT(DD, TT, 2) WKV_SHORT(DD, TT, 4) WKV_SHORT(DD, TT, 8)
  if (s.dtype == WKV_BF16) { WKV_SHORT_ROWS(64, DT_BF16) WKV_SHORT_ROWS(128, DT_BF16) }
  else if (s.dtype == WKV_F16) { WKV_SHORT_ROWS(64, DT_F16) WKV_SHORT_ROWS(128, DT_F16) }
  else { WKV_SHORT_ROWS(64, DT_F32) WKV_SHORT_ROWS(128, DT_F32) }
#undef WKV_SHORT_ROWS
#undef WKV_SHORT
#undef WKV_SHORT_KEYS
  return hipErrorInvalidValue;
}

}  // namespace wkv
