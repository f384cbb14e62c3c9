// Window pooling (WindowKV Eq. 3-4) and top-k window selection (Section 2.2.1).
//
// Both stages touch only the token-score array (4 bytes per prefix token and KV head), about
// 1/64 of the bytes of the key stream that produced it, so they are latency bound rather than
// bandwidth bound: the design goal is few launches and no serial host involvement.
#include "wkv_device.h"
#include "wkv_pool.h"

namespace wkv {

constexpr int POOL_THREADS = 256;
constexpr int POOL_TOKENS = SCORE_SEG;      // tokens a workgroup stages

__global__ __launch_bounds__(POOL_THREADS) void pool_kernel(Shape s, BatchParams bp, const float *__restrict__ t,
                                                                 float *__restrict__ s_out) {
  __shared__ __attribute__((aligned(16))) float t_s[POOL_TOKENS];
  // Three trips to memory: the arguments, the sequence's record, its tokens (which came one trip after the other before).
  asm volatile("" ::"s"(s.B), "s"(s.Hkv), "s"(s.hkv_magic), "s"(s.w_obs), "s"(s.t_stride), "s"(s.nw_max), "s"(t), "s"(s_out));
  const int bh = blockIdx.y, b = divide(bh, s.hkv_magic), g = blockIdx.z;
  const SeqParam sp = bp.seq[b];
  asm volatile("" ::"s"(sp.L), "s"(sp.win), "s"(sp.p), "s"(sp.win_magic));
  const int n_review = sp.L - s.w_obs;
  const int nw = divide(n_review + sp.win - 1, sp.win_magic);
  const int64_t row = (int64_t)g * s.B * s.Hkv + bh;
  const float *trow = t + row * s.t_stride;
  float *srow = s_out + row * s.nw_max;
  const int per = divide(POOL_TOKENS, sp.win_magic);        // windows that fit the staging area
  // sequences with small windows need fewer workgroups than the grid has per row; the last one fills up
  const int w0 = blockIdx.x * per, w1 = min(w0 + per, nw);
  if (w0 < w1) {
    const int tok0 = w0 * sp.win, n = min(w1 * sp.win, n_review) - tok0;
    float x[POOL_TOKENS / POOL_THREADS];                    // (requested together)
#pragma unroll
    for (int i = 0; i < POOL_TOKENS / POOL_THREADS; ++i) x[i] = trow[tok0 + min((int)threadIdx.x + i * POOL_THREADS, n - 1)];
#pragma unroll
    for (int i = 0; i < POOL_TOKENS / POOL_THREADS; ++i) t_s[threadIdx.x + i * POOL_THREADS] = x[i];
    __syncthreads();
    pool_windows<POOL_THREADS>(t_s, w0, w1, sp.win, sp.p, n_review, srow);
  }
  for (int w = max(w0, nw) + threadIdx.x; w < (blockIdx.x == gridDim.x - 1 ? s.nw_max : min(w0 + per, s.nw_max)); w += POOL_THREADS)
    srow[w] = -INFINITY;
}

hipError_t launch_pool(const Shape &s, const BatchParams &bp, int32_t n_groups, const float *t,
                       float *s_out, hipStream_t stream) {
  if (s.nw_max <= 0) return hipSuccess;
  int blocks = 1;
  for (int b = 0; b < s.B; ++b) {
    const int nw = (bp.seq[b].L - s.w_obs + bp.seq[b].win - 1) / bp.seq[b].win, per = POOL_TOKENS / bp.seq[b].win;
    blocks = max(blocks, (nw + per - 1) / per);
  }
  dim3 grid(blocks, s.B * s.Hkv, n_groups);
  hipLaunchKernelGGL(pool_kernel, grid, dim3(POOL_THREADS), 0, stream, s, bp, t, s_out);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// Top-k windows.  One workgroup per (group, sequence, KV head).  Bound by its chain of
// synchronised steps, not by data (a row is a few KB), so every step is one that needs few of them:
//   1. window scores -> order-preserving uint32 keys in LDS, their smallest and largest on the way
//   2. the k-th largest key T by digits of the range the keys really span: two bins per thread over [lo, hi],
//      descend into the bin that holds the k-th, until the windows that still fit are exactly a bin
//      or a bin is one key wide (9 to 11 bits a pass: at most four passes, two for ordinary scores.
//      Window scores differ in their low bits only, so digits taken from the top of the word put
//      nearly all of them into one bin and serialise the LDS counters)
//   3. window w is kept iff key > T, or key == T and fewer than take_eq equal windows precede it
//      (=> lower index wins ties).  Its output slot is (#greater before w) + min(#equal before w,
//      take_eq): ballots per wave and 1024 windows, one scan over all their counts, so the list comes
//      out ascending without a sort
//   4. expansion to token positions, the observation window appended, -1 padding
// The 32K-token configuration (64 rows of 2046 windows, k = 256): 12.2 us with 8-bit digits from the
// top and three synchronisations per 1024 windows in step 3, 9.2 us so; a mixed batch (512 rows of up to 3900
// windows): 19.7 us, 18.0 us so with 1024 threads, 13.8 us with 512.  With scans by DPP and a thread's scores requested
// together: 9.6 -> 8.0 us and 12.0 -> 10.2 us.  The arguments came in a chain of six trips to memory, each asked for where it was
// used, the scores in a seventh: with two, score, pool, selection and gather of 4096 tokens in fp32 one by one 56.7 -> 54.3 us (half of that the
// pooling's tokens, requested together), and merged with the gather (below) 512 tokens of two heads 16.3 -> 15.7, 4096 tokens 22.7 -> 22.05,
// 16384 tokens 42.2 -> 41.6.
// ------------------------------------------------------------------------------------------
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int TOPK_THREADS = 1024;
constexpr int SMALL_THREADS = 256;        // where 8192 windows are enough
constexpr int TOPK_WAVES = TOPK_THREADS / 64;
constexpr int TOPK_ITERS = WKV_MAX_WINDOWS / TOPK_THREADS;
static_assert(TOPK_ITERS <= 32, "one mask bit per window of a thread");

__device__ __forceinline__ uint32_t float_to_key(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// A thread's first scores of a row (past the row's room: the last one again), requested before its sequence is known.
constexpr int SCORES_AT_ONCE = 4;
template <int NT>
struct FirstScores {
  float x[SCORES_AT_ONCE];
  __device__ __forceinline__ FirstScores(const float *__restrict__ srow, int nw_max) {
#pragma unroll
    for (int i = 0; i < SCORES_AT_ONCE; ++i) x[i] = 0.0f;
    if (nw_max > 0)
#pragma unroll
      for (int i = 0; i < SCORES_AT_ONCE; ++i) x[i] = srow[min((int)threadIdx.x + i * NT, nw_max - 1)];
  }
};

// Steps 1-3 for the row of window scores srow: the selected windows, ascending, are left in keys (LDS, nw_max entries)
// and, if wrow is not null, written there.  Returns the number of review tokens they hold.
template <int NT>
__device__ __forceinline__ int select_windows(const SeqParam &sp, int w_obs, const float *__restrict__ srow, const FirstScores<NT> &first,
                                              uint32_t *keys, int32_t *__restrict__ wrow) {
  __shared__ uint32_t hist[2 * NT];
  __shared__ uint32_t wave_a[NT / 64], wave_b[NT / 64];
  __shared__ uint32_t counts[TOPK_ITERS * TOPK_WAVES];      // windows per wave and 1024: greater | equal << 16
  __shared__ uint32_t sh_bin, sh_above, sh_count;
  const int n_review = sp.L - w_obs;
  const int nw = divide(n_review + sp.win - 1, sp.win_magic);
  const int k = sp.k;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int n_rev_kept = 0;

  if (k > 0) {
    // ---- 1. keys and their range ------------------------------------------------------------
    uint32_t kmin = 0xffffffffu, kmax = 0u;
    constexpr int AT_ONCE = SCORES_AT_ONCE;
    float x[AT_ONCE];
#pragma unroll
    for (int i = 0; i < AT_ONCE; ++i) x[i] = first.x[i];
    for (int w0 = tid;;) {
#pragma unroll
      for (int i = 0; i < AT_ONCE; ++i) {
        const int w = w0 + i * NT;
        const bool in = w < nw;
        const uint32_t key = float_to_key(x[i]);
        if (in) keys[w] = key;
        kmin = min(kmin, in ? key : 0xffffffffu);
        kmax = max(kmax, in ? key : 0u);
      }
      w0 += AT_ONCE * NT;
      if (w0 >= nw) break;
#pragma unroll
      for (int i = 0; i < AT_ONCE; ++i) x[i] = srow[min(w0 + i * NT, nw - 1)];
    }
    kmin = ~wave_largest(~kmin);
    kmax = wave_largest(kmax);
    if (lane == 0) { wave_a[wave] = kmin; wave_b[wave] = kmax; }
    hist[tid] = 0u; hist[tid + NT] = 0u;
    __syncthreads();
    uint32_t lo = wave_a[0], hi = wave_b[0];
#pragma unroll
    for (int i = 1; i < NT / 64; ++i) { lo = min(lo, wave_a[i]); hi = max(hi, wave_b[i]); }

    // ---- 2. the k-th largest key ----------------------------------------------------------------
    uint32_t remaining = (uint32_t)k, take_eq, T;
    constexpr int digit_bits = NT == 1024 ? 11 : NT == 512 ? 10 : 9;
    static_assert(2 * NT == 1 << digit_bits, "two bins a thread");
    for (;;) {
      const int bits = 32 - __clz((int)((hi - lo) | 1u));
      const int shift = max(bits - digit_bits, 0);
      for (int w = tid; w < nw; w += NT) {
        const uint32_t key = keys[w];
        if (key >= lo && key <= hi) atomicAdd(&hist[(key - lo) >> shift], 1u);
      }
      __syncthreads();
      // windows in strictly higher bins: thread tid looks at the 2*tid-th and the next bin from the top
      const uint32_t c0 = hist[2 * NT - 1 - 2 * tid], c1 = hist[2 * NT - 2 - 2 * tid];
      const uint32_t incl = wave_sums(c0 + c1);
      if (lane == 63) wave_a[wave] = incl;
      __syncthreads();
      uint32_t above = incl - c0 - c1;
#pragma unroll
      for (int i = 0; i < NT / 64; ++i) above += i < wave ? wave_a[i] : 0u;
      if (above < remaining && above + c0 >= remaining) { sh_bin = 2 * NT - 1 - 2 * tid; sh_above = above; sh_count = c0; }
      above += c0;
      if (above < remaining && above + c1 >= remaining) { sh_bin = 2 * NT - 2 - 2 * tid; sh_above = above; sh_count = c1; }
      hist[2 * NT - 1 - 2 * tid] = 0u; hist[2 * NT - 2 - 2 * tid] = 0u;
      __syncthreads();
      const uint32_t bin_lo = lo + (sh_bin << shift);
      remaining -= sh_above;
      if (shift == 0) { T = bin_lo; take_eq = remaining; break; }              // one key wide: ties by index
      const uint32_t bin_hi = bin_lo + min((1u << shift) - 1u, hi - bin_lo);
      if (sh_count == remaining) {                      // the whole bin fits: everything from its lower edge on
        if (bin_lo != 0u) { T = bin_lo - 1u; take_eq = 0u; break; }
      }
      lo = bin_lo;
      hi = bin_hi;
    }

    // ---- 3. ordered compaction -------------------------------------------------------------
    uint32_t gt_bits = 0u, eq_bits = 0u;          // this thread's windows, one bit per 1024
    const int iters = (nw + NT - 1) / NT;
    for (int i = 0; i < iters; ++i) {
      const int w = i * NT + tid;
      const uint32_t key = w < nw ? keys[w] : 0u;
      const bool gt = w < nw && key > T, eq = w < nw && key == T;
      gt_bits |= (uint32_t)gt << i;
      eq_bits |= (uint32_t)eq << i;
      const int n_gt = __popcll(__ballot(gt)), n_eq = __popcll(__ballot(eq));
      if (lane == 0) counts[i * (NT / 64) + wave] = (uint32_t)n_gt | (uint32_t)n_eq << 16;
    }
    __syncthreads();                              // every key has been read: the array is free
    if (wave == 0) {                              // exclusive scan of the counts, in window order
      uint32_t base = 0u;
      for (int c = 0; c < iters * (NT / 64); c += 64) {
        const uint32_t v = c + lane < iters * (NT / 64) ? counts[c + lane] : 0u;
        const uint32_t incl = wave_sums(v);
        if (c + lane < iters * (NT / 64)) counts[c + lane] = base + incl - v;
        base += last_lane(incl);
      }
    }
    __syncthreads();
    const unsigned long long below = (1ull << lane) - 1ull;
    for (int i = 0; i < iters; ++i) {
      const bool gt = gt_bits >> i & 1u, eq = eq_bits >> i & 1u;
      const unsigned long long bgt = __ballot(gt), beq = __ballot(eq);
      const uint32_t before = counts[i * (NT / 64) + wave];
      const uint32_t gt_before = (before & 0xffffu) + __popcll(bgt & below), eq_before = (before >> 16) + __popcll(beq & below);
      if (gt || (eq && eq_before < take_eq)) {
        const uint32_t slot = gt_before + min(eq_before, take_eq);
        keys[slot] = (uint32_t)(i * NT + tid);
        if (wrow) wrow[slot] = i * NT + tid;
      }
    }
    __syncthreads();
    // Only the last window of the sequence can be partial, and if selected it is the last of
    // the ascending list, so slot m < k starts at m*win.
    n_rev_kept = k * sp.win;
    const int missing = ((int)keys[k - 1] + 1) * sp.win - n_review;
    if (missing > 0) n_rev_kept -= missing;
  }
  return n_rev_kept;
}

// Position of retained row r: row r - m*win of the m-th selected window, or of the observation window; -1 past the last.
struct TokenOf {
  const uint32_t *keys;                         // the selected windows
  int win, L, n_rev_kept, nk;
  uint32_t magic;
  __device__ __forceinline__ TokenOf(const SeqParam &sp, int w_obs, const uint32_t *sel, int kept)
      : keys(sel), win(sp.win), L(sp.L), n_rev_kept(kept), nk(kept + w_obs), magic(sp.win_magic) {}
  __device__ __forceinline__ int operator()(int r) const {
    if (r < n_rev_kept) {
      const int m = divide(r, magic);
      return (int)keys[m] * win + (r - m * win);
    }
    return r < nk ? L - nk + r : -1;
  }
};

template <int NT>
__global__ __launch_bounds__(NT) void topk_kernel(Shape s, BatchParams bp, GroupK gk,
                                                            const float *__restrict__ sc,
                                                            int32_t *__restrict__ win_idx,
                                                            int32_t *__restrict__ tok_idx,
                                                            int32_t *__restrict__ n_keep) {
  extern __shared__ uint32_t keys[];            // [nw_max], later reused for the selected list
  // Two trips to memory: the arguments; the sequence's record, the group's budget and the first scores.
  asm volatile("" ::"s"(s.B), "s"(s.Hkv), "s"(s.hkv_magic), "s"(s.w_obs), "s"(s.nw_max), "s"(s.k_max), "s"(s.nkeep_max), "s"(gk.in_use), "s"(sc),
               "s"(win_idx), "s"(tok_idx), "s"(n_keep));
  const int bh = blockIdx.x, b = divide(bh, s.hkv_magic), g = blockIdx.y;
  const int64_t row = (int64_t)g * s.B * s.Hkv + bh;
  const float *srow = sc + row * s.nw_max;
  const FirstScores<NT> first(srow, s.nw_max);
  SeqParam sp = bp.seq[b];
  const int own = g * s.B + b;                  // the group's own budget, if it has one: a half of a word, so that it is a scalar load
  const uint32_t two = gk.in_use ? ((const uint32_t *)gk.k)[own >> 1] : 0u;
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::"s"(sp.L), "s"(sp.win), "s"(sp.k), "s"(sp.win_magic), "s"(two));
  if (gk.in_use) sp.k = (int)(own & 1 ? two >> 16 : two & 0xffffu);
  int32_t *wrow = win_idx + row * s.k_max;
  const int n_rev_kept = select_windows<NT>(sp, s.w_obs, srow, first, keys, wrow);
  for (int i = sp.k + threadIdx.x; i < s.k_max; i += NT) wrow[i] = -1;
  const TokenOf token(sp, s.w_obs, keys, n_rev_kept);
  for (int r = threadIdx.x; r < s.nkeep_max; r += NT) tok_idx[row * s.nkeep_max + r] = token(r);
  if (threadIdx.x == 0) n_keep[row] = token.nk;
}

// Selection and gather in one launch, for calls with few (row, tensor) pairs: every workgroup selects the windows of its
// row for itself and copies its share of the kept rows of one layer's K or V.  The selection is a few
// microseconds of latency whether one workgroup of a row does it or all of them, and a launch less is worth
// more than that.  The pairs times `splits` fit the device at once; with more, the repeated selection would
// cost a round of its own.  A 4096-token group of four layers: 5.3 + 6.7 us apart, 9.5 us so with 256 threads (14 us
// with 1024: sixteen waves at every synchronisation); 16384 tokens: 5.7 + 14.9 us, 18.1 us so.  8.7 and 18.1 us with scans through
// LDS and a workgroup's rows copied four a lane at a time, 7.8 and 17.4 us with scans by DPP, the next rows requested before these are stored, and a
// pair's workgroups interleaved; six or eight rows a lane, 640 to 1024 workgroups: within 2 %, one shape's gain another's loss.
template <int LPR>  // 16-byte pieces per row
__global__ __launch_bounds__(SMALL_THREADS) void select_gather_kernel(Shape s, SmallJob job, const float *__restrict__ sc,
                                                                     int32_t *__restrict__ win_idx, int32_t *__restrict__ tok_idx,
                                                                     int32_t *__restrict__ n_keep) {
  extern __shared__ uint32_t keys[];
  constexpr int ROWS = SMALL_THREADS / LPR, AHEAD = 4;
  // Two trips to memory: the arguments; the sequence's record, its budget and the first scores.
  const int split = blockIdx.x, bh = blockIdx.y, layer = blockIdx.z >> 1, is_v = blockIdx.z & 1;
  const char *src = (const char *)job.in[layer][is_v];
  char *dst = (char *)job.out[layer][is_v];
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::"s"(src), "s"(dst), "s"(s.B), "s"(s.Hkv), "s"(s.hkv_magic), "s"(s.w_obs), "s"(s.nw_max), "s"(s.k_max), "s"(s.nkeep_max), "s"(s.fill_padding),
               "s"(s.kv_sb), "s"(s.kv_sh), "s"(s.kv_st), "s"(s.o_sb), "s"(s.o_sh), "s"(s.o_st), "s"(job.gamma), "s"(job.gamma_magic), "s"(job.esize),
               "s"(sc), "s"(win_idx), "s"(tok_idx), "s"(n_keep));
  const int b = divide(bh, s.hkv_magic), h = bh - b * s.Hkv, g = divide(layer, job.gamma_magic);
  const int64_t row = (int64_t)g * s.B * s.Hkv + bh;
  const float *srow = sc + row * s.nw_max;
  const FirstScores<SMALL_THREADS> first(srow, s.nw_max);
  SeqParam sp = job.seq[b];
  sp.k = job.k[g * s.B + b];
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::"s"(sp.L), "s"(sp.win), "s"(sp.k), "s"(sp.win_magic));
  const bool writer = split == 0 && blockIdx.z == 2 * g * job.gamma;       // this row's index outputs are this workgroup's
  int32_t *wrow = writer ? win_idx + row * s.k_max : nullptr;
  const int n_rev_kept = select_windows<SMALL_THREADS>(sp, s.w_obs, srow, first, keys, wrow);
  const TokenOf token(sp, s.w_obs, keys, n_rev_kept);
  const int nk = token.nk, n_write = s.fill_padding ? s.nkeep_max : nk;

  const int piece = threadIdx.x % LPR;
  src += ((int64_t)b * s.kv_sb + (int64_t)h * s.kv_sh) * job.esize + piece * 16;
  dst += ((int64_t)b * s.o_sb + (int64_t)h * s.o_sh) * job.esize + piece * 16;
  const int64_t in_step = s.kv_st * job.esize, out_step = s.o_st * job.esize;
  // rows ROWS * gridDim.x apart: the workgroups of a pair write one dense stretch; the next AHEAD rows are requested before these are stored
  const int step = ROWS * (int)gridDim.x;
  int r0 = split * ROWS + threadIdx.x / LPR;
  u32x4 v[AHEAD];
  auto request = [&](int r0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) {
      const int r = r0 + u * step;
      v[u] = u32x4{0u, 0u, 0u, 0u};
      if (r < nk) v[u] = __builtin_nontemporal_load((const u32x4 *)(src + (int64_t)token(r) * in_step));
    }
  };
  request(r0);
  for (; r0 < n_write; r0 += step * AHEAD) {
    u32x4 out[AHEAD];
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) out[u] = v[u];
    request(r0 + step * AHEAD);
#pragma unroll
    for (int u = 0; u < AHEAD; ++u)
      if (r0 + u * step < n_write) __builtin_nontemporal_store(out[u], (u32x4 *)(dst + (int64_t)(r0 + u * step) * out_step));
  }
  if (!writer) return;
  for (int i = sp.k + threadIdx.x; i < s.k_max; i += SMALL_THREADS) wrow[i] = -1;
  for (int r = threadIdx.x; r < s.nkeep_max; r += SMALL_THREADS) tok_idx[row * s.nkeep_max + r] = token(r);
  if (threadIdx.x == 0) n_keep[row] = nk;
}

hipError_t launch_select_gather(const Shape &s, const BatchParams &bp, const GroupK &gk, const LayerPtrs &lp, int32_t n_groups, int32_t gamma,
                                const float *sc, int32_t *win_idx, int32_t *tok_idx, int32_t *n_keep, hipStream_t stream) {
  SmallJob job;
  job.gamma = gamma;
  job.gamma_magic = division_magic(gamma);
  job.esize = (int32_t)elem_bytes(s.dtype);
  for (int b = 0; b < s.B; ++b) job.seq[b] = bp.seq[b];
  for (int i = 0; i < n_groups * s.B; ++i) job.k[i] = gk.in_use ? gk.k[i] : bp.seq[i % s.B].k;
  for (int l = 0; l < n_groups * gamma; ++l) {
    job.in[l][0] = lp.k_in[l]; job.in[l][1] = lp.v_in[l];
    job.out[l][0] = lp.k_out[l]; job.out[l][1] = lp.v_out[l];
  }
  const int pairs = 2 * n_groups * gamma * s.B * s.Hkv;
  const int lpr = (int)(s.d * job.esize / 16), rows = SMALL_THREADS / lpr;
  const int splits = max(min(SMALL_WORKGROUPS / pairs, (s.nkeep_max + rows - 1) / rows), 1);
  dim3 grid(splits, s.B * s.Hkv, 2 * n_groups * gamma);
  const size_t lds = (size_t)(s.nw_max > 0 ? s.nw_max : 1) * sizeof(uint32_t);
  if (lpr == 8) hipLaunchKernelGGL(select_gather_kernel<8>, grid, dim3(SMALL_THREADS), lds, stream, s, job, sc, win_idx, tok_idx, n_keep);
  else if (lpr == 16) hipLaunchKernelGGL(select_gather_kernel<16>, grid, dim3(SMALL_THREADS), lds, stream, s, job, sc, win_idx, tok_idx, n_keep);
  else hipLaunchKernelGGL(select_gather_kernel<32>, grid, dim3(SMALL_THREADS), lds, stream, s, job, sc, win_idx, tok_idx, n_keep);
  return hipGetLastError();
}

hipError_t launch_topk(const Shape &s, const BatchParams &bp, const GroupK &gk, int32_t n_groups, const float *sc,
                       int32_t *win_idx, int32_t *tok_idx, int32_t *n_keep, hipStream_t stream) {
  const size_t lds = (size_t)(s.nw_max > 0 ? s.nw_max : 1) * sizeof(uint32_t);
  if (lds > 48 * 1024) {     // beyond the default dynamic-LDS limit: raise it (per device, any thread)
    hipError_t e = hipFuncSetAttribute((const void *)topk_kernel<TOPK_THREADS>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       WKV_MAX_WINDOWS * (int)sizeof(uint32_t));
    if (e != hipSuccess) return e;
  }
  dim3 grid(s.B * s.Hkv, n_groups);
  // Half the threads where a thread still has few windows: cheaper synchronisation, and more rows on a compute unit.
  if (s.nw_max <= 4096)
    hipLaunchKernelGGL(topk_kernel<TOPK_THREADS / 2>, grid, dim3(TOPK_THREADS / 2), lds, stream, s, bp, gk, sc, win_idx, tok_idx, n_keep);
  else
    hipLaunchKernelGGL(topk_kernel<TOPK_THREADS>, grid, dim3(TOPK_THREADS), lds, stream, s, bp, gk, sc, win_idx, tok_idx, n_keep);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// Jaccard similarity of the retained positions of every pair of index sets (Section 3.2).
// One workgroup per (set i, set j, sequence, KV head): both rows are ascending, so each thread
// looks its elements of row i up in row j by binary search; |A u B| = |A| + |B| - |A n B|.
// ------------------------------------------------------------------------------------------
constexpr int JAC_THREADS = 256;

__global__ __launch_bounds__(JAC_THREADS) void jaccard_kernel(Shape s, int32_t n_sets, const int32_t *__restrict__ tok_idx,
                                                              const int32_t *__restrict__ n_keep,
                                                              float *__restrict__ out) {
  __shared__ int wave_hits[JAC_THREADS / 64];
  const int bh = blockIdx.x, i = blockIdx.y, j = blockIdx.z;
  const int64_t rows = (int64_t)s.B * s.Hkv;
  const int32_t *a = tok_idx + ((int64_t)i * rows + bh) * s.nkeep_max;
  const int32_t *b = tok_idx + ((int64_t)j * rows + bh) * s.nkeep_max;
  const int na = min(max(n_keep[(int64_t)i * rows + bh], 0), s.nkeep_max);
  const int nb = min(max(n_keep[(int64_t)j * rows + bh], 0), s.nkeep_max);
  int hits = 0;
  for (int k = threadIdx.x; k < na; k += JAC_THREADS) {
    const int32_t x = a[k];
    int lo = 0, hi = nb;                       // first position of row j not below x
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (b[mid] < x) lo = mid + 1; else hi = mid;
    }
    hits += lo < nb && b[lo] == x;
  }
  for (int off = 32; off > 0; off >>= 1) hits += __shfl_xor(hits, off);
  if ((threadIdx.x & 63) == 0) wave_hits[threadIdx.x >> 6] = hits;
  __syncthreads();
  if (threadIdx.x == 0) {
    int inter = 0;
    for (int w = 0; w < JAC_THREADS / 64; ++w) inter += wave_hits[w];
    const int uni = na + nb - inter;
    out[((int64_t)i * n_sets + j) * rows + bh] = uni == 0 ? 1.0f : (float)inter / (float)uni;
  }
}

hipError_t launch_jaccard(const Shape &s, int32_t n_sets, const int32_t *tok_idx, const int32_t *n_keep, float *out,
                          hipStream_t stream) {
  dim3 grid(s.B * s.Hkv, n_sets, n_sets);
  hipLaunchKernelGGL(jaccard_kernel, grid, dim3(JAC_THREADS), 0, stream, s, n_sets, tok_idx, n_keep, out);
  return hipGetLastError();
}

}  // namespace wkv
