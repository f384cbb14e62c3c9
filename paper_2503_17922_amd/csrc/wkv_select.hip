// Window pooling (WindowKV Eq. 3-4) and top-k window selection (Section 2.2.1).
//
// Both stages touch only the token-score array (4 bytes per prefix token and KV head), about
// 1/64 of the bytes of the key stream that produced it, so they are latency bound rather than
// bandwidth bound: the design goal is few launches and no serial host involvement.
#include "wkv_device.h"
#include "wkv_pool.h"
#include "wkv_select.h"

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
// Top-k windows (the steps are in wkv_select.h).  One workgroup per (group, sequence, KV head).
// ------------------------------------------------------------------------------------------
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
  write_indices<NT>(s, sp.k, TokenOf(sp, s.w_obs, keys, n_rev_kept), wrow, tok_idx + row * s.nkeep_max, n_keep + row);
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
  copy_kept_rows<LPR, SMALL_THREADS>(s, job.esize, b, h, token, split, gridDim.x, src, dst);
  if (writer) write_indices<SMALL_THREADS>(s, sp.k, token, wrow, tok_idx + row * s.nkeep_max, n_keep + row);
}

hipError_t launch_select_gather(const Shape &s, const BatchParams &bp, const GroupK &gk, const LayerPtrs &lp, int32_t n_groups, int32_t gamma,
                                const float *sc, int32_t *win_idx, int32_t *tok_idx, int32_t *n_keep, hipStream_t stream) {
  const SmallJob job = small_job(s, bp, gk, lp, n_groups, gamma);
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
