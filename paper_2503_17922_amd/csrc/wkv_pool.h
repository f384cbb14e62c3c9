// Window pooling (WindowKV Eq. 3-4): s_w = sum(Top-p(W_w)) / min(p, win).  Shared by the pooling kernel
// and the score kernels' epilogues, so that all of them give the same bits.
#pragma once

#include "wkv_internal.h"

namespace wkv {

// One window of at most W tokens by one thread, in registers: the tokens (float4 loads where the window's
// size and address allow) are put in descending order by a fully unrolled bitonic network (min/max
// pairs, nothing indexed dynamically) and the first p are summed.  Which of several equal values
// counts as "in the top p" does not change that sum.
template <int W>
__device__ __forceinline__ float pool_window_regs(const float *__restrict__ trow, int w, int win, int n_review, int p) {
  float v[W];
  const int tok0 = w * win;
  const int size = min(win, n_review - tok0);
  if (size == win && (win & 3) == 0 && ((uintptr_t)(trow + tok0) & 15) == 0) {
#pragma unroll
    for (int i = 0; i < W; i += 4) {
      const float4 q = i < win ? *(const float4 *)(trow + tok0 + i) : make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
      v[i] = q.x; v[i + 1] = q.y; v[i + 2] = q.z; v[i + 3] = q.w;
    }
  } else {
#pragma unroll
    for (int i = 0; i < W; ++i) v[i] = i < size ? trow[tok0 + i] : -INFINITY;
  }
  float acc = 0.0f;
  if (p >= size) {
#pragma unroll
    for (int i = 0; i < W; ++i) acc += i < size ? v[i] : 0.0f;
  } else {
#pragma unroll
    for (int k = 2; k <= W; k <<= 1)
#pragma unroll
      for (int j = k >> 1; j > 0; j >>= 1)
#pragma unroll
        for (int i = 0; i < W; ++i) {
          const int l = i ^ j;
          if (l > i) {
            const float lo = fminf(v[i], v[l]), hi = fmaxf(v[i], v[l]);
            const bool descending = (i & k) == 0;
            v[i] = descending ? hi : lo;
            v[l] = descending ? lo : hi;
          }
        }
#pragma unroll
    for (int i = 0; i < W; ++i) acc += i < p ? v[i] : 0.0f;     // p < size: none of these is padding
  }
  return acc / (float)p;
}

// Windows w0 .. w1-1 of one sequence by a workgroup of NT threads, on the token scores in LDS (t_s[i] is
// token w0*win + i, 16-byte aligned, complete before the call: the caller synchronises).  Up to 64 tokens a
// window is one thread's; larger windows would not fit its registers, so there every token counts how
// many of its window come before it (larger, or equal at a lower position), the ones past the p-th are
// cleared, and a thread per window adds up what is left.
template <int NT>
__device__ __forceinline__ void pool_windows(float *t_s, int w0, int w1, int win, int p, int n_review, float *__restrict__ srow) {
  const float *trow = t_s - w0 * win;
  if (win <= 8) {
    for (int w = w0 + threadIdx.x; w < w1; w += NT) srow[w] = pool_window_regs<8>(trow, w, win, n_review, p);
  } else if (win <= 16) {
    for (int w = w0 + threadIdx.x; w < w1; w += NT) srow[w] = pool_window_regs<16>(trow, w, win, n_review, p);
  } else if (win <= 32) {
    for (int w = w0 + threadIdx.x; w < w1; w += NT) srow[w] = pool_window_regs<32>(trow, w, win, n_review, p);
  } else if (win <= 64) {
    for (int w = w0 + threadIdx.x; w < w1; w += NT) srow[w] = pool_window_regs<64>(trow, w, win, n_review, p);
  } else {
    const int n = min(w1 * win, n_review) - w0 * win;
    if (p < win) {
      uint32_t drop = 0u;                              // one bit per token of this thread: at most 32 (see the assert)
      static_assert(SCORE_SEG <= 32 * NT, "tokens per thread");
      for (int e = threadIdx.x, i = 0; e < n; e += NT, ++i) {
        const int first = e / win * win, last = min(first + win, n);
        const float v = t_s[e];
        int rank = 0;
        for (int j = first; j < last; ++j) rank += t_s[j] > v || (t_s[j] == v && j < e);
        drop |= (uint32_t)(rank >= p) << i;
      }
      __syncthreads();
      for (int e = threadIdx.x, i = 0; e < n; e += NT, ++i)
        if (drop >> i & 1u) t_s[e] = 0.0f;
      __syncthreads();
    }
    for (int w = w0 + threadIdx.x; w < w1; w += NT) {
      const int first = (w - w0) * win, last = min(first + win, n);
      float acc = 0.0f;
      for (int j = first; j < last; ++j) acc += t_s[j];
      srow[w] = acc / (float)p;
    }
  }
}

}  // namespace wkv
