// Selection of windows and what follows from it (WindowKV Section 2.2.1 and 2.2.2), shared by the top-k kernel and the ones that also
// copy the kept rows.
#pragma once

#include "wkv_device.h"

namespace wkv {

// ------------------------------------------------------------------------------------------
// Top-k windows by one workgroup.  Bound by its chain of
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
// 16384 tokens 42.2 -> 41.6.  A thread's first keys in registers, up to 64 counts scanned by every wave for itself: 21.1 -> 20.75 and 39.0 -> 38.6.
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
    uint32_t own[AT_ONCE];                        // the thread's first windows' stay with it, the others' go to LDS
#pragma unroll
    for (int i = 0; i < AT_ONCE; ++i) {
      const bool in = tid + i * NT < nw;
      own[i] = float_to_key(first.x[i]);
      kmin = min(kmin, in ? own[i] : 0xffffffffu);
      kmax = max(kmax, in ? own[i] : 0u);
    }
    for (int w0 = tid + AT_ONCE * NT; w0 < nw; w0 += AT_ONCE * NT) {
      float x[AT_ONCE];
#pragma unroll
      for (int i = 0; i < AT_ONCE; ++i) x[i] = srow[min(w0 + i * NT, nw - 1)];
#pragma unroll
      for (int i = 0; i < AT_ONCE; ++i) {         // (past the end: the last one's key again, written nowhere)
        const uint32_t key = float_to_key(x[i]);
        if (w0 + i * NT < nw) keys[w0 + i * NT] = key;
        kmin = min(kmin, key);
        kmax = max(kmax, key);
      }
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
#pragma unroll
      for (int i = 0; i < AT_ONCE; ++i)
        if (tid + i * NT < nw && own[i] >= lo && own[i] <= hi) atomicAdd(&hist[(own[i] - lo) >> shift], 1u);
      for (int w = tid + AT_ONCE * NT; w < nw; w += NT) {
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
    auto classify = [&](int i, bool in, uint32_t key) __attribute__((always_inline)) {
      const bool gt = in && key > T, eq = in && key == T;
      gt_bits |= (uint32_t)gt << i;
      eq_bits |= (uint32_t)eq << i;
      const int n_gt = __popcll(__ballot(gt)), n_eq = __popcll(__ballot(eq));
      if (lane == 0) counts[i * (NT / 64) + wave] = (uint32_t)n_gt | (uint32_t)n_eq << 16;
    };
#pragma unroll
    for (int i = 0; i < AT_ONCE; ++i)
      if (i * NT < nw) classify(i, tid + i * NT < nw, own[i]);
    for (int i = AT_ONCE; i < iters; ++i) {
      const int w = i * NT + tid;
      classify(i, w < nw, w < nw ? keys[w] : 0u);
    }
    __syncthreads();                              // every key has been read: the array is free
    // exclusive scan of the counts, in window order: up to 64 by every wave for itself, else by the first one
    const int n_counts = iters * (NT / 64);
    uint32_t mine = 0u;
    if (n_counts <= 64) {
      const uint32_t v = lane < n_counts ? counts[lane] : 0u;
      mine = wave_sums(v) - v;
    } else {
      if (wave == 0) {
        uint32_t base = 0u;
        for (int c = 0; c < n_counts; c += 64) {
          const uint32_t v = c + lane < n_counts ? counts[c + lane] : 0u;
          const uint32_t incl = wave_sums(v);
          if (c + lane < n_counts) counts[c + lane] = base + incl - v;
          base += last_lane(incl);
        }
      }
      __syncthreads();
    }
    const unsigned long long below = (1ull << lane) - 1ull;
    for (int i = 0; i < iters; ++i) {
      const bool gt = gt_bits >> i & 1u, eq = eq_bits >> i & 1u;
      const unsigned long long bgt = __ballot(gt), beq = __ballot(eq);
      const int at = i * (NT / 64) + wave;
      const uint32_t before = n_counts <= 64 ? (uint32_t)__builtin_amdgcn_readlane((int)mine, __builtin_amdgcn_readfirstlane(at)) : counts[at];
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

// The index outputs of a row.
template <int NT>
__device__ __forceinline__ void write_indices(const Shape &s, int k, const TokenOf &token, int32_t *__restrict__ wrow, int32_t *__restrict__ trow,
                                              int32_t *__restrict__ n_keep) {
  for (int i = k + threadIdx.x; i < s.k_max; i += NT) wrow[i] = -1;
  for (int r = threadIdx.x; r < s.nkeep_max; r += NT) trow[r] = token(r);
  if (threadIdx.x == 0) *n_keep = token.nk;
}

// This workgroup's share (one of n_splits) of the kept rows of one tensor, LPR lanes of 16 bytes per row.
template <int LPR, int NT>
__device__ __forceinline__ void copy_kept_rows(const Shape &s, int64_t esize, int b, int h, const TokenOf &token, int split, int n_splits, const char *src,
                                               char *dst) {
  constexpr int ROWS = NT / LPR, AHEAD = 4;
  const int n_write = s.fill_padding ? s.nkeep_max : token.nk;
  const int piece = threadIdx.x % LPR;
  src += ((int64_t)b * s.kv_sb + (int64_t)h * s.kv_sh) * esize + piece * 16;
  dst += ((int64_t)b * s.o_sb + (int64_t)h * s.o_sh) * esize + piece * 16;
  const int64_t in_step = s.kv_st * esize, out_step = s.o_st * esize;
  // rows ROWS * gridDim.x apart: the workgroups of a pair write one dense stretch; the next AHEAD rows are requested before these are stored
  const int step = ROWS * n_splits;
  int r0 = split * ROWS + threadIdx.x / LPR;
  u32x4 v[AHEAD];
  auto request = [&](int r0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) {
      const int r = r0 + u * step;
      v[u] = u32x4{0u, 0u, 0u, 0u};
      if (r < token.nk) v[u] = __builtin_nontemporal_load((const u32x4 *)(src + (int64_t)token(r) * in_step));
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
}

}  // namespace wkv
