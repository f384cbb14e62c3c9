// Shared-index row gather (WindowKV Section 2.2.2): every layer of a group keeps the K and V
// rows at the group's retained positions.  A pure copy, bound by HBM bandwidth.
//
// Mapping: a row of head_dim elements is 128, 256 or 512 bytes; `LPR` lanes (16 B each) cover one
// row, so a wave moves 1 KB per load instruction.  A workgroup is one wave with GATHER_UNROLL such
// pieces in flight, GATHER_APART pieces apart, so that the workgroups that run side by side write one dense stretch of
// a tensor.  grid.x walks the row blocks of the compact cache, grid.y the (sequence, KV head) pairs, grid.z the
// (layer, K|V) tensors.  Selected rows come in runs of `win` consecutive tokens, i.e. 2-32 KB contiguous reads.
//
// The memory takes a copy best when what is written at a time lies close together: copies of 512 MB by waves or
// workgroups that take the next 1 to 4 KB 6.4-6.6 TB/s, by workgroups with two pieces of 4 KB one after the other 5.9, by long-lived
// workgroups with a share each 5.2-5.7, however much they keep in flight; 6.4 with rows in runs of 4 KB picked from eight
// times as much.  Gather alone, batch of mixed lengths (6.4 GB with the rows past n_keep) / 32K-token model (1.1 GB):
// workgroups of 256 threads with two adjacent pieces 1134-1144 / 175-176 us, waves with two pieces 1, 4, 8, 16 or 32 KB apart
// 1105, 1106, 1073, 1086, 1080 / 178, 176, 174-176, 174, 175, with one piece 1126 / 178, with three or four slower, K and V of a
// row by one wave 1068 / 178, pipelined loops over 4 to 32 pieces up to 8 % slower.
#include "wkv_internal.h"

namespace wkv {

constexpr int GATHER_THREADS = 64;
constexpr int GATHER_UNROLL = 2;
constexpr int GATHER_APART = 8;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// What the kernel needs of a Shape; strides in bytes.
struct GatherShape {
  int32_t Hkv, rows;                             // KV heads; sequences times KV heads
  int32_t nkeep_max, fill_padding, max_tok;      // max_tok: token capacity of the full cache
  uint32_t kv_magic, gamma_magic;                // division_magic of Hkv and of the layers per group
  int64_t in_b, in_h, in_t, out_b, out_h, out_t;
};

template <int LPR>  // lanes per row
__global__ __launch_bounds__(GATHER_THREADS) void gather_kernel(GatherShape s, LayerPtrs lp, const int32_t *__restrict__ tok_idx,
                                                                const int32_t *__restrict__ n_keep) {
  constexpr int ROWS = GATHER_THREADS / LPR;     // of a piece
  const int bh = blockIdx.y, b = divide(bh, s.kv_magic), h = bh - b * s.Hkv;
  const int layer = blockIdx.z >> 1;
  const bool is_v = blockIdx.z & 1;
  const int row = divide(layer, s.gamma_magic) * s.rows + bh;          // of the index arrays
  const int32_t *idx = tok_idx + (int64_t)row * s.nkeep_max;
  const int first = ((int)blockIdx.x / GATHER_APART * (GATHER_APART * GATHER_UNROLL) + (int)blockIdx.x % GATHER_APART) * ROWS;
  const int r0 = first + threadIdx.x / LPR;

  // (requested together with n_keep, which tells whether they count)
  int tok[GATHER_UNROLL];
#pragma unroll
  for (int u = 0; u < GATHER_UNROLL; ++u) tok[u] = idx[min(r0 + u * (GATHER_APART * ROWS), s.nkeep_max - 1)];
  const int nk = min(n_keep[row], s.nkeep_max);
  const int n_write = s.fill_padding ? s.nkeep_max : nk;   // rows past n_keep: zero-filled or left alone
  if (first >= n_write) return;
  const char *src = (const char *)(is_v ? lp.v_in[layer] : lp.k_in[layer]) + b * s.in_b + h * s.in_h + threadIdx.x % LPR * 16;
  char *dst = (char *)(is_v ? lp.v_out[layer] : lp.k_out[layer]) + b * s.out_b + h * s.out_h + threadIdx.x % LPR * 16;
  u32x4 v[GATHER_UNROLL];
#pragma unroll
  for (int u = 0; u < GATHER_UNROLL; ++u) {
    v[u] = u32x4{0u, 0u, 0u, 0u};
    // indices are caller data: never read out of bounds
    if (r0 + u * (GATHER_APART * ROWS) < nk && tok[u] >= 0 && tok[u] < s.max_tok)
      v[u] = __builtin_nontemporal_load((const u32x4 *)(src + (int64_t)tok[u] * s.in_t));
  }
#pragma unroll
  for (int u = 0; u < GATHER_UNROLL; ++u)
    if (r0 + u * (GATHER_APART * ROWS) < n_write)
      __builtin_nontemporal_store(v[u], (u32x4 *)(dst + (int64_t)(r0 + u * (GATHER_APART * ROWS)) * s.out_t));
}

hipError_t launch_gather(const Shape &s, const LayerPtrs &lp, int32_t n_layers, int32_t gamma,
                         const int32_t *tok_idx, const int32_t *n_keep, hipStream_t stream) {
  if (s.nkeep_max <= 0) return hipSuccess;
  const int64_t esize = elem_bytes(s.dtype);
  const GatherShape gs = {s.Hkv, s.B * s.Hkv, s.nkeep_max, s.fill_padding, s.t_stride + s.w_obs, division_magic(s.Hkv), division_magic(gamma),
                          s.kv_sb * esize, s.kv_sh * esize, s.kv_st * esize, s.o_sb * esize, s.o_sh * esize, s.o_st * esize};
  const int lpr = (int)(s.d * esize / 16);   // 8 (bf16 d=64), 16, 16, or 32 (f32 d=128)
  const int rows = GATHER_THREADS / lpr * GATHER_APART * GATHER_UNROLL;          // of GATHER_APART workgroups
  dim3 grid((s.nkeep_max + rows - 1) / rows * GATHER_APART, s.B * s.Hkv, n_layers * 2);
  dim3 block(GATHER_THREADS);
  switch (lpr) {
    case 8:  hipLaunchKernelGGL(gather_kernel<8>, grid, block, 0, stream, gs, lp, tok_idx, n_keep); break;
    case 16: hipLaunchKernelGGL(gather_kernel<16>, grid, block, 0, stream, gs, lp, tok_idx, n_keep); break;
    case 32: hipLaunchKernelGGL(gather_kernel<32>, grid, block, 0, stream, gs, lp, tok_idx, n_keep); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace wkv
