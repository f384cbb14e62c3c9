// Shared-index row gather (WindowKV Section 2.2.2): every layer of a group keeps the K and V
// rows at the group's retained positions.  A pure copy, bound by HBM bandwidth.
//
// Mapping: a row of head_dim elements is 128, 256 or 512 bytes; `LPR` lanes (16 B each) cover one
// row, so a wave moves 1 KB per load instruction.  A workgroup of NT threads has GATHER_UNROLL such
// pieces in flight, APART pieces apart, so that the workgroups that run side by side write one dense stretch of
// a tensor.  grid.x walks the row blocks of the compact cache, grid.y the (sequence, KV head) pairs, grid.z the
// (layer, K|V) tensors.  Selected rows come in runs of `win` consecutive tokens, i.e. 2-32 KB contiguous reads.
//
// The memory takes a copy best when what is written at a time lies close together: copies of 512 MB by waves or
// workgroups that take the next 1 to 4 KB 6.4-6.6 TB/s, by workgroups with two pieces of 4 KB one after the other 5.9, by long-lived
// workgroups with a share each 5.2-5.7, however much they keep in flight; 6.4 with rows in runs of 4 KB picked from eight
// times as much.  Gather alone, batch of mixed lengths (6.4 GB with the rows past n_keep) / 32K-token model (1.1 GB):
// workgroups of 256 threads with two adjacent pieces 1137 / 177 us, of one wave with two pieces 1, 8 or 16 KB apart 1095, 1020, 1070 /
// 175, 173-176, 175, with one piece 1126 / 178, with three or four slower, K and V of a row by one wave 1068 / 178, pipelined loops
// over 4 to 32 pieces up to 8 % slower.
//
// The chip starts at most 1.9 workgroups a nanosecond (8 XCDs, one in 10 cycles each), which with single waves is just what the copy needs:
// every workgroup without rows costs as much as one with 2 KB.  Hence the grid ends with the last row (APART is smaller at the
// end of a tensor's rows; rounded up to whole stretches of 64 rows, 130 rows a KV head took 1.02-1.20 times as long as by 256
// threads, 0.97 so), and batches of very different lengths take larger workgroups (gather_threads).
#include "wkv_internal.h"

namespace wkv {

constexpr int GATHER_UNROLL = 2;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// What the kernel needs of a Shape; strides in bytes.
struct GatherShape {
  int32_t Hkv, rows;                             // KV heads; sequences times KV heads
  int32_t nkeep_max, fill_padding, max_tok;      // max_tok: token capacity of the full cache
  int32_t last, last_apart;                      // the workgroups from this one on have their pieces so far apart
  uint32_t kv_magic, gamma_magic;                // division_magic of Hkv and of the layers per group
  int64_t in_b, in_h, in_t, out_b, out_h, out_t;
};

template <int LPR, int NT, int APART>  // lanes per row, threads, pieces from one to the next
__global__ __launch_bounds__(NT) void gather_kernel(GatherShape s, LayerPtrs lp, const int32_t *__restrict__ tok_idx,
                                                    const int32_t *__restrict__ n_keep) {
  constexpr int ROWS = NT / LPR;                 // of a piece
  // Three trips to memory: the arguments, the positions with their count, the rows.  The barriers keep what is requested together
  // together; by itself the compiler asked for n_keep, then for the positions, then for the tensors' addresses, and for the second row when the
  // first had come: group by group, 32K-token model 198 -> 194 us, batch of mixed lengths 1113 -> 1071, 16K with 64 query heads 139 -> 133.5 (one piece
  // a wave 200, 1183 and 141.5, three 198, 1110 and 140.5, four 207, 1143 and 147; 16 pieces apart the same as 8).
  const int layer = blockIdx.z >> 1;
  const bool is_v = blockIdx.z & 1;
  const void *const *in = is_v ? lp.v_in : lp.k_in;
  void *const *out = is_v ? lp.v_out : lp.k_out;
  const char *src = (const char *)in[layer];
  char *dst = (char *)out[layer];
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::"s"(src), "s"(dst), "s"(tok_idx), "s"(n_keep), "s"(s.kv_magic), "s"(s.Hkv), "s"(s.gamma_magic), "s"(s.rows), "s"(s.nkeep_max),
               "s"(s.fill_padding), "s"(s.max_tok), "s"(s.last), "s"(s.last_apart), "s"(s.in_b), "s"(s.in_h), "s"(s.in_t), "s"(s.out_b), "s"(s.out_h), "s"(s.out_t));
  const int bh = blockIdx.y, b = divide(bh, s.kv_magic), h = bh - b * s.Hkv;
  const int row = divide(layer, s.gamma_magic) * s.rows + bh;          // of the index arrays
  const int32_t *idx = tok_idx + (int64_t)row * s.nkeep_max;
  const int step = ((int)blockIdx.x < s.last ? APART : s.last_apart) * ROWS;
  const int first = ((int)blockIdx.x / APART * (APART * GATHER_UNROLL) + (int)blockIdx.x % APART) * ROWS;
  const int r0 = first + threadIdx.x / LPR;

  int tok[GATHER_UNROLL];
#pragma unroll
  for (int u = 0; u < GATHER_UNROLL; ++u) tok[u] = idx[min(r0 + u * step, s.nkeep_max - 1)];
  int nk = n_keep[row];
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::"s"(nk));
#pragma unroll
  for (int u = 0; u < GATHER_UNROLL; ++u) asm volatile("" ::"v"(tok[u]));
  nk = min(nk, s.nkeep_max);
  const int n_write = s.fill_padding ? s.nkeep_max : nk;   // rows past n_keep: zero-filled or left alone
  if (first >= n_write) return;
  src += b * s.in_b + h * s.in_h + threadIdx.x % LPR * 16;
  dst += b * s.out_b + h * s.out_h + threadIdx.x % LPR * 16;
  u32x4 v[GATHER_UNROLL];
#pragma unroll
  for (int u = 0; u < GATHER_UNROLL; ++u) {
    v[u] = u32x4{0u, 0u, 0u, 0u};
    // indices are caller data: never read out of bounds
    if (r0 + u * step < nk && tok[u] >= 0 && tok[u] < s.max_tok)
      v[u] = __builtin_nontemporal_load((const u32x4 *)(src + (int64_t)tok[u] * s.in_t));
  }
#pragma unroll
  for (int u = 0; u < GATHER_UNROLL; ++u)
    if (r0 + u * step < n_write)
      __builtin_nontemporal_store(v[u], (u32x4 *)(dst + (int64_t)(r0 + u * step) * s.out_t));
}

template <int NT, int APART>
static hipError_t launch_gather_t(const Shape &s, const LayerPtrs &lp, int32_t n_layers, int32_t gamma, const int32_t *tok_idx, const int32_t *n_keep,
                                  hipStream_t stream) {
  const int64_t esize = elem_bytes(s.dtype);
  const int lpr = (int)(s.d * esize / 16);   // 8 (bf16 d=64), 16, 16, or 32 (f32 d=128)
  const GatherGrid g = gather_grid(s.nkeep_max, NT / lpr, APART);
  const GatherShape gs = {s.Hkv, s.B * s.Hkv, s.nkeep_max, s.fill_padding, s.t_stride + s.w_obs, g.last, g.last_apart, division_magic(s.Hkv),
                          division_magic(gamma), s.kv_sb * esize, s.kv_sh * esize, s.kv_st * esize, s.o_sb * esize, s.o_sh * esize, s.o_st * esize};
  dim3 grid(g.workgroups, s.B * s.Hkv, n_layers * 2);
  dim3 block(NT);
  switch (lpr) {
    case 8:  hipLaunchKernelGGL((gather_kernel<8, NT, APART>), grid, block, 0, stream, gs, lp, tok_idx, n_keep); break;
    case 16: hipLaunchKernelGGL((gather_kernel<16, NT, APART>), grid, block, 0, stream, gs, lp, tok_idx, n_keep); break;
    case 32: hipLaunchKernelGGL((gather_kernel<32, NT, APART>), grid, block, 0, stream, gs, lp, tok_idx, n_keep); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_gather(const Shape &s, const BatchParams &bp, const LayerPtrs &lp, int32_t n_layers, int32_t gamma,
                         const int32_t *tok_idx, const int32_t *n_keep, hipStream_t stream) {
  if (s.nkeep_max <= 0) return hipSuccess;
  switch (gather_threads(s, bp)) {
    case 64:  return launch_gather_t<64, 8>(s, lp, n_layers, gamma, tok_idx, n_keep, stream);
    case 128: return launch_gather_t<128, 4>(s, lp, n_layers, gamma, tok_idx, n_keep, stream);
    default:  return launch_gather_t<256, 1>(s, lp, n_layers, gamma, tok_idx, n_keep, stream);
  }
}

}  // namespace wkv
