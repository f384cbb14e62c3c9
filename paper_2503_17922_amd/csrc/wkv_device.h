// Device-side helpers shared by the score kernels (not part of the ABI).
#pragma once

#include "wkv_internal.h"

namespace wkv {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(8 * sizeof(_Float16)))) _Float16 f16x8;

// D = A (16 x 32) * B (32 x 16) + C on the matrix pipe; the 16-byte operands hold 8 bfloat16 or
// (F16) 8 IEEE half values and travel as bf16x8 either way.
template <bool F16>
__device__ __forceinline__ f32x4 mfma_16x16x32(bf16x8 a, bf16x8 b, f32x4 c) {
  if constexpr (F16)
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// One step of the contraction of TS rows of A with TS rows of B, 16 bytes of each per lane (lane l: row l % TS, piece
// l / TS).  16-bit types: one 16x16x32 or 32x32x16 instruction.  fp32: four 16x16x4 ones; the
// order in which they take the channels is the same for both operands, which is all a sum needs.
enum { DT_BF16 = 0, DT_F16 = 1, DT_F32 = 2 };
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
template <int TS> struct TileOf { typedef f32x4 acc; };
template <> struct TileOf<32> { typedef f32x16 acc; };
template <int DT, int TS>
__device__ __forceinline__ typename TileOf<TS>::acc mfma_step(bf16x8 a, bf16x8 b, typename TileOf<TS>::acc c) {
  if constexpr (DT == DT_F32) {
    static_assert(TS == 16, "fp32 tiles");
    const f32x4 av = __builtin_bit_cast(f32x4, a), bv = __builtin_bit_cast(f32x4, b);
#pragma unroll
    for (int i = 0; i < 4; ++i) c = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i], bv[i], c, 0, 0, 0);
    return c;
  } else if constexpr (TS == 16) {
    return mfma_16x16x32<DT == DT_F16>(a, b, c);
  } else if constexpr (DT == DT_F16) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  } else {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
}

// A word that no kernel writes while this one runs, by a scalar load; the address is the same in all lanes.  (Behind an asm statement the
// compiler takes a vector load by itself, as it cannot tell that nothing was written.)
template <typename T>
__device__ __forceinline__ T load_scalar(const T *p) { return *(const __attribute__((address_space(4))) T *)(uintptr_t)p; }

__device__ __forceinline__ uint32_t lds_address(const void *p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char *)p;
}
// A DMA instruction: 64 lanes fetch 16 bytes each from addresses of their own, to lds, lds + 16, ... in lane order.
// m0 holds the LDS address; naming it as overwritten keeps the compiler's own uses of it, should there be any,
// clear of this one (it is a reserved register, which clang warns of: nothing relies on its being preserved).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void dma_to_lds(uint32_t lds, const char *p) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds), "v"(p) : "memory", "m0");
}
#pragma clang diagnostic pop

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float fast_log2(float x) { return __builtin_amdgcn_logf(x); }

__device__ __forceinline__ float bf16_to_float(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// Merge (m2, z2) into (m, z): both describe sum 2^(v - m) over disjoint key sets.
__device__ __forceinline__ void merge_stats(float &m, float &z, float m2, float z2) {
  const float mn = fmaxf(m, m2);
  if (mn == -INFINITY) { m = mn; z = 0.0f; return; }
  z = z * fast_exp2(m - mn) + z2 * fast_exp2(m2 - mn);
  m = mn;
}

// ---- exchange between the four quads of a wave (lanes l, l+16, l+32, l+48) ------------------------
// (A swap's two results are read as integers first: bit-casting an element of the returned vector in place gives
// element 0 for both.)
struct Pair { float a, b; };
__device__ __forceinline__ Pair swap_halves(float x, float y) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  const unsigned a = r[0], b = r[1];
  return {__uint_as_float(a), __uint_as_float(b)};
}
__device__ __forceinline__ Pair swap_rows(float x, float y) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  const unsigned a = r[0], b = r[1];
  return {__uint_as_float(a), __uint_as_float(b)};
}
// Sums over the halves of the wave (the rows of each half): the lower lanes get that of x, the upper ones that of y.
__device__ __forceinline__ float add_halves(float x, float y) { const Pair p = swap_halves(x, y); return p.a + p.b; }
__device__ __forceinline__ float add_rows(float x, float y) { const Pair p = swap_rows(x, y); return p.a + p.b; }
// With one value: the sum / maximum over the lanes with equal lane % 16, in all of them.
__device__ __forceinline__ float quads_sum(float x) { x = add_halves(x, x); return add_rows(x, x); }
__device__ __forceinline__ float quads_max(float x) {
  Pair p = swap_halves(x, x);
  x = fmaxf(p.a, p.b);
  p = swap_rows(x, x);
  return fmaxf(p.a, p.b);
}

// ---- scans over the wave --------------------------------------------------------------------------
// Over the lanes of a wave by DPP steps (a shuffle through LDS takes 100 cycles and more, and there are a dozen of these in a
// row): shifts within rows of 16 lanes, then the last lane of a row, of two rows, into the ones after.  Lanes
// without a source add 0, the smallest key.
template <class F>
__device__ __forceinline__ uint32_t wave_scan(uint32_t x, F op) {
  x = op(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, false));     // row_shr:1
  x = op(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, false));     // row_shr:2
  x = op(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, false));     // row_shr:4
  x = op(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, false));     // row_shr:8
  x = op(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false));     // row_bcast:15
  return op(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false));  // row_bcast:31
}
// Sums up to and including each lane; the largest of all lanes.
__device__ __forceinline__ uint32_t wave_sums(uint32_t x) {
  return wave_scan(x, [](uint32_t a, uint32_t b) __attribute__((always_inline)) { return a + b; });
}
__device__ __forceinline__ uint32_t last_lane(uint32_t x) { return (uint32_t)__builtin_amdgcn_readlane((int)x, 63); }
__device__ __forceinline__ uint32_t wave_largest(uint32_t x) {
  return last_lane(wave_scan(x, [](uint32_t a, uint32_t b) __attribute__((always_inline)) { return max(a, b); }));
}

// ---- MFMA building blocks ----------------------------------
constexpr int MF_THREADS = 256;           // of a workgroup of the single-read kernel
constexpr int MF_WAVES = 4;              // waves that share the key tiles of an iteration
constexpr int MF_KT = 2;                 // key tiles of 16 per wave iteration (share each B fragment)
constexpr float MF_BIG = 1.0e30f;        // a tile sum above this re-references the row (2^100)
constexpr float MF_LOW = 1.0e-12f;       // so does a running sum below this (2^-40): terms that underflow are 2^-86 of it

// Arrange the M query rows of KV head h as MFMA B fragments in LDS.
// Fragment (mt, ks) is 64 x 16 bytes: lane l holds row 16*mt + l%16, bytes 64*ks + 16*(l/16)..+15 of it.
template <int D, int MT, int NT>                          // NT threads stage MT row tiles (16-bit elements)
struct QStage {
  static constexpr int KS = D / 32;
  static constexpr int TOTAL = MT * KS * 64;               // 16-byte pieces of the fragments
  static constexpr int N = (TOTAL + NT - 1) / NT;          // per thread
  uint4 v[N];
  // Issue every load of this thread at once (independent of each other, so their latencies
  // overlap; a load-then-store loop would pay one round trip per piece).
  __device__ __forceinline__ void load(const Shape &s, const void *qbase, int b, int h, int tid = threadIdx.x) {
#pragma unroll
    for (int k = 0; k < N; ++k) {
      const int i = tid + k * NT;
      const int l = i & 63, f = i >> 6, ks = f % KS, mt = f / KS;
      const int r = mt * 16 + (l & 15);
      v[k] = make_uint4(0u, 0u, 0u, 0u);
      if (i < TOTAL && r < s.M) {
        const int hq = h * s.G + r / s.w_obs, io = r % s.w_obs;
        const int64_t off = (int64_t)b * s.q_sb + (int64_t)hq * s.q_sh + (int64_t)io * s.q_st;
        v[k] = *(const uint4 *)((const char *)qbase + off * 2 + ks * 64 + (l >> 4) * 16);
      }
    }
  }
  __device__ __forceinline__ void store(uint4 *qfrag, int tid = threadIdx.x) const {
#pragma unroll
    for (int k = 0; k < N; ++k)
      if (tid + k * NT < TOTAL) qfrag[tid + k * NT] = v[k];
  }
};

// Sum over the 16 lanes of a DPP row (lanes with equal l/16); every lane gets the total.
__device__ __forceinline__ float row16_sum(float x) {
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0xB1, 0xF, 0xF, false));  // quad_perm [1,0,3,2]
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x4E, 0xF, 0xF, false));  // quad_perm [2,3,0,1]
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x141, 0xF, 0xF, false)); // row_half_mirror
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x140, 0xF, 0xF, false)); // row_mirror
  return x;
}

template <int KS>
struct KFrags {
  bf16x8 f[MF_KT][KS];
};

// Loads the A fragments of MF_KT key tiles starting at key j0 (rows clamped into [0, L-1];
// callers pass L >= 1).  kbase: the lane's 16-byte piece of key row 0; st: bytes between key rows.
template <int KS>
__device__ __forceinline__ void load_k(KFrags<KS> &kf, const char *kbase, int64_t st, int j0, int col, int L) {
#pragma unroll
  for (int n = 0; n < MF_KT; ++n) {
    const int j = min(j0 + n * 16 + col, L - 1);
    const char *kp = kbase + (int64_t)j * st;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) kf.f[n][ks] = *(const bf16x8 *)(kp + ks * 64);
  }
}

}  // namespace wkv
