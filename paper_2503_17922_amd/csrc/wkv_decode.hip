// One decode step over the compact cache: the new token's K/V row is appended and its query
// heads attend to every retained row (softmax(q.K^T * scale).V, nothing masked).
//
// With one query row per head this is a matrix-vector product per KV head: every K and V row
// is read once and used for G = Hq/Hkv dot products, so the step is bound by the HBM stream of
// the two caches; what matters is that the arithmetic per row stays well below the memory rate.
//
//   partial kernel  grid (B*Hkv, splits): a workgroup walks one key range of one KV head, over the rows
//                   that are in the cache already.
//                   fp32 inputs: everything on the vector ALU, as follows.  16-bit inputs: the
//                   scores come from the matrix pipe (decode_partial_mfma_kernel below), the
//                   value side keeps this layout.  A
//                   16-byte piece of a row per lane, so D*esize/16 lanes cover a row and a wave
//                   load instruction reads 64/that many consecutive rows (fully coalesced).  Each
//                   lane group keeps its own online-softmax state (running max, sum, output
//                   piece) per query head, so nothing crosses lanes inside the loop except the
//                   dot-product reduction within a row's lanes; lane groups, then waves, merge
//                   once at the end and the workgroup writes (m, l, o) to the workspace.
//   combine kernel  grid (B*Hkv, G): merges the key ranges of one query head and the new token (one dot
//                   product; its row is appended to the caches here), normalises, writes fp32 output, bumps
//                   the row count.
#include <atomic>
#include <mutex>
#include <type_traits>

#include "wkv_device.h"

namespace wkv {

// Scratch memory of wkv_decode_step_static: part of the device image, one copy per GPU at that
// GPU's own address.  In host code the name is only a handle for hipGetSymbolAddress; the device
// address found there (per device, once) is what the kernels get.
static __device__ __align__(256) unsigned char scratch[WKV_DECODE_STATIC_SCRATCH_BYTES];

constexpr int DEC_THREADS = 256;
constexpr int DEC_WAVES = DEC_THREADS / 64;
constexpr int WIDE_THREADS = 512;   // where a range is a block for each of eight waves (see launch_partial_g)
constexpr int DEC_U = 4;            // row tiles per wave batch (loads in flight: 2 * DEC_U per lane)

// A 16-byte piece of a cache row.  STREAM: a nontemporal load, which puts nothing into the memory-side cache; a kernel
// that only reads such a stream reaches 7.0 TB/s with it, 6.1 without (1 GB in 1536 ranges).
template <bool STREAM>
__device__ __forceinline__ uint4 load_piece(const void *p) {
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  return __builtin_bit_cast(uint4, STREAM ? __builtin_nontemporal_load((const u32x4 *)p) : *(const u32x4 *)p);
}

struct half_t { uint16_t bits; };             // element tag of IEEE half tensors (uint16_t stands for bfloat16)

template <typename T> struct Piece;           // the 16-byte piece of a row held by one lane
template <> struct Piece<half_t> {
  static constexpr int E = 8;
  static __device__ __forceinline__ void unpack(const uint4 &r, float (&f)[8]) {
    const f16x8 h = __builtin_bit_cast(f16x8, r);
#pragma unroll
    for (int i = 0; i < 8; ++i) f[i] = (float)h[i];
  }
  static __device__ __forceinline__ float value(const half_t *p) { return (float)__builtin_bit_cast(_Float16, p->bits); }
};
template <> struct Piece<uint16_t> {
  static constexpr int E = 8;
  static __device__ __forceinline__ void unpack(const uint4 &r, float (&f)[8]) {
    const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      f[2 * i] = __uint_as_float(w[i] << 16);
      f[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
  }
  static __device__ __forceinline__ float value(const uint16_t *p) { return bf16_to_float(*p); }
};
template <> struct Piece<float> {
  static constexpr int E = 4;
  static __device__ __forceinline__ void unpack(const uint4 &r, float (&f)[4]) {
    f[0] = __uint_as_float(r.x); f[1] = __uint_as_float(r.y); f[2] = __uint_as_float(r.z); f[3] = __uint_as_float(r.w);
  }
  static __device__ __forceinline__ float value(const float *p) { return *p; }
};

// Sum over the LPK (8, 16 or 32) adjacent lanes that hold one row; every lane gets the total.
template <int LPK>
__device__ __forceinline__ float row_lanes_sum(float x) {
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0xB1, 0xF, 0xF, false));  // quad_perm [1,0,3,2]
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x4E, 0xF, 0xF, false));  // quad_perm [2,3,0,1]
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x141, 0xF, 0xF, false)); // row_half_mirror
  if (LPK >= 16)
    x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x140, 0xF, 0xF, false)); // row_mirror
  if (LPK >= 32) x += __shfl_xor(x, 16);
  return x;
}

// Sum and maximum over the wave, in every lane: DPP steps inside rows of 16 lanes, then two permlane swaps.
__device__ __forceinline__ float wave_sum(float x) { return quads_sum(row16_sum(x)); }
__device__ __forceinline__ float wave_max(float x) {
  x = fmaxf(x, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0xB1, 0xF, 0xF, false)));  // quad_perm [1,0,3,2]
  x = fmaxf(x, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x4E, 0xF, 0xF, false)));  // quad_perm [2,3,0,1]
  x = fmaxf(x, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x141, 0xF, 0xF, false))); // row_half_mirror
  x = fmaxf(x, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x140, 0xF, 0xF, false))); // row_mirror
  return quads_max(x);
}

// Merge the online-softmax state (m2, l2, o2) into (m, l, o); all in base 2.
template <int E>
__device__ __forceinline__ void merge_state(float &m, float &l, float (&o)[E], float m2, float l2, const float (&o2)[E]) {
  const float mn = fmaxf(m, m2);
  if (mn == -INFINITY) return;                      // both empty
  const float a = fast_exp2(m - mn), b = fast_exp2(m2 - mn);
  l = l * a + l2 * b;
#pragma unroll
  for (int c = 0; c < E; ++c) o[c] = o[c] * a + o2[c] * b;
  m = mn;
}

// Partial results in the workspace: the outputs [B*Hkv][splits][G][D] of every key range (only of ranges that
// hold rows), then their (m, l) [B*Hkv][splits][G].  A range past the end of a row has m = -inf; m of range 0
// is NaN where the cache cannot take the new row.
// (Byte offsets fit 32 bits: at most 65535 heads of one range each, or 1536 ranges, times eight query heads of 130 floats.  A launch runs
// through its code once, at some 7 cycles an instruction, and products of 64 bits are a dozen of them.)
__device__ __forceinline__ uint32_t part_index(const DecodeShape &s, int bh, int split, int g) {
  return ((uint32_t)bh * s.n_splits + split) * s.G + g;
}
__device__ __forceinline__ float2 &part_stats(const DecodeShape &s, float *part, uint32_t at) {
  return *(float2 *)((char *)part + (s.stats_at + at * 8u));
}
__device__ __forceinline__ const float2 &part_stats(const DecodeShape &s, const float *part, uint32_t at) {
  return *(const float2 *)((const char *)part + (s.stats_at + at * 8u));
}

// Merge the per-wave states in LDS ([wave][head][D outputs, m, l]) and store the workgroup's
// partial result: one thread per (head, channel); the statistics are recomputed per thread.
template <int D, int G>
__device__ __forceinline__ void merge_waves_and_store(const DecodeShape &s, float (&wave_state)[DEC_WAVES][G][D + 2],
                                                      int bh, int split, float *__restrict__ part) {
  __syncthreads();
  for (int i = threadIdx.x; i < G * D; i += DEC_THREADS) {
    const int g = i / D, c = i % D;
    float mm = wave_state[0][g][D];
#pragma unroll
    for (int w = 1; w < DEC_WAVES; ++w) mm = fmaxf(mm, wave_state[w][g][D]);
    float ll = 0.0f, oo = 0.0f;
    if (mm != -INFINITY) {
#pragma unroll
      for (int w = 0; w < DEC_WAVES; ++w) {
        const float a = fast_exp2(wave_state[w][g][D] - mm);
        ll += wave_state[w][g][D + 1] * a;
        oo += wave_state[w][g][c] * a;
      }
    }
    const uint32_t at = part_index(s, bh, split, g);
    part[at * D + c] = oo;
    if (c == 0) part_stats(s, part, at) = make_float2(mm, ll);
  }
}

// A key range without rows says so in its statistics; so does range 0 of a row that cannot take another token.
template <int G>
__device__ __forceinline__ bool nothing_to_do(const DecodeShape &s, int bh, int split, int n, int c0, int cend,
                                              float *__restrict__ part) {
  if (__builtin_expect(c0 < cend, 1)) return false;
  if (threadIdx.x < G)
    part_stats(s, part, part_index(s, bh, split, threadIdx.x)) =
        make_float2(split == 0 && (n < 0 || n >= s.capacity) ? __uint_as_float(0x7fc00000u) : -INFINITY, 0.0f);
  return true;
}

// Which range of which cache this workgroup takes, and the rows of that cache.  It looks at the count of its own cache alone: a caller may
// write the counts of other sequences meanwhile (a slot of the batch that is being filled anew).  Ranges dealt out by all counts, whole ones first,
// would leave ranges of the others to nobody when a count changes between the start of two workgroups; they took, us a layer, own count / all: mixed
// batches of 32q/8kv heads, 8 up to 8000 rows 27.6 / 26.5, 24 up to 4000 45.1 / 38.4, 64 up to 2000 59.5 / 55.1; 64 of 4128 167.5 / 168.3, 16 48.7 / 49.4.
struct KeyRange {
  int head, range, n;
  __device__ __forceinline__ KeyRange(const DecodeShape &s, const int32_t *__restrict__ n_valid) {
    const RangeOf it(blockIdx.x, blockIdx.y, s.B * s.Hkv, s.heads_magic);
    head = it.head; range = it.range; n = load_scalar(n_valid + head);
  }
};

template <typename T, int D, int G, bool STREAM>
__global__ __launch_bounds__(DEC_THREADS) void decode_partial_kernel(DecodeShape s, const T *__restrict__ q_new,
                                                                     const T *__restrict__ k_cache,
                                                                     const T *__restrict__ v_cache,
                                                                     const int32_t *__restrict__ n_valid,
                                                                     float *__restrict__ part) {
  constexpr int E = Piece<T>::E;
  constexpr int LPK = D / E;                 // lanes per row
  constexpr int KPT = 64 / LPK;              // rows per wave load instruction
  __shared__ float wave_state[DEC_WAVES][G][D + 2];

  const KeyRange item(s, n_valid);
  const int bh = item.head, b = divide(bh, s.kv_magic), h = bh - b * s.Hkv, split = item.range;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int slot = lane / LPK, piece = lane % LPK;
  const int n = item.n, c0 = split * s.chunk, cend = min(c0 + s.chunk, n < s.capacity ? n : 0);
  if (nothing_to_do<G>(s, bh, split, n, c0, cend, part)) return;

  const T *kc = k_cache + (int64_t)b * s.sb + (int64_t)h * s.sh;
  const T *vc = v_cache + (int64_t)b * s.sb + (int64_t)h * s.sh;

  // this lane's piece of the G query rows, pre-multiplied by scale * log2(e)
  float qv[G][E];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    float f[E];
    Piece<T>::unpack(*(const uint4 *)(q_new + ((int64_t)bh * G + g) * D + piece * E), f);
#pragma unroll
    for (int c = 0; c < E; ++c) qv[g][c] = f[c] * s.c1;
  }

  float m[G], l[G], o[G][E];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    m[g] = -INFINITY; l[g] = 0.0f;
#pragma unroll
    for (int c = 0; c < E; ++c) o[g][c] = 0.0f;
  }

  // rows of this wave: tiles of KPT rows, tile index wave, wave + DEC_WAVES, ...; DEC_U tiles per batch
  uint4 kr[DEC_U], vr[DEC_U];
  auto load_batch = [&](int t0) {
#pragma unroll
    for (int u = 0; u < DEC_U; ++u) {
      const int64_t off = (int64_t)min(c0 + (t0 + u * DEC_WAVES) * KPT + slot, cend - 1) * s.st + piece * E;
      kr[u] = load_piece<STREAM>(kc + off);
      vr[u] = load_piece<STREAM>(vc + off);
    }
  };
  int t0 = wave;
  load_batch(t0);
  for (; c0 + t0 * KPT < cend; t0 += DEC_U * DEC_WAVES) {
    uint4 kcur[DEC_U], vcur[DEC_U];
#pragma unroll
    for (int u = 0; u < DEC_U; ++u) { kcur[u] = kr[u]; vcur[u] = vr[u]; }
    load_batch(t0 + DEC_U * DEC_WAVES);          // next batch (past the end: the last row again)

    float sc[DEC_U][G];
#pragma unroll
    for (int u = 0; u < DEC_U; ++u) {
      float kf[E];
      Piece<T>::unpack(kcur[u], kf);
      const int j = c0 + (t0 + u * DEC_WAVES) * KPT + slot;
#pragma unroll
      for (int g = 0; g < G; ++g) {
        float a = 0.0f;
#pragma unroll
        for (int c = 0; c < E; ++c) a = fmaf(qv[g][c], kf[c], a);
        a = row_lanes_sum<LPK>(a);
        sc[u][g] = j < cend ? a : -INFINITY;
      }
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
      float bm = sc[0][g];
#pragma unroll
      for (int u = 1; u < DEC_U; ++u) bm = fmaxf(bm, sc[u][g]);
      const float mn = fmaxf(m[g], bm);
      if (mn != -INFINITY) {
        const float corr = fast_exp2(m[g] - mn);    // m = -inf: 0
        m[g] = mn;
        l[g] *= corr;
#pragma unroll
        for (int c = 0; c < E; ++c) o[g][c] *= corr;
      }
    }
#pragma unroll
    for (int u = 0; u < DEC_U; ++u) {
      float vf[E];
      Piece<T>::unpack(vcur[u], vf);
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const float p = m[g] == -INFINITY ? 0.0f : fast_exp2(sc[u][g] - m[g]);
        l[g] += p;
#pragma unroll
        for (int c = 0; c < E; ++c) o[g][c] = fmaf(p, vf[c], o[g][c]);
      }
    }
  }

  // merge the KPT lane groups of the wave (lanes with equal piece)
#pragma unroll
  for (int g = 0; g < G; ++g) {
#pragma unroll
    for (int off = LPK; off < 64; off <<= 1) {
      float o2[E];
      const float m2 = __shfl_xor(m[g], off), l2 = __shfl_xor(l[g], off);
#pragma unroll
      for (int c = 0; c < E; ++c) o2[c] = __shfl_xor(o[g][c], off);
      merge_state<E>(m[g], l[g], o[g], m2, l2, o2);
    }
    if (slot == 0) {
#pragma unroll
      for (int c = 0; c < E; ++c) wave_state[wave][g][piece * E + c] = o[g][c];
      if (piece == 0) { wave_state[wave][g][D] = m[g]; wave_state[wave][g][D + 1] = l[g]; }
    }
  }
  merge_waves_and_store<D, G>(s, wave_state, bh, split, part);
}

// ---- bf16 / fp16: scores on the matrix pipe --------------------------------------------------
// The G query rows (padded to 16) are the B operand of v_mfma_f32_16x16x32_bf16 (_f16) and 16 cache rows
// the A operand, loaded in operand layout as in the score kernels, so a block of 16 rows costs
// D/32 MFMAs instead of 16 * G dot-product reductions, and each lane takes the exponent of 4
// scores instead of G per row.  V is contracted over rows, the wrong way round for an MFMA operand, and
// stays on the vector ALU in the row-piece layout above.  In the 16x16 result the lanes of one quad (16
// lanes) hold rows 4*quad .. 4*quad+3, lane g of the quad those of head g; a quad's lanes take these very
// rows on the value side, so the probability of a row and head is a broadcast inside a DPP row and
// nothing goes through LDS in the loop.  Every lane of a wave uses the same running maximum per head, so
// the lane groups' outputs simply add up at the end: permlane swaps, which halve the number of values
// at each step.
// A long cache is bound by the stream of its rows.  A single sequence (a block or two per wave) is bound by
// the length of the code itself, fetched anew in every launch, and by LDS round trips: hence no
// LDS in the loop and no shuffles through it at the end.  One 32q/8kv-head layer with 4128 rows in ranges of
// 64, bf16: 10.6 us with probabilities through LDS and ds_bpermute reductions, 8.6 us so.  A wave requests two blocks at a time, all it
// has in a range of 128 rows, and waits for memory once; the arithmetic of both is one piece of code, and the heads' numbers are
// divided by multiplication.  Such a layer with its merge 11.3 us with one block requested ahead of the one in hand (the compiler
// put the request of the second behind the arrival of the first), 10.1 us so; eleven sequences of mixed lengths, 28q/4kv heads, f16, a layer
// 16.6 and 14.8 us; 64 sequences 169 and 167.  Ranges of 64 rows, one block without a state for each of four waves, against the
// present kernels: one sequence 8.53 -> 9.07, two 11.06 -> 11.65, the eleven 14.24 -> 14.21.  Two blocks and a state take 102 to 125 registers with
// 128 channels and up to four heads (four waves a SIMD), 134 to 162 with more (three), one block without a state 56 to 60 (eight).
// Ranges of a block a wave without a state before it, a lane's rows by one multiplication each, the caches'
// addresses while the row count is under way; here and in the merge offsets of 32 bits into the partial results: one sequence of 4128 rows through 32
// layers 309 -> 298 us, of 20000 rows 22.0 -> 20.6 a layer, three of 4128 14.4 -> 13.7, fp32 with four 21.3 -> 20.8.
// The value of lane N of each 16-lane DPP row, in all its lanes.
template <int N>
__device__ __forceinline__ float row_bcast(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x150 + N, 0xF, 0xF, true));   // row_newbcast
}
template <int N, class F>
__device__ __forceinline__ void static_for(F &&f) {
  if constexpr (N > 0) { static_for<N - 1>(f); f(std::integral_constant<int, N - 1>{}); }
}
// STREAM: 0 plain loads, 1 values stream, 2 keys too (see launch_partial_g).
template <int D, int G, bool F16, int STREAM, int NT>
__global__ __launch_bounds__(NT, 3) void decode_partial_mfma_kernel(
    DecodeShape s, const uint16_t *__restrict__ q_new, const uint16_t *k_cache,
    const uint16_t *v_cache, const int32_t *__restrict__ n_valid, float *__restrict__ part) {
  constexpr int E = 8, WAVES = NT / 64;
  constexpr bool PAIRS = WAVES == DEC_WAVES;
  constexpr int LPK = D / E;                 // lanes per row (value side): 16 or 8
  constexpr int VT = D / 32;                 // value loads per block of 16 rows: rows of a quad / rows it reads at once
  constexpr int KS = D / 32;                 // MFMA steps over the channels
  __shared__ __attribute__((aligned(16))) float o_s[WAVES][G][D];
  __shared__ float2 ml_s[WAVES][G];

  // (all arguments together, ahead of the row count that depends on one of them)
  asm volatile("" ::"s"(s.B), "s"(s.Hkv), "s"(s.heads_magic), "s"(s.kv_magic), "s"(s.chunk), "s"(s.capacity), "s"(s.c1), "s"(s.sb), "s"(s.sh), "s"(s.st),
               "s"(s.n_splits), "s"(s.G), "s"(s.stats_at), "s"(q_new), "s"(k_cache), "s"(v_cache), "s"(n_valid), "s"(part));
  const KeyRange item(s, n_valid);
  const int bh = item.head, b = divide(bh, s.kv_magic), h = bh - b * s.Hkv, split = item.range;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 15, quad = lane >> 4;            // score side: head, 4 rows
  const int piece = lane % LPK, sub = col / LPK;          // value side: 16-byte piece, which of the quad's rows in flight
  const int64_t head_at = ((int64_t)b * s.sb + (int64_t)h * s.sh) * 2, row_bytes = s.st * 2;
  const char *kc = (const char *)k_cache + head_at, *vc = (const char *)v_cache + head_at;

  if (!PAIRS) {
    __builtin_amdgcn_sched_barrier(0);       // (all that while the row count is under way)
    asm volatile("" ::"s"(kc), "s"(vc));
  }
  const int n = item.n, c0 = split * s.chunk, cend = min(c0 + s.chunk, n < s.capacity ? n : 0);
  if (nothing_to_do<G>(s, bh, split, n, c0, cend, part)) return;

  // query rows as B fragments: lane (head col, quad) holds channels 32*ks + 8*quad .. +7; columns past the
  // last head repeat it and are not used
  bf16x8 qb[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    qb[ks] = *(const bf16x8 *)(q_new + ((int64_t)bh * G + min(col, G - 1)) * D + ks * 32 + quad * 8);
  }

  float m = -INFINITY, l = 0.0f;             // of head `col` (lanes with col < G), l over this lane's rows only
  float o[G * E];                            // [head][channel of the piece]

  // Blocks of 16 rows, every WAVES-th of the range, by four waves two at a time: a range of 128 rows is one round trip to memory.
  struct Block { uint4 k[KS], v[VT]; };
  // (Rows past the range: its last one again.)
  auto load_block = [&](Block &x, int blk) __attribute__((always_inline)) {
    const char *kr = kc, *vr = vc;
    int64_t ka, va[VT];
    if constexpr (PAIRS) {
      const int r0 = c0 + blk * 16;
      ka = min(r0 + col, cend - 1) * row_bytes;
#pragma unroll
      for (int t = 0; t < VT; ++t) va[t] = min(r0 + quad * 4 + t * (4 / VT) + sub, cend - 1) * row_bytes;
    } else {
      // A lane's rows by one multiplication each, from the block's first, as row_bytes above 2^32 is as good as never: a launch of one short block a
      // wave waits for its addresses.  (Of two blocks at once the longer scalar chain costs more: eleven mixed sequences with 28q/4kv heads 58.5 -> 59.5 us.)
      const int r0 = min(c0 + blk * 16, cend - 1), rows = cend - 1 - r0;       // (uniform)
      const uint32_t low = (uint32_t)row_bytes, high = (uint32_t)(row_bytes >> 32), rk = min(col, rows);
      kr += r0 * row_bytes; vr += r0 * row_bytes;
      ka = (int64_t)((uint64_t)rk * low);
#pragma unroll
      for (int t = 0; t < VT; ++t) va[t] = (int64_t)((uint64_t)(uint32_t)min(quad * 4 + t * (4 / VT) + sub, rows) * low);
      if (__builtin_expect(high != 0, 0)) {
        ka += (int64_t)(rk * high) << 32;
#pragma unroll
        for (int t = 0; t < VT; ++t) va[t] += (int64_t)((uint32_t)min(quad * 4 + t * (4 / VT) + sub, rows) * high) << 32;
      }
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) x.k[ks] = load_piece<(STREAM > 1)>(kr + ka + (quad * 16 + ks * 64));
#pragma unroll
    for (int t = 0; t < VT; ++t) x.v[t] = load_piece<(STREAM > 0)>(vr + va[t] + piece * 16);
  };
  auto attend = [&](const Block &x, int blk) __attribute__((always_inline)) {
    // scores of 16 rows x 16 (padded) heads
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      acc = mfma_16x16x32<F16>(*(const bf16x8 *)&x.k[ks], qb[ks], acc);
    const int r0 = c0 + blk * 16 + quad * 4;
    float sc[4], pr[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) sc[e] = r0 + e < cend ? acc[e] * s.c1 : -INFINITY;
    float mn = quads_max(fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3])));
    if (PAIRS) mn = fmaxf(m, mn);
    // -inf: every row so far has a logit of -inf (an infinite key, products that overflow) and weighs nothing
    const bool none = mn == -INFINITY;
    const float corr = none || !PAIRS ? 1.0f : fast_exp2(m - mn);        // m = -inf: 0
    m = mn;
#pragma unroll
    for (int e = 0; e < 4; ++e) pr[e] = none ? 0.0f : fast_exp2(sc[e] - mn);
    l = (PAIRS ? l * corr : 0.0f) + ((pr[0] + pr[1]) + (pr[2] + pr[3]));
    if (PAIRS && __any(corr != 1.0f && col < G))
      static_for<G>([&](auto g) {
        const float c = row_bcast<g>(corr);
#pragma unroll
        for (int i = 0; i < E; ++i) o[g * E + i] *= c;
      });
    if (!PAIRS) __builtin_amdgcn_sched_barrier(0);             // (no value is waited for before the scores are done)
#pragma unroll
    for (int t = 0; t < VT; ++t) {
      float vf[E];
      if constexpr (F16) Piece<half_t>::unpack(x.v[t], vf); else Piece<uint16_t>::unpack(x.v[t], vf);
      static_for<G>([&](auto g) {
        float p = row_bcast<g>(pr[t * (4 / VT)]);
        if constexpr (LPK == 8) {                // two rows of the quad at once: its upper 8 lanes take the second
          const float p1 = row_bcast<g>(pr[t * 2 + 1]);
          p = sub ? p1 : p;
        }
#pragma unroll
        for (int i = 0; i < E; ++i) o[g * E + i] = PAIRS || t > 0 ? fmaf(p, vf[i], o[g * E + i]) : p * vf[i];
      });
    }
  };
  if constexpr (!PAIRS) {                      // one block a wave, nothing before it (launch_partial_g)
    if (c0 + wave * 16 < cend) {
      Block x;
      load_block(x, wave);
      __builtin_amdgcn_sched_barrier(0);       // the values too, before the scores wait for the keys
      attend(x, wave);
    } else {
#pragma unroll
      for (int i = 0; i < G * E; ++i) o[i] = 0.0f;
    }
  } else {
#pragma unroll
    for (int i = 0; i < G * E; ++i) o[i] = 0.0f;
    for (int blk = wave; c0 + blk * 16 < cend; blk += WAVES) {
      Block x, next;
      load_block(x, blk);
      // (past the end: the last row again, which the chip has at hand.  Around a branch instead: one sequence of 4128 rows, 64q/8kv heads 10.30 ->
      // 10.66 us a layer, eleven mixed with 12q/2kv 12.03 -> 12.85, sixteen of 70 rows 8.60 -> 8.83, 64 of 4128 rows 167.4 -> 168.7)
      load_block(next, blk + WAVES);
      __builtin_amdgcn_sched_barrier(0);       // both are requested before the first is looked at
      for (bool more = c0 + (blk + WAVES) * 16 < cend;; more = false) {            // (one copy of the code, which every launch fetches anew)
        attend(x, blk);
        if (!more) break;
        blk += WAVES;
        x = next;
      }
      __builtin_amdgcn_s_waitcnt(0x0f70);      // vmcnt(0), reached by now but for rows requested past the end; else the compiler waits for the queries among the first requests
    }
  }

  // The wave's totals.  After the two swap steps lane (quad, piece) holds 2*G of a piece's sums: those of
  // values quad * 2*G .. +2*G-1 of [head][channel] (quad 0: the first quarter, 1: the second, ...).
  constexpr int N = G * E;
#pragma unroll
  for (int i = 0; i < N / 2; ++i) o[i] = add_halves(o[i], o[i + N / 2]);
#pragma unroll
  for (int i = 0; i < N / 4; ++i) {
    o[i] = add_rows(o[i], o[i + N / 4]);
    if constexpr (LPK == 8)
      o[i] += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, o[i]), 0x128, 0xF, 0xF, false));   // row_ror:8
  }
  l = quads_sum(l);
  if (sub == 0) {
#pragma unroll
    for (int i = 0; i < N / 4; i += 2) {
      const int at = quad * (N / 4) + i;         // value `at` is channel at % 8 of head at / 8; pairs never cross a head
      *(float2 *)&o_s[wave][at / E][piece * E + at % E] = make_float2(o[i], o[i + 1]);
    }
  }
  if (lane < G) ml_s[wave][lane] = make_float2(m, l);        // lane = head (quad 0)
  __syncthreads();

  // merge the waves: a thread takes four channels of one head
  for (int i = threadIdx.x; i < G * (D / 4); i += NT) {
    const int g = i / (D / 4), c = i % (D / 4) * 4;
    float mm = -INFINITY, ll = 0.0f;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) mm = fmaxf(mm, ml_s[w][g].x);
    float4 oo = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      const float a = mm == -INFINITY ? 0.0f : fast_exp2(ml_s[w][g].x - mm);      // (no row of the range weighs anything)
      const float4 x = *(const float4 *)&o_s[w][g][c];
      ll = fmaf(ml_s[w][g].y, a, ll);
      oo.x = fmaf(x.x, a, oo.x); oo.y = fmaf(x.y, a, oo.y); oo.z = fmaf(x.z, a, oo.z); oo.w = fmaf(x.w, a, oo.w);
    }
    const uint32_t at = part_index(s, bh, split, g);
    *(float4 *)((char *)part + (at * D + c) * 4u) = oo;
    if (c == 0) part_stats(s, part, at) = make_float2(mm, ll);
  }
}

// One workgroup per (sequence, KV head, query head): D/4 lanes hold a row of outputs, so GROUPS key ranges
// are summed side by side.  Bound by its chain of round trips to memory (the data is a few KB a head), hence
// the outputs of the first ranges are requested together with the statistics that weigh them.  At 8 KV heads and
// 33 ranges 3.3 us from first wave to last with shuffles through LDS and four ranges ahead (the 33rd took a round trip of its
// own), 2.6 us with DPP reductions and six.
// With few ranges one wave does it all and weighs them without LDS, a lane each (16 sequences of 500 rows 11.53 -> 11.28 us a layer; four
// waves that each weigh up to 64 ranges for themselves, 9.55 -> 9.84 us for one sequence of 4128 rows: not so).
template <typename T, int D, int NT>
__global__ __launch_bounds__(NT) void decode_combine_kernel(DecodeShape s, const T *__restrict__ q_new,
                                                                     const T *__restrict__ k_new, const T *__restrict__ v_new,
                                                                     T *k_cache, T *v_cache, const float *__restrict__ part,
                                                                     int32_t *n_valid, float *__restrict__ out) {
  constexpr int COLS = D / 4, GROUPS = NT / COLS, AHEAD = NT == 64 ? 4 : 6, WAVES = NT / 64;
  constexpr int E = Piece<T>::E, LPK = D / E;
  constexpr bool FEW = NT == 64;
  __shared__ float wgt[FEW ? 1 : NT + AHEAD * GROUPS];             // (the ones past the last range are 0)
  __shared__ __attribute__((aligned(16))) float acc_s[GROUPS][D];
  __shared__ float q_k[2];
  __shared__ float wave_m[WAVES], wave_l[WAVES];
  // Two trips to memory: the arguments, then everything that follows from them.
  asm volatile("" ::"s"(s.B), "s"(s.Hkv), "s"(s.G), "s"(s.d), "s"(s.kv_magic), "s"(s.capacity), "s"(s.n_splits), "s"(s.c1), "s"(s.sb), "s"(s.sh), "s"(s.st),
               "s"(s.keep_count), "s"(s.stats_at), "s"(q_new), "s"(k_new), "s"(v_new), "s"(k_cache), "s"(v_cache), "s"(part), "s"(n_valid), "s"(out));
  const int bh = blockIdx.x, g = blockIdx.y, b = divide(bh, s.kv_magic), h = bh - b * s.Hkv;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int grp = tid / COLS, col = tid % COLS;
  const int64_t hq = (int64_t)bh * s.G + g;

  // statistics of this head's ranges (one per thread), outputs of the first ranges, the new token
  float2 ml = make_float2(-INFINITY, 0.0f);
  if (tid < s.n_splits) ml = part_stats(s, part, part_index(s, bh, tid, g));
  const char *po = (const char *)part + part_index(s, bh, 0, g) * (D * 4u);         // range sp: sp * range_bytes further on
  const uint32_t range_bytes = s.G * (D * 4u), last_range = (s.n_splits - 1) * range_bytes;
  uint32_t out_at = grp * range_bytes;
  float4 pre[AHEAD];
  auto request = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) {
      pre[u] = *(const float4 *)(po + (min(out_at, last_range) + col * 16u));
      out_at += GROUPS * range_bytes;
    }
  };
  request();
  const bool appends = g == 0 && tid < 2 * LPK;             // the new row, by head 0's workgroup: keys, then values
  uint4 row_piece = make_uint4(0, 0, 0, 0);
  if (appends) row_piece = *(const uint4 *)((tid < LPK ? k_new : v_new) + (int64_t)bh * D + tid % LPK * E);
  T v_piece[(D + NT - 1) / NT];                             // the new values of this thread's outputs
#pragma unroll
  for (int i = 0; i < (D + NT - 1) / NT; ++i) v_piece[i] = v_new[(int64_t)bh * D + min(tid + i * NT, D - 1)];
  const bool takes_dot = wave == WAVES - 1;       // this wave also takes q . k_new
  uint4 q_piece = make_uint4(0, 0, 0, 0), k_piece = q_piece;
  if (takes_dot && lane < LPK) {
    q_piece = *(const uint4 *)(q_new + hq * D + lane * E);
    k_piece = *(const uint4 *)(k_new + (int64_t)bh * D + lane * E);
  }
  // (of head 0's workgroup alone, which raises it at the end; in a vector register, as a scalar would be waited for at once)
  int n = -1;
  if (appends) n = n_valid[bh];
  __builtin_amdgcn_sched_barrier(0);
  float dot = 0.0f;
  if (takes_dot) {
    float qf[E], kf[E];
    Piece<T>::unpack(q_piece, qf);
    Piece<T>::unpack(k_piece, kf);
#pragma unroll
    for (int c = 0; c < E; ++c) dot = fmaf(qf[c], kf[c], dot);
  }
  float logit, m, l, a, w_new, first;                   // first: m of range 0; NaN: the cache is full or its count is invalid
  if (takes_dot) dot = wave_sum(dot) * s.c1;
  if constexpr (FEW) {
    logit = dot;
    first = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, ml.x), 0));
    m = fmaxf(logit, wave_max(ml.x));
    a = fast_exp2(ml.x - m);                            // a range without rows: 0
    w_new = fast_exp2(logit - m);
    l = w_new + wave_sum(ml.x == -INFINITY ? 0.0f : ml.y * a);
  } else {
    if (takes_dot && lane == 0) q_k[0] = dot;
    m = wave_max(ml.x);
    if (lane == 0) wave_m[wave] = m;
    if (tid == 0) q_k[1] = ml.x;
    __syncthreads();
    logit = q_k[0];
    first = q_k[1];
    m = logit;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) m = fmaxf(m, wave_m[w]);
    a = fast_exp2(ml.x - m);                            // a range without rows: 0
    l = wave_sum(ml.x == -INFINITY ? 0.0f : ml.y * a);
    wgt[tid] = tid < s.n_splits ? a : 0.0f;
    if (tid < AHEAD * GROUPS) wgt[NT + tid] = 0.0f;
    if (lane == 0) wave_l[wave] = l;
    __syncthreads();
    w_new = fast_exp2(logit - m);
    l = w_new;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) l += wave_l[w];
  }

  // (outputs of a range without rows are whatever memory held: skipped, not multiplied by zero)
  float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int sp0 = 0; sp0 < s.n_splits; sp0 += AHEAD * GROUPS) {          // (uniform: the weights come from other lanes)
    const int sp = sp0 + grp;
    float w[AHEAD];
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) {
      const int at = sp + u * GROUPS;
      if constexpr (FEW) {
        w[u] = __shfl(a, at);                          // (by all lanes)
        if (at >= s.n_splits) w[u] = 0.0f;
      } else {
        w[u] = wgt[at];
      }
    }
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) {
      const bool counts = w[u] != 0.0f;
      o.x = counts ? fmaf(pre[u].x, w[u], o.x) : o.x; o.y = counts ? fmaf(pre[u].y, w[u], o.y) : o.y;
      o.z = counts ? fmaf(pre[u].z, w[u], o.z) : o.z; o.w = counts ? fmaf(pre[u].w, w[u], o.w) : o.w;
    }
    if (sp0 + AHEAD * GROUPS < s.n_splits) request();
  }
  *(float4 *)&acc_s[grp][col * 4] = o;
  // (nobody reads the new row from the caches in this launch)
  const bool fits = n >= 0 && n < s.capacity;
  if (appends && fits)
    *(uint4 *)((tid < LPK ? k_cache : v_cache) + ((int64_t)b * s.sb + (int64_t)h * s.sh + (int64_t)n * s.st + tid % LPK * E)) = row_piece;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < (D + NT - 1) / NT; ++k) {
    const int c = tid + k * NT;
    if (c >= D) break;
    float x = 0.0f;
#pragma unroll
    for (int i = 0; i < GROUPS; ++i) x += acc_s[i][c];
    x = fmaf(w_new, Piece<T>::value(&v_piece[k]), x) / l;
    out[hq * D + c] = first != first ? first : x;
  }
  if (g == 0 && tid == 0 && !s.keep_count && fits) n_valid[bh] = n + 1;
}

template <typename T, int D, int G>
static void launch_partial_g(const DecodeShape &s, dim3 grid, const void *q, const void *kc, const void *vc,
                             const int32_t *n_valid, float *part, hipStream_t stream) {
  // Where a model's caches exceed the memory-side cache, no row is found there at the next token, and the values, as both
  // caches in fp32, are best streamed.  How many layers there are and (n_valid is on the device) how many rows the library
  // cannot know: the line is that of 32 layers of full caches.  Us a layer with plain loads / with values streamed, where the rows
  // were in that cache (one to four layers, again and again) and where they were not (32 layers, or three sets of 8): 8 MB a layer
  // 9.8 / 10.2 and 10.1-10.6 / 10.3-10.6; 17 MB 10.3-10.9 / 10.5-11.1 and 11.9-12.1 / 11.2-11.8; 34 MB 13.5 / 13.5 and
  // 14.4 / 14.2; 67 MB 19.2 / 19.4 and 21.7 / 20.9; eleven sequences of mixed lengths, f16 (38 MB) 16.1 / 16.3 and 17.9 / 16.8; eight in
  // fp32 (271 MB) 59.5 / 53.4.
  // Keys of 16-bit caches are read in operand layout, 64 bytes of a row at a time, and a streamed line may be gone when
  // its other half is asked for: they stream only where a layer's caches by themselves exceed the memory-side cache.  Full caches gain
  // there, mixed ones, which leave more of the chip waiting for single loads, lose some of it again.  64 sequences of 4128 rows (1.1 GB
  // a layer): 193 us plain, 173 with values streamed, 170 with both; 256 of 300 rows (556 MB of capacity) 73, 70 and 63; 48 of 300 to 4000
  // rows (294 MB of 789) 80, 75 and 80; of the eleven sequences above: 17.9, 16.8 and 17.5.
  const int64_t bytes = 2 * (int64_t)s.B * s.Hkv * s.capacity * D * (int64_t)sizeof(T);
  const int stream_level = bytes > MEMORY_CACHE_BYTES ? 2 : bytes > MEMORY_CACHE_BYTES / 32 ? 1 : 0;
#define WKV_PARTIAL(KERNEL, E, NT) \
  hipLaunchKernelGGL(KERNEL, grid, dim3(NT), 0, stream, s, (const E *)q, (const E *)kc, (const E *)vc, n_valid, part)
  if constexpr (sizeof(T) == 2) {   // bf16 / fp16: scores on the matrix pipe
    constexpr bool F16 = !__is_same(T, uint16_t);
    // Ranges of 128 rows by eight waves with a block each instead of four with two: half the arithmetic in a row, no state before the block, twice the
    // states to merge; the device holds 1024 workgroups of either kind (four waves of five heads and more: 768).  us a layer with four / eight waves,
    // 128 channels: 32q/8kv heads, one sequence of 4128 rows 8.77 / 8.52, 6000 10.15 / 10.19, two of 4128 11.26 / 11.02, three 13.59 / 13.30, eight of 1000 10.90 / 10.74; three of
    // 1000 to 3000 11.04 / 11.25, four of 500 to 3000 11.01 / 11.23; 32q/16kv, one of 4128 10.70 / 10.51; 32q/32kv, six of 100 to 700 10.68 / 10.75.  The line is from kernels
    // whose single block had a state, for which more heads and 64 channels lost by eight waves.  On these: 40q/8kv, one of 4128 9.22 / 8.88; 12q/2kv, eleven mixed 11.67 / 11.50;
    // 28q/4kv, eleven mixed 14.23 / 15.27; 64q/8kv, one of 4128 9.97 / 9.58, three of 1000 to 3000 13.02 / 11.49, eight of 1000 12.35 / 11.80; 64 channels, 32q/8kv, one of 4128 7.82 /
    // 7.75, two 8.88 / 8.64, three of 1000 to 3000 9.15 / 8.84; 64q/8kv, three of 1000 to 3000 10.90 / 9.44.
    constexpr bool WIDE = D == 128 && G <= 4;
    if constexpr (WIDE)
      if (s.chunk <= WIDE_THREADS / 64 * 16 && stream_level < 2) {
        if (stream_level == 1) WKV_PARTIAL((decode_partial_mfma_kernel<D, G, F16, 1, WIDE_THREADS>), uint16_t, WIDE_THREADS);
        else WKV_PARTIAL((decode_partial_mfma_kernel<D, G, F16, 0, WIDE_THREADS>), uint16_t, WIDE_THREADS);
        return;
      }
    // (longer ranges than those are of caches that stream: as many as there can be of a cache, 128 rows each, are 16 MB)
    static_assert(!WIDE || (int64_t)DEC_MAX_SPLITS * 128 * 2 * D * (int64_t)sizeof(T) > MEMORY_CACHE_BYTES / 32, "plain loads");
    if (stream_level == 2) WKV_PARTIAL((decode_partial_mfma_kernel<D, G, F16, 2, DEC_THREADS>), uint16_t, DEC_THREADS);
    else if (WIDE || stream_level == 1) WKV_PARTIAL((decode_partial_mfma_kernel<D, G, F16, 1, DEC_THREADS>), uint16_t, DEC_THREADS);
    else if constexpr (!WIDE) WKV_PARTIAL((decode_partial_mfma_kernel<D, G, F16, 0, DEC_THREADS>), uint16_t, DEC_THREADS);
  } else {
    if (stream_level) WKV_PARTIAL((decode_partial_kernel<T, D, G, true>), T, DEC_THREADS);
    else WKV_PARTIAL((decode_partial_kernel<T, D, G, false>), T, DEC_THREADS);
  }
#undef WKV_PARTIAL
}

template <typename T, int D>
static hipError_t launch_decode_t(const DecodeShape &s, const void *q, const void *kn, const void *vn, void *kc, void *vc,
                                  int32_t *n_valid, float *out, float *part, hipStream_t stream) {
  const dim3 grid(s.B * s.Hkv, s.n_splits);
#define WKV_DEC_CASE(GG) \
  case GG: launch_partial_g<T, D, GG>(s, grid, q, kc, vc, n_valid, part, stream); break;
  switch (s.G) {
    WKV_DEC_CASE(1) WKV_DEC_CASE(2) WKV_DEC_CASE(3) WKV_DEC_CASE(4) WKV_DEC_CASE(5) WKV_DEC_CASE(6)
    WKV_DEC_CASE(7) WKV_DEC_CASE(8)
    default: return hipErrorInvalidValue;
  }
#undef WKV_DEC_CASE
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // a wave reads eight ranges (16 at 64 channels) in its first round trip: with no more than that, one wave a head
  static_assert(DEC_MAX_SPLITS <= DEC_THREADS, "one thread per range");
  const dim3 heads(s.B * s.Hkv, s.G);
#define WKV_COMBINE(NT) \
  hipLaunchKernelGGL((decode_combine_kernel<T, D, NT>), heads, dim3(NT), 0, stream, s, (const T *)q, (const T *)kn, (const T *)vn, \
                     (T *)kc, (T *)vc, (const float *)part, n_valid, out)
  if (s.n_splits <= 1024 / D) WKV_COMBINE(64);
  else WKV_COMBINE(DEC_THREADS);
#undef WKV_COMBINE
  return hipGetLastError();
}

hipError_t launch_decode(const DecodeShape &s, const void *q_new, const void *k_new, const void *v_new, void *k_cache,
                         void *v_cache, int32_t *n_valid, float *out, float *part, hipStream_t stream) {
#define WKV_DEC_TYPE(TT) \
  return s.d == 128 ? launch_decode_t<TT, 128>(s, q_new, k_new, v_new, k_cache, v_cache, n_valid, out, part, stream) \
                    : launch_decode_t<TT, 64>(s, q_new, k_new, v_new, k_cache, v_cache, n_valid, out, part, stream);
  if (s.dtype == WKV_BF16) WKV_DEC_TYPE(uint16_t)
  if (s.dtype == WKV_F16) WKV_DEC_TYPE(half_t)
  WKV_DEC_TYPE(float)
#undef WKV_DEC_TYPE
}

constexpr int MAX_DEVICES = 64;
static std::atomic<void *> scratch_ptr[MAX_DEVICES];
static std::mutex scratch_mutex;

hipError_t launch_decode_static(const DecodeShape &s, const void *q_new, const void *k_new, const void *v_new,
                                void *k_cache, void *v_cache, int32_t *n_valid, float *out, hipStream_t stream) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
  void *p = scratch_ptr[dev].load(std::memory_order_acquire);
  if (!p) {                                 // first call on this device (which is the current one)
    std::lock_guard<std::mutex> lock(scratch_mutex);
    p = scratch_ptr[dev].load(std::memory_order_relaxed);
    if (!p) {
      e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
      if (e != hipSuccess) return e;
      if (!p) return hipErrorInvalidSymbol;
      scratch_ptr[dev].store(p, std::memory_order_release);
    }
  }
  // every partial result a combine reads is written by the partial kernel of the same call:
  // nothing in the array has to be cleared
  return launch_decode(s, q_new, k_new, v_new, k_cache, v_cache, n_valid, out, (float *)p, stream);
}

}  // namespace wkv
