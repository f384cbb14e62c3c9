// Internal declarations shared by the translation units of libwkv (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "wkv.h"

namespace wkv {

// The chip's memory-side cache.
constexpr int64_t MEMORY_CACHE_BYTES = (int64_t)256 << 20;

// n / d == divide(n, division_magic(d)) while n * d < 2^32.
inline uint32_t division_magic(int32_t d) { return d == 1 ? 0u : 0xffffffffu / (uint32_t)d + 1u; }
__host__ __device__ inline int32_t divide(uint32_t n, uint32_t magic) {
  return (int32_t)(magic == 0u ? n : (uint32_t)((uint64_t)n * magic >> 32));
}

inline int64_t elem_bytes(int32_t dtype) { return dtype == WKV_F32 ? 4 : 2; }

// Per-sequence parameters, passed to kernels by value inside the kernel argument block so
// that no host-to-device copy (and no allocation) is ever needed for metadata.
struct SeqParam {
  int32_t L;    // prefix length
  int32_t win;  // review-window size (omega)
  int32_t p;    // top-p, already clamped to [1, win]
  int32_t k;    // windows to keep
  uint32_t win_magic;   // division_magic(win): token numbers are divided by window sizes by multiplication
};
struct BatchParams {
  SeqParam seq[WKV_MAX_BATCH];
};

// Per-group device pointers of the scored layer.
struct GroupPtrs {
  const void *q[WKV_MAX_GROUPS];
  const void *k[WKV_MAX_GROUPS];
  const float *lse[WKV_MAX_GROUPS];   // caller's softmax log-sum-exp of the observation rows, or all null
};

// Per-layer device pointers for the gather.
struct LayerPtrs {
  const void *k_in[WKV_MAX_LAYERS];
  const void *v_in[WKV_MAX_LAYERS];
  void *k_out[WKV_MAX_LAYERS];
  void *v_out[WKV_MAX_LAYERS];
};

// Windows to keep per (group, sequence) when the groups have budgets of their own (Section
// 2.2.3); index g * B + b.  Not in use: every group keeps SeqParam::k windows.
constexpr int32_t MAX_GROUP_K = 1024;
struct GroupK {
  int32_t in_use;
  uint16_t k[MAX_GROUP_K];
};

// The same for a call small enough for one launch of selection and gather: everything its kernel needs besides
// Shape, in a block a quarter of the size.
constexpr int32_t SMALL_BATCH = 8, SMALL_GROUPS = 8, SMALL_LAYERS = 8;
constexpr int32_t SMALL_WORKGROUPS = 512;         // what the device holds at once
constexpr int32_t SMALL_WINDOWS = 8192;
struct SmallJob {
  SeqParam seq[SMALL_BATCH];
  int32_t k[SMALL_GROUPS * SMALL_BATCH];        // windows to keep, index g * B + b
  const void *in[SMALL_LAYERS][2];
  void *out[SMALL_LAYERS][2];
  int32_t gamma, esize;
  uint32_t gamma_magic;       // division_magic of gamma
};

// Problem shape as the kernels see it.
struct Shape {
  int32_t B, Hq, Hkv, d, w_obs, G;
  int32_t M;          // G * w_obs softmax rows per KV head
  int32_t t_stride, nw_max, k_max, nkeep_max;
  int32_t dtype;
  int32_t fill_padding;   // gather: zero the compact-cache rows past n_keep
  uint32_t w_magic;   // r / w_obs == r * w_magic >> 16 for row numbers r < 256
  uint32_t hkv_magic; // division_magic(Hkv)
  float c1;           // logit scale * log2(e): logits are handled in base-2 units
  int64_t q_sb, q_sh, q_st;
  int64_t kv_sb, kv_sh, kv_st;
  int64_t o_sb, o_sh, o_st;
};

inline SmallJob small_job(const Shape &s, const BatchParams &bp, const GroupK &gk, const LayerPtrs &lp, int32_t n_groups, int32_t gamma) {
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
  return job;
}

// How the score passes split the key axis into workgroup chunks.
// Token scores that the score pass stages in LDS before it pools them or writes them out.
constexpr int32_t SCORE_SEG = 2048;

// One pass: sequence b of a row takes the workgroups first[b] .. first[b+1]-1, chunk[b] keys each (the last one what
// is left).  At least one each, so that the padding of its outputs has an owner.
constexpr int32_t CHUNK_UNIT = 64;                // a tile of 16 keys for every key slot of a workgroup
struct PassPlan {
  int32_t first[WKV_MAX_BATCH + 1];
  uint8_t chunk[WKV_MAX_BATCH];                   // in units of CHUNK_UNIT keys
};
struct ScorePlan {
  PassPlan pass[2];            // statistics, scores
  int32_t n_chunks1;           // most workgroups of a sequence in the statistics pass
  int32_t m_pad;               // rows padded to a multiple of 16
  int32_t tile;                // rows of a tile: 32 or 16 (fp32: 16)
  bool nontemporal;            // a long stream: the key loads put nothing into the memory-side cache
  bool own_rings;              // with two row groups of 16-bit inputs every wave fetches its key tiles itself
  bool fold_in_pass2;          // pass 2 folds the pass-1 partials itself (few chunks per row)
};

// What the score kernels read of their arguments, laid out for few dependent scalar loads: a workgroup's first request waits for every one of
// them (a cold one takes 0.2 to 0.3 us), so the first trip fetches what lies at fixed places, `ends` of the first sequences among
// it, and the second the one record of the workgroup's sequence and the pointers of its group.  With five trips in the first pass and eight in
// the second, 1.4 and 1.8 us to the first key request; a call over 512 tokens of two KV heads 17.95 -> 16.25 us so, 4096 tokens 24.3 -> 23.7.
struct ScoreSeq {
  int32_t L, first, n_parts;   // prefix length, first workgroup of this pass, workgroups of the statistics pass
  uint32_t packed;             // chunk in CHUNK_UNITs | win << 8 | p << 16
  uint32_t win_magic;
  int32_t last;                // last workgroup of this pass
};
constexpr int32_t ENDS_AT_ONCE = 8;
struct ScoreArgs {
  int32_t ends[WKV_MAX_BATCH]; // first workgroup after the sequence; INT32_MAX past the last sequence
  ScoreSeq seq[WKV_MAX_BATCH];
  GroupPtrs gp;
  int32_t m_pad, n_chunks1, fold;       // fold: this pass folds the partials of the statistics pass
  uint32_t hkv_magic;
  int32_t row_bits, last_x, last_y, last_z, items;    // the launch grid (see ScoreGrid) and the workgroups of a row
};
// Which row (group, KV head) and which of its workgroups a workgroup of the score passes is.  Workgroup numbers are dealt round-robin to
// the 8 XCDs, each with an L2 of its own: where the rows of a sequence allow, all workgroups of a row are on one XCD (of two to seven rows on a
// share of them), so that its queries and partials come into one L2 instead of all eight.  Then x of the grid is the XCD, y and z the
// rows and the row's workgroups: 2^row_bits rows in x, 8 >> row_bits workgroups of each.  Only where every XCD gets its equal share so;
// else, and with more rows than a grid has in y or `divide` takes (65535), x is the workgroup, y the KV head and z the group.  Plain / by XCD: 8 heads of 4096 tokens 23.7 / 22.6 us, of 16384 43.4 / 42.1, in fp32 stage by
// stage 61.2 / 58.7; a mixed batch of 8 in 8 groups 1902 / 1877; ragged f16 with 224 rows a head in 4 groups 68.8 / 67.0; 32768 tokens in 8 groups, whose
// queries are 1/16 of the keys, the same.
struct ScoreGrid {
  int32_t x, y, z, row_bits;
};
inline ScoreGrid score_grid(int32_t heads, int32_t groups, int32_t items) {
  const int64_t rows = (int64_t)heads * groups;
  int32_t bits = 0;
  while (bits < 3 && rows % (2 << bits) == 0) ++bits;
  const int32_t per = 8 >> bits;        // workgroups of a row side by side
  if (bits == 0 || rows > 65535 || items > 65535 || (items % per != 0 && rows != 1 << bits)) return {items, heads, groups, 0};
  return {8, (int32_t)(rows >> bits), (items + per - 1) / per, bits};
}
struct ScoreItem {
  int32_t group, head, item;   // item: past the row's last one for a few workgroups where 8 >> row_bits does not divide them
  __host__ __device__ ScoreItem(int32_t x, int32_t y, int32_t z, int32_t row_bits, int32_t heads, uint32_t heads_magic) {
    const int32_t row = (x & ((1 << row_bits) - 1)) + (y << row_bits), of = divide(row, heads_magic);
    group = row_bits ? of : z;
    head = row_bits ? row - of * heads : y;
    item = row_bits ? (z << (3 - row_bits)) + (x >> row_bits) : x;
  }
};

// ---- single-read score kernel ("resident keys") ----------------------------------------------------
constexpr int32_t RK_SLICE = 256;        // keys a workgroup holds in registers between its two phases
// Synchronisation words in the workspace (uint32, cleared at the start of every call): a few
// global ones, then RK_SYNC_WORDS per (group, sequence, KV head) row.
constexpr int32_t RK_GLOBAL_WORDS = 4;
constexpr int32_t RK_FAIL = 0;           // global: a bounded wait ran out; the two-pass kernels redo the scores
constexpr int32_t RK_SYNC_WORDS = 4;
constexpr int32_t RK_ARRIVED = 0;        // per row: slices whose phase-1 partials are in the workspace
constexpr int32_t RK_READY = 1;          // per row: the normalisers of the row are published

struct ResidentPlan {
  int32_t use;                           // the call takes the single-read kernel
  int32_t n_items, items_per_group;      // slices in the call / in one group
  int32_t nsl_max;                       // most slices of any row
  int32_t m_pad;
  int32_t spin_limit;                    // polls before a waiting workgroup gives up
  // The batched call's score kernel pools (Eq. 3-4).  The two-pass kernels always can; slices of the
  // single-read kernel hold whole windows only if every window size divides their length.
  int32_t pools;
};

struct Workspace {
  float2 *partials;   // [n_groups][B][Hkv][n_chunks1][m_pad] (running max, sum) in base 2
  float *lse;         // [n_groups][B][Hkv][m_pad] base-2 log-sum-exp of every softmax row
  float *t;           // [n_groups][B][Hkv][t_stride]
  float *s;           // [n_groups][B][Hkv][nw_max]
  unsigned long long *rk_partials;   // [rows][nsl_max][m_pad] (m, z) of every slice (single-read kernel)
  uint32_t *rk_sync;                 // [RK_GLOBAL_WORDS + rows * RK_SYNC_WORDS]
  size_t t_offset, s_offset;   // byte offsets of t and s from the base
  size_t bytes;
};

// Selection and gather in one launch?  Up to 40 MB of compact cache, 60 MB of one sequence: the workgroups that the device holds at once
// (the selection is repeated in each) keep fewer rows in flight than the gather's own launch, which costs more than
// the launch saves from there on; sequences of their own lengths leave some of them idle sooner.  Whole calls in one launch / in two, one sequence:
// 50 MB 53.2 / 54.5 and 52.8 / 54.0 us, 58 MB 58.7 / 59.6, 68 MB 66.4 / 67.0 and 56.3 / 54.9; batches of mixed lengths: 59 MB 77.0 / 74.4, 75 MB
// 59.9 / 58.2; 34 MB 45.9 / 47.3, 17 MB 33.7 / 35.5 (either).
constexpr int64_t SMALL_BYTES = 40 << 20, SMALL_BYTES_ONE = 60 << 20;
inline bool selects_and_gathers(const Shape &s, int32_t n_groups, int32_t gamma) {
  const int64_t pairs = (int64_t)2 * n_groups * gamma * s.B * s.Hkv;
  return s.B <= SMALL_BATCH && n_groups <= SMALL_GROUPS && n_groups * gamma <= SMALL_LAYERS && s.nw_max <= SMALL_WINDOWS &&
         pairs <= SMALL_WORKGROUPS && pairs * s.nkeep_max * s.d * elem_bytes(s.dtype) <= (s.B == 1 ? SMALL_BYTES_ONE : SMALL_BYTES);
}

// The whole call in one launch?  Every workgroup scores a whole row by itself (wkv_short.hip), which takes the place of the two passes where a row
// is short, and as many workgroups as (row, tensor) pairs do so side by side: one a compute unit.  (t_stride + w_obs is the room of the caches: a short
// prompt in caches with room for more than the rule takes goes by the passes.)
constexpr int32_t SHORT_WORKGROUPS = 256;
// Key tiles of 16 that a wave of eight holds, at most, by the row tiles of 16 (1, 2, 4 or 8): four are 512 keys.  0: not in one launch.  16-bit types take what
// fits the registers; all of it gains, 16 to 128 rows a KV head, 200 to 1000 keys: 0.48 to 0.84 of the time of the passes with the merged selection
// and gather, 1, 2, 4 and 8 sequences alike.  fp32 is a matrix product of 1/16 the rate, done by every workgroup: 16 rows of 64 channels 0.50 to 0.77,
// 32 rows 0.64, 16 rows of 128 channels 0.61; 32 rows of 1000 keys would take 1.39, 64 rows of 512 keys 1.24, 32 rows of 128 channels 1.27.
// With handed-over normalisers (given) there is one pass less to replace: 0.75 to 0.91 of the time of the launches (medians of some 20 calls each) where it is taken; it
// would be 1.10 with 16-bit types, 64 channels, 33 to 64 rows of 1024 keys, 1.08 and 1.14 with 65 to 128 rows of 64 and 128 channels, 1.04 with 128 channels, 17 to
// 32 rows of 1024 keys; fp32, 64 channels, 16 rows of 1024 keys 1.10, 32 rows 1.01, 128 channels 1.02.
constexpr int32_t short_key_tiles(int32_t d, int32_t esize, int32_t row_tiles, bool given = false) {
  if (given) return esize == 4 ? (d == 64 && row_tiles == 1 ? 4 : 0) : row_tiles == 1 || (d == 64 && row_tiles == 2) ? 8 : row_tiles <= 4 ? 4 : 0;
  if (esize == 4) return row_tiles == 1 ? (d == 64 ? 8 : 4) : d == 64 && row_tiles == 2 ? 4 : 0;
  return row_tiles <= 2 || (d == 64 && row_tiles == 4) ? 8 : 4;
}
inline int32_t short_row_tiles(const Shape &s) { return s.M <= 16 ? 1 : s.M <= 32 ? 2 : s.M <= 64 ? 4 : s.M <= 128 ? 8 : 0; }
// Windows of more than 64 tokens have their tokens ranked by a loop over the window, one token a thread and then the next; every workgroup of a row does it here, those of
// the score pass share it.  In sequences of more than SHORT_TOKENS, two tokens a thread, that makes 1.05 of the time of the passes, 1.31 with handed-over
// normalisers (all other calls 0.72 and 0.86; up to that 1.01 and 1.05 at most).
constexpr int32_t SHORT_TOKENS = 512;
inline bool whole_call_in_one(const Shape &s, const BatchParams &bp, int32_t n_groups, int32_t gamma, bool given) {
  const int32_t tiles = short_row_tiles(s);
  bool in = tiles > 0 && s.t_stride + s.w_obs <= 128 * short_key_tiles(s.d, (int32_t)elem_bytes(s.dtype), tiles, given) && selects_and_gathers(s, n_groups, gamma) &&
            2 * n_groups * gamma * s.B * s.Hkv <= SHORT_WORKGROUPS;
  for (int32_t b = 0; in && b < s.B; ++b) in = bp.seq[b].win <= 64 || bp.seq[b].L - s.w_obs <= SHORT_TOKENS;
  return in;
}

// Workgroups over the rows of a compact cache, two pieces of `rows` rows each, `apart` pieces from one to the other; the ones from
// `last` on share what is left, last_apart pieces apart: all but the very last hold two pieces.
struct GatherGrid {
  int32_t workgroups, last, last_apart;
};
inline GatherGrid gather_grid(int32_t nkeep_max, int32_t rows, int32_t apart) {
  const int32_t pieces = (nkeep_max + rows - 1) / rows, last = pieces / (2 * apart) * apart, last_apart = (pieces % (2 * apart) + 1) / 2;
  return {last + last_apart, last, last_apart};
}

// Threads of a gather's workgroup: single waves, unless much of the compact cache lies past the sequences' budgets; the workgroups
// there zero it or find nothing to do, and each of them costs a start.  By 256 threads / one wave / as chosen, batches of 4 to 16, us:
//   past the budgets left alone, budgets of less than 0.4 of the room in the mean: 128 threads.  0.16 25.5 / 34.8 / 22.0, 0.21 21.1 / 26.2 / 19.1, 0.29
//   15.4 / 16.1 / 14.0, 0.33 20.2 / 22.7 / 19.7; from there on 0.41 222.7 / 212.7 / 216.2, 0.48 162.1 / 129.7 / 132.4, 0.56 162.8 / 146.0 / 147.7.
//   zeroed, less than 3/8, rows of 128 bytes less than a third: 256 threads.  0.15 121.0 / 134.9, 0.22 217 / 230, 0.25 70.1 / 71.6, 0.32 66.8 / 73.8, 0.36
//   57.0 / 61.9; from there on 0.46 213.5 / 192.5, 0.54 217.4 / 199.6; rows of 128 bytes 0.24 53.0 / 55.4, 0.36 85.7 / 66.4, 0.38 156.4 / 124.3.
inline int32_t gather_threads(const Shape &s, const BatchParams &bp) {
  int64_t kept = 0;
  for (int32_t b = 0; b < s.B; ++b) kept += bp.seq[b].k * bp.seq[b].win + s.w_obs;
  const int64_t room = (int64_t)s.B * s.nkeep_max;
  if (s.fill_padding) return (s.d * elem_bytes(s.dtype) > 128 ? 8 * kept < 3 * room : 3 * kept < room) ? 256 : 64;
  return 5 * kept < 2 * room ? 128 : 64;
}

// ---- host-side helpers (wkv_host.cpp) ---------------------------------------------------
void set_error(const char *fmt, ...);
wkv_status validate(const wkv_problem *p, wkv_dims *dims);
void fill_shape(const wkv_problem *p, const wkv_dims &dims, Shape *s, BatchParams *bp);
ScorePlan plan_score(const Shape &s, const BatchParams &bp, int32_t n_groups);
void fill_score_args(const Shape &s, const BatchParams &bp, const ScorePlan &plan, const GroupPtrs &gp, int32_t n_groups, int32_t pass,
                     bool fold, ScoreArgs *a, ScoreGrid *grid);
ResidentPlan plan_resident(const Shape &s, const BatchParams &bp, const ScorePlan &plan, int32_t n_groups, int32_t flags);
Workspace carve_workspace(const Shape &s, const ScorePlan &plan, const ResidentPlan &rp, int32_t n_groups, void *base);

// ---- launchers (one per kernel family) ----------------------------------------------------
// All return hipSuccess or the launch error. Pointers are device pointers unless noted.
// `mid`, if not null, is recorded between the stats pass and the score pass.
// `only_if`, if not null, points to a device word: the kernels return at once unless it is non-zero.
hipError_t launch_score(const Shape &s, const BatchParams &bp, const ScorePlan &plan,
                        const GroupPtrs &gp, int32_t n_groups, bool have_lse, float2 *partials, float *lse,
                        float *t_out, float *s_pool, hipStream_t stream, hipEvent_t mid = nullptr,
                        const uint32_t *only_if = nullptr);
// Clears the synchronisation words, then the single-read score kernel (Eq. 1-2, pooled if s_pool).
hipError_t launch_resident(const Shape &s, const BatchParams &bp, const ResidentPlan &rp, const GroupPtrs &gp,
                           int32_t n_groups, unsigned long long *partials, float *lse, uint32_t *sync, float *t_out,
                           float *s_pool, hipStream_t stream);
hipError_t launch_pool(const Shape &s, const BatchParams &bp, int32_t n_groups, const float *t,
                       float *s_out, hipStream_t stream);
hipError_t launch_topk(const Shape &s, const BatchParams &bp, const GroupK &gk, int32_t n_groups, const float *sc,
                       int32_t *win_idx, int32_t *tok_idx, int32_t *n_keep, hipStream_t stream);
// The same, and the rows of the layers `lp`, gamma per group, in one launch (see selects_and_gathers).
hipError_t launch_select_gather(const Shape &s, const BatchParams &bp, const GroupK &gk, const LayerPtrs &lp, int32_t n_groups, int32_t gamma,
                                const float *sc, int32_t *win_idx, int32_t *tok_idx, int32_t *n_keep, hipStream_t stream);
// Scores, selection and the rows in one launch (see whole_call_in_one).
hipError_t launch_short(const Shape &s, const BatchParams &bp, const GroupK &gk, const GroupPtrs &gp, const LayerPtrs &lp, int32_t n_groups, int32_t gamma,
                        float *sc, int32_t *win_idx, int32_t *tok_idx, int32_t *n_keep, hipStream_t stream);
hipError_t launch_gather(const Shape &s, const BatchParams &bp, const LayerPtrs &lp, int32_t n_layers, int32_t gamma,
                         const int32_t *tok_idx, const int32_t *n_keep, hipStream_t stream);

hipError_t launch_jaccard(const Shape &s, int32_t n_sets, const int32_t *tok_idx, const int32_t *n_keep, float *out,
                          hipStream_t stream);

// ---- decode over the compact cache --------------------------------------------------------
constexpr int32_t DEC_MAX_SPLITS = 256;   // key ranges per (sequence, KV head): one per thread of the combine kernel

struct DecodeShape {
  int32_t B, Hq, Hkv, d, G, dtype;
  int32_t capacity;          // token rows per (sequence, KV head) in the caches
  int32_t n_splits, chunk;   // key ranges per (sequence, KV head) and their length
  int32_t keep_count;        // leave n_valid as it is (the caller advances it after the group's last layer)
  float c1;                  // scale * log2(e)
  int64_t sb, sh, st;        // cache strides in elements
  uint32_t heads_magic, kv_magic;      // division_magic of the heads (B * Hkv) and of Hkv
  uint32_t stats_at;         // bytes from the partial outputs to their statistics
};
// Which key range workgroup (x, y) of the partial kernel's grid (heads, ranges) takes.  Range by range: the first ranges of all caches
// go first, the ones that many caches of a mixed batch do not reach last.  The heads start nine further on in every range, so
// that the ranges of one cache fall on other XCDs (workgroup numbers are dealt to the 8 of them in turn) and compute units each time.
// Head by head, with 2, 4, 8 or 24 ranges, the first ranges of all heads share an XCD and those of the late ones idle: 48 sequences of 300 to
// 4000 rows, 32q/8kv, 128 channels 95 us a layer and 67 so, 11 with 32 KV heads 94 and 73; without the nine, 16 of up to 32000 rows
// and 4 KV heads 108 and 79.  Equal lengths 1 to 2 % faster so, but 8 sequences of 32768 rows 177 us head by head and 182 so.
// (magic: division_magic(heads); the compiler's divisions by two run-time numbers are a good part of the code that stands
// before the first load.  Exact, as x < heads and 9 * y < 9 * 1536 / heads.)
struct RangeOf {
  int32_t head, range;
  __host__ __device__ RangeOf(int32_t x, int32_t y, int32_t heads, uint32_t magic)
      : head(x + 9 * y - divide((uint32_t)(x + 9 * y), magic) * heads), range(y) {}
};
struct Decode {
  DecodeShape shape;
  size_t ws_bytes;           // partial results: [B*Hkv][n_splits][G] times d + 2 floats
};
wkv_status validate_decode(const wkv_decode_shape *p, Decode *out);
hipError_t launch_decode(const DecodeShape &s, const void *q_new, const void *k_new, const void *v_new, void *k_cache,
                         void *v_cache, int32_t *n_valid, float *out, float *part, hipStream_t stream);

// The same launches with the partial results in the library's own static scratch array of the
// current device (no workspace argument; the caller has checked that the shape fits).
hipError_t launch_decode_static(const DecodeShape &s, const void *q_new, const void *k_new, const void *v_new,
                                void *k_cache, void *v_cache, int32_t *n_valid, float *out, hipStream_t stream);

}  // namespace wkv
