// Host-side logic of libwkv: argument validation, derived sizes, launch planning and the
// scalar helpers.  Nothing in this file touches the GPU, so all of it is testable on a
// machine without one.
#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>

#include "wkv_internal.h"

namespace wkv {

static thread_local char g_err[512] = "";

void set_error(const char *fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
}

static inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

wkv_status validate(const wkv_problem *p, wkv_dims *dims) {
  g_err[0] = 0;
  if (!p) { set_error("problem is NULL"); return WKV_ERR_INVALID_ARG; }
  if (!p->seq_len || !p->win || !p->top_p || !p->k_windows) {
    set_error("seq_len / win / top_p / k_windows must be non-NULL host arrays");
    return WKV_ERR_INVALID_ARG;
  }
  if (p->batch < 1) { set_error("batch must be >= 1 (got %d)", p->batch); return WKV_ERR_INVALID_ARG; }
  if (p->batch > WKV_MAX_BATCH) {
    set_error("batch %d exceeds WKV_MAX_BATCH=%d; split the call", p->batch, WKV_MAX_BATCH);
    return WKV_ERR_UNSUPPORTED;
  }
  if (p->n_kv_heads < 1 || p->n_q_heads < 1 || p->n_q_heads % p->n_kv_heads != 0) {
    set_error("n_q_heads (%d) must be a positive multiple of n_kv_heads (%d)", p->n_q_heads, p->n_kv_heads);
    return WKV_ERR_INVALID_ARG;
  }
  if ((int64_t)p->batch * p->n_kv_heads > 65535) {
    set_error("batch * n_kv_heads exceeds 65535 (launch grid limit); split the call"); return WKV_ERR_UNSUPPORTED;
  }
  if (p->dtype != WKV_F32 && p->dtype != WKV_BF16 && p->dtype != WKV_F16) {
    set_error("unknown dtype %d", p->dtype); return WKV_ERR_INVALID_ARG;
  }
  if (p->head_dim != 64 && p->head_dim != 128) {
    set_error("head_dim %d is not supported (64 or 128)", p->head_dim); return WKV_ERR_UNSUPPORTED;
  }
  if (p->flags & ~(WKV_KEEP_PADDING | WKV_SCORE_TWO_PASS | WKV_SCORE_SINGLE_READ | WKV_DEBUG_WAIT_GIVES_UP)) {
    set_error("unknown bits in flags (0x%x)", p->flags); return WKV_ERR_INVALID_ARG;
  }
  if ((p->flags & WKV_SCORE_TWO_PASS) && (p->flags & WKV_SCORE_SINGLE_READ)) {
    set_error("WKV_SCORE_TWO_PASS and WKV_SCORE_SINGLE_READ exclude each other"); return WKV_ERR_INVALID_ARG;
  }
  if (p->w_obs < 1) { set_error("w_obs must be >= 1"); return WKV_ERR_INVALID_ARG; }
  const int64_t G = p->n_q_heads / p->n_kv_heads;
  if (G * p->w_obs > WKV_MAX_OBS_ROWS) {
    set_error("(Hq/Hkv)*w_obs = %lld exceeds WKV_MAX_OBS_ROWS=%d", (long long)(G * p->w_obs), WKV_MAX_OBS_ROWS);
    return WKV_ERR_UNSUPPORTED;
  }
  if (p->max_seq_len < p->w_obs) { set_error("max_seq_len < w_obs"); return WKV_ERR_INVALID_ARG; }
  if (!(p->scale >= 0.0f) || std::isinf(p->scale)) {
    set_error("scale must be finite and >= 0 (0 selects 1/sqrt(head_dim))"); return WKV_ERR_INVALID_ARG;
  }
  const int64_t d = p->head_dim;
  if (p->q_stride_t < d || p->kv_stride_t < d || p->out_stride_t < d) {
    set_error("token strides must be >= head_dim"); return WKV_ERR_INVALID_ARG;
  }
  // 16-byte vector loads: every row start must be 16-byte aligned relative to the base.
  const int64_t vec = 16 / elem_bytes(p->dtype);
  const int64_t strides[9] = {p->q_stride_b, p->q_stride_h, p->q_stride_t, p->kv_stride_b, p->kv_stride_h,
                              p->kv_stride_t, p->out_stride_b, p->out_stride_h, p->out_stride_t};
  for (int i = 0; i < 9; ++i) {
    if (strides[i] < 0 || strides[i] % vec != 0) {
      set_error("strides must be non-negative multiples of %lld elements (16 bytes)", (long long)vec);
      return WKV_ERR_INVALID_ARG;
    }
  }
  if (p->kv_stride_h < d || p->q_stride_h < d || p->out_stride_h < d) {
    set_error("head strides must be >= head_dim"); return WKV_ERR_INVALID_ARG;
  }

  wkv_dims dm;
  std::memset(&dm, 0, sizeof(dm));
  dm.obs_rows = (int32_t)(G * p->w_obs);
  dm.t_stride = p->max_seq_len - p->w_obs;
  for (int b = 0; b < p->batch; ++b) {
    const int64_t L = p->seq_len[b], w = p->win[b], tp = p->top_p[b], k = p->k_windows[b];
    if (L < p->w_obs || L > p->max_seq_len) {
      set_error("seq_len[%d]=%lld outside [w_obs=%d, max_seq_len=%d]", b, (long long)L, p->w_obs, p->max_seq_len);
      return WKV_ERR_INVALID_ARG;
    }
    if (w < 1) { set_error("win[%d] must be >= 1", b); return WKV_ERR_INVALID_ARG; }
    if (w > WKV_MAX_WIN) { set_error("win[%d]=%lld exceeds WKV_MAX_WIN=%d", b, (long long)w, WKV_MAX_WIN); return WKV_ERR_UNSUPPORTED; }
    if (tp < 1) { set_error("top_p[%d] must be >= 1", b); return WKV_ERR_INVALID_ARG; }
    const int64_t nw = ceil_div(L - p->w_obs, w);
    if (nw > WKV_MAX_WINDOWS) { set_error("sequence %d has %lld windows (> WKV_MAX_WINDOWS=%d)", b, (long long)nw, WKV_MAX_WINDOWS); return WKV_ERR_UNSUPPORTED; }
    if (k < 0 || k > nw) { set_error("k_windows[%d]=%lld outside [0, NW=%lld]", b, (long long)k, (long long)nw); return WKV_ERR_INVALID_ARG; }
    if (nw > dm.nw_max) dm.nw_max = (int32_t)nw;
    if (k > dm.k_max) dm.k_max = (int32_t)k;
    if (k * w + p->w_obs > dm.nkeep_max) dm.nkeep_max = (int32_t)(k * w + p->w_obs);
    dm.total_tokens += L;
  }
  if (dims) *dims = dm;
  return WKV_OK;
}

void fill_shape(const wkv_problem *p, const wkv_dims &dims, Shape *s, BatchParams *bp) {
  s->B = p->batch; s->Hq = p->n_q_heads; s->Hkv = p->n_kv_heads; s->d = p->head_dim;
  s->w_obs = p->w_obs; s->G = p->n_q_heads / p->n_kv_heads; s->M = dims.obs_rows;
  s->t_stride = dims.t_stride; s->nw_max = dims.nw_max; s->k_max = dims.k_max;
  s->nkeep_max = dims.nkeep_max; s->dtype = p->dtype;
  s->fill_padding = (p->flags & WKV_KEEP_PADDING) ? 0 : 1;
  const double scale = p->scale > 0.0f ? (double)p->scale : 1.0 / std::sqrt((double)p->head_dim);
  s->w_magic = 65536u / (uint32_t)p->w_obs + 1u;
  s->hkv_magic = division_magic(p->n_kv_heads);
  s->c1 = (float)(scale * 1.4426950408889634074);
  s->q_sb = p->q_stride_b; s->q_sh = p->q_stride_h; s->q_st = p->q_stride_t;
  s->kv_sb = p->kv_stride_b; s->kv_sh = p->kv_stride_h; s->kv_st = p->kv_stride_t;
  s->o_sb = p->out_stride_b; s->o_sh = p->out_stride_h; s->o_st = p->out_stride_t;
  std::memset(bp, 0, sizeof(*bp));
  for (int b = 0; b < p->batch; ++b) {
    bp->seq[b].L = p->seq_len[b];
    bp->seq[b].win = p->win[b];
    bp->seq[b].win_magic = division_magic(p->win[b]);
    bp->seq[b].p = p->top_p[b] < p->win[b] ? p->top_p[b] : p->win[b];
    bp->seq[b].k = p->k_windows[b];
  }
}

// Number of (row, chunk) work items that hold at least one key, for chunks of `chunk` keys.
static int64_t count_items(const BatchParams &bp, int32_t B, int64_t rows_per_seq, int32_t drop, int32_t chunk) {
  int64_t n = 0;
  for (int32_t b = 0; b < B; ++b) n += ((uint32_t)std::max(bp.seq[b].L - drop, 0) + (uint32_t)chunk - 1u) / (uint32_t)chunk;
  return n * rows_per_seq;
}

// Keys per workgroup.  A workgroup's fixed cost (its query fragments, the first key tiles, the
// epilogue) is several microseconds: the launch is fastest when its non-empty work items fill the
// `slots` that the device holds at a time a whole number of times, with chunks as long as that allows.
// Chunks are multiples of CHUNK_UNIT keys; `drop` keys at the end of every sequence are not part of the pass.
// Longer chunks never make more items, so the shortest that fills the slots so many times is found by halving: 64
// sequences in 8 groups are validated and planned in 4.2 us, 24 us by trying one length after the other.
static int32_t pick_chunk(const BatchParams &bp, int32_t B, int64_t rows_per_seq, int32_t drop, int32_t lo, int32_t hi,
                          int64_t slots) {
  int64_t total = 0;
  for (int32_t b = 0; b < B; ++b) total += (int64_t)std::max(bp.seq[b].L - drop, 0) * rows_per_seq;
  if (total <= 0) return lo;
  const int64_t items_hi = count_items(bp, B, rows_per_seq, drop, hi);
  for (int64_t rounds = 1; rounds <= 64; ++rounds) {
    const int64_t c = ceil_div(ceil_div(total, slots * rounds), CHUNK_UNIT);
    if (c * CHUNK_UNIT < lo) return lo;
    if (c * CHUNK_UNIT > hi || items_hi > slots * rounds) continue;
    int32_t at = (int32_t)c, fits = hi / CHUNK_UNIT;        // in units; `fits` does
    while (at < fits) {
      const int32_t mid = (at + fits) / 2;
      if (count_items(bp, B, rows_per_seq, drop, mid * CHUNK_UNIT) > slots * rounds) at = mid + 1;
      else fits = mid;
    }
    return fits * CHUNK_UNIT;
  }
  return hi;
}

// Chunks of at most c keys per sequence, equal among themselves.  Only what holds keys becomes a workgroup: the
// dispatcher deals workgroup numbers round-robin to the 8 XCDs, and numbers without work would leave some
// of them more of the rest than others.
static void plan_pass(const BatchParams &bp, int32_t B, int32_t drop, int32_t c, PassPlan *pp) {
  std::memset(pp, 0, sizeof(*pp));
  for (int32_t b = 0; b < B; ++b) {
    const int64_t keys = std::max(bp.seq[b].L - drop, 1), n = ceil_div(keys, c);
    pp->chunk[b] = (uint8_t)ceil_div(ceil_div(keys, n), CHUNK_UNIT);
    pp->first[b + 1] = pp->first[b] + (int32_t)ceil_div(keys, pp->chunk[b] * CHUNK_UNIT);
  }
}

// Rows of a tile of the score passes.  32-row tiles take 15 % less time for the same logits (wkv_score.hip), but a wave's rows in
// steps of 32.  Whole calls with 16- / with 32-row tiles, each on keys that the memory-side cache holds from the call before and on keys
// that it does not, bf16:
//   two row groups        always 32.  128 channels, 256 rows: 290 MB of keys 240, 241 / 213, 211 us, 540 MB 436, 438 / 397, 394; 64 channels, 224 rows,
//                         290 MB 352, 349 / 285, 286.
//   97 to 112 rows        16, as 32-row tiles make 128 of them: 128 channels, 17 MB 27.7, 29.2 / 28.5, 30.4; 101 MB 61.7, 65.7 / 63.4, 68.3; 201 MB
//                         101, 108 / 104, 124; 64 channels, 201 MB 125, 128 / 123, 135; 290 MB 177, 176 / 181, 182.  Where little is computed 32 all the
//                         same: 128 channels and at most 128 keys a workgroup, 4 MB 21.4, 22.6 / 20.8, 21.9; 64 channels up to HEAVY logits,
//                         33 MB 39.7, 41.8 / 38.6, 40.8.
//   at most 16 rows       32: 128 channels, 12 MB 19.6, 22.6 / 19.6, 21.9, 33 MB 26.6, 28.8 / 26.9, 29.0; 64 channels, 33 MB 29.4, 31.3 / 28.2, 30.3.
//   other rows            32, but 16 on nontemporal streams of 128 channels, which are bound by power: 128 rows, 400 MB 186, 189 / 189, 194, 540 MB
//                         259, 259 / 260, 262; 64 rows, 290 MB 132, 133 / 133, 133; 201 MB 92.8, 99.1 / 91.0, 98.2.  64 channels, 128 rows, 540 MB
//                         330, 335 / 315, 319; 32 rows, 400 MB 181, 179 / 176, 174.
constexpr int64_t HEAVY = (int64_t)3 << 24;       // logits of a call: 196608 a compute unit
static int32_t score_tile(const Shape &s, const ScorePlan &pl, int64_t keys, bool two_groups) {
  if (s.dtype == WKV_F32) return 16;
  if (two_groups) return 32;
  if (pl.m_pad != 112) return pl.nontemporal && s.d == 128 ? 16 : 32;
  if (s.d == 64) return keys * pl.m_pad > HEAVY ? 16 : 32;
  return *std::max_element(pl.pass[0].chunk, pl.pass[0].chunk + s.B) > 2 ? 16 : 32;
}

ScorePlan plan_score(const Shape &s, const BatchParams &bp, int32_t n_groups) {
  ScorePlan pl;
  pl.m_pad = (s.M + 15) / 16 * 16;
  const int64_t rows_per_seq = (int64_t)s.Hkv * n_groups;
  // Workgroups that the device holds at a time (256 compute units): two per unit with one row group (half the
  // LDS and the registers), else one.  Up to 1024 keys per compute unit one is better all the same: the
  // shorter chain of a smaller chunk does not make up for the second prologue and the larger fold.  Whole calls with one / with two, keys held / not held
  // by the memory-side cache, 16-bit, thousands of keys:
  //   128 channels, 128 rows   131 33.9 / 37.3, 34.0 / 37.6 us; 262 50.3 / 54.7, 53.9 / 58.5; 1300 182 / 167, 2097 270 / 243; mixed lengths 733 117.7 / 116.3,
  //                            125.0 / 122.5, 1011 150.7 / 147.6
  //   64 channels, 128 rows    131 29.7 / 30.6; 262 41.6 / 43.7; 393 48.7 / 48.3, 50.4 / 50.6; 524 58.2 / 56.8; 1049 96.3 / 86.1
  // (Between 1024 and 2560 keys per unit one still takes less with 128 channels or few rows: 128 rows 524 73.1 / 79.5, 64 rows 67.3 / 70.4, 64 channels and
  // 64 rows 45.0 / 48.1.)
  const int32_t wave_rows = s.dtype == WKV_F32 && s.d == 128 ? 64 : 128;
  int64_t keys = 0;
  for (int32_t b = 0; b < s.B; ++b) keys += bp.seq[b].L * rows_per_seq;
  const int64_t slots = pl.m_pad <= wave_rows && keys > 256 * 1024 ? 512 : 256;
  const int32_t shortest = 2 * CHUNK_UNIT, longest = 8192;
  plan_pass(bp, s.B, 0, pick_chunk(bp, s.B, rows_per_seq, 0, shortest, longest, slots), &pl.pass[0]);
  plan_pass(bp, s.B, s.w_obs, pick_chunk(bp, s.B, rows_per_seq, s.w_obs, shortest, longest, slots), &pl.pass[1]);
  // Keys that the memory-side cache holds until the second pass are better left there; a larger stream reads
  // faster past it.  Whole calls with plain / nontemporal loads, keys held / not held from the call before: 128 rows of 128 channels, 192 MB 104 / 112, 113 / 113 us,
  // 254 MB 129 / 144, 139 / 144, 320 MB 162 / 164, 170 / 165, 384 MB 196 / 192, 201 / 192; 64 rows, 254 MB 119 / 128, 128 / 129, 320 MB 146 / 146, 153 / 147;
  // 256 rows, 254 MB 195 / 200, 200 / 201, 320 MB 256 / 253, 257 / 254; 64 channels, 128 rows, 254 MB 150 / 166, 158 / 161, 384 MB 232 / 235, 231 / 235.  fp32, 32 rows:
  // 134 MB 74.9 / 79.0, 335 MB 170.3 / 166.9, 1.07 GB 503 / 445; 128 rows and more wait for the matrix pipe, 1 GB 1182 / 1178.
  pl.nontemporal = keys * s.d * elem_bytes(s.dtype) > MEMORY_CACHE_BYTES;
  // Key tiles fetched twice, once per row group, against a barrier per tile: worth it while a chunk is short enough for
  // the two waves to stay together and the cache has room for what they lose; not for the few tiles of the smallest calls.  Whole calls with a barrier / with
  // rings of their own, keys held / not held by the memory-side cache from the call before, us:
  //   128 channels, to 192 rows    7 MB 23.4 / 24.1, 24.4 / 25.0; 8 MB 22.9 / 23.2, 23.8 / 24.5; 17 MB 33.1 / 32.2, 33.8 / 32.7; 32 MB one length 40.6 / 41.9, 41.0 / 42.2, mixed
  //                                45.4 / 44.7, 45.8 / 44.8; 53 MB mixed 70.7 / 69.4, 75.0 / 73.2; 99 MB mixed 94.4 / 93.1, 100.4 / 102.0; 105 MB mixed 132.8 / 128.0,
  //                                138.3 / 134.5; 96 MB one length 75.5 / 77.2, 80.8 / 82.0; 128 MB 90.4 / 97.2, 97.0 / 108.4
  //   more rows                    8 MB 28.7 / 29.1, 29.7 / 29.8; 19 MB 36.7 / 35.3; 53 MB mixed 83.6 / 78.6, 86.9 / 83.2; 64 MB 65.9 / 64.1, 70.6 / 70.7; 105 MB mixed 146.6 / 136.1,
  //                                150.9 / 143.3; 109 MB 95.8 / 92.9, 101.5 / 101.7; 128 MB 106.3 / 106.0, 114.3 / 121.1
  //   64 channels                  4 MB 22.8 / 22.4; 16 MB 37.3 / 35.6; 96 MB 99.3 / 91.0, 102.3 / 97.7; 160 MB 164.3 / 159.6, 170.3 / 172.7 and 150.5 / 139.5, 156.6 / 150.7;
  //                                192 MB 189.7 / 179.2, 193.4 / 184.4; 240 MB 197.4 / 194.2, 204.9 / 211.4
  const int64_t bytes = keys * s.d * elem_bytes(s.dtype);
  pl.own_rings = s.d == 64 ? bytes <= MEMORY_CACHE_BYTES * 3 / 4 : bytes > ((int64_t)9 << 20) && bytes <= MEMORY_CACHE_BYTES * 7 / 16;
  pl.tile = score_tile(s, pl, keys, pl.m_pad > wave_rows);
  pl.n_chunks1 = 0;
  for (int32_t b = 0; b < s.B; ++b) pl.n_chunks1 = std::max(pl.n_chunks1, pl.pass[0].first[b + 1] - pl.pass[0].first[b]);
  // every pass-2 workgroup re-reads the partials of its rows when it folds them itself: 64 KB at 128 rows and 64
  // chunks, about what the extra launch costs
  pl.fold_in_pass2 = pl.n_chunks1 <= 64;
  return pl;
}

void fill_score_args(const Shape &s, const BatchParams &bp, const ScorePlan &plan, const GroupPtrs &gp, int32_t n_groups, int32_t pass,
                     bool fold, ScoreArgs *a, ScoreGrid *grid) {
  const PassPlan &pp = plan.pass[pass], &stats = plan.pass[0];
  for (int32_t b = 0; b < WKV_MAX_BATCH; ++b) a->ends[b] = b < s.B ? pp.first[b + 1] : INT32_MAX;
  for (int32_t b = 0; b < s.B; ++b) {
    const SeqParam &q = bp.seq[b];
    a->seq[b] = {q.L, pp.first[b], stats.first[b + 1] - stats.first[b], pp.chunk[b] | (uint32_t)q.win << 8 | (uint32_t)q.p << 16, q.win_magic,
                 pp.first[b + 1] - 1};
  }
  a->gp = gp;
  a->m_pad = plan.m_pad;
  a->n_chunks1 = plan.n_chunks1;
  a->fold = fold;
  a->hkv_magic = division_magic(s.Hkv);
  a->items = pp.first[s.B];
  *grid = score_grid(s.Hkv, n_groups, a->items);
  a->row_bits = grid->row_bits;
  a->last_x = grid->x - 1; a->last_y = grid->y - 1; a->last_z = grid->z - 1;
}

// The single-read kernel applies to 16-bit inputs with at most 128 softmax rows per KV head (its
// workgroups keep the row statistics of one row tile set in registers).  It is taken only when the
// caller asks for it: on MI355X the exchange of the row statistics between workgroups costs more
// than the second read of the keys it saves (measured at the 32K configuration: 0.57 ms against
// 0.20 ms for the two passes), so the library never chooses it by itself.
ResidentPlan plan_resident(const Shape &s, const BatchParams &bp, const ScorePlan &plan, int32_t n_groups, int32_t flags) {
  ResidentPlan rp;
  std::memset(&rp, 0, sizeof(rp));
  rp.m_pad = plan.m_pad;
  int64_t per_group = 0;
  for (int32_t b = 0; b < s.B; ++b) {
    const int64_t nsl = ceil_div(bp.seq[b].L, RK_SLICE);
    per_group += nsl * s.Hkv;
    if (nsl > rp.nsl_max) rp.nsl_max = (int32_t)nsl;
  }
  const int64_t items = per_group * n_groups;
  rp.items_per_group = (int32_t)per_group;
  rp.n_items = (int32_t)items;
  // a wait that is still unanswered after this many polls (tens of milliseconds) gives up
  rp.spin_limit = (flags & WKV_DEBUG_WAIT_GIVES_UP) ? 0 : (1 << 16);
  const bool can = s.dtype != WKV_F32 && plan.m_pad <= 128 && s.t_stride > 0 && items < (int64_t)1 << 30;
  rp.use = can && (flags & WKV_SCORE_SINGLE_READ);
  rp.pools = 1;
  for (int32_t b = 0; rp.use && b < s.B; ++b) rp.pools = rp.pools && RK_SLICE % bp.seq[b].win == 0;
  return rp;
}

static inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

Workspace carve_workspace(const Shape &s, const ScorePlan &plan, const ResidentPlan &rp, int32_t n_groups, void *base) {
  Workspace w;
  const size_t rows = (size_t)n_groups * s.B * s.Hkv;
  const size_t part = align256(rows * plan.m_pad * plan.n_chunks1 * sizeof(float2));
  const size_t tb = align256(rows * (size_t)(s.t_stride > 0 ? s.t_stride : 1) * sizeof(float));
  const size_t sb = align256(rows * (size_t)(s.nw_max > 0 ? s.nw_max : 1) * sizeof(float));
  const size_t lb = align256(rows * plan.m_pad * sizeof(float));
  // single-read kernel: the (m, z) partials of every slice and the synchronisation words
  const size_t rkp = rp.use ? align256(rows * (size_t)rp.nsl_max * rp.m_pad * sizeof(unsigned long long)) : 0;
  const size_t rks = rp.use ? align256((RK_GLOBAL_WORDS + rows * RK_SYNC_WORDS) * sizeof(uint32_t)) : 0;
  w.t_offset = part;
  w.s_offset = part + tb;
  w.bytes = part + tb + sb + lb + rkp + rks;
  char *b = (char *)base;          // a null base asks for the sizes only: no pointer is formed from it
  w.partials = b ? (float2 *)b : nullptr;
  w.t = b ? (float *)(b + w.t_offset) : nullptr;
  w.s = b ? (float *)(b + w.s_offset) : nullptr;
  w.lse = b ? (float *)(b + part + tb + sb) : nullptr;
  w.rk_partials = b && rp.use ? (unsigned long long *)(b + part + tb + sb + lb) : nullptr;
  w.rk_sync = b && rp.use ? (uint32_t *)(b + part + tb + sb + lb + rkp) : nullptr;
  return w;
}

wkv_status validate_decode(const wkv_decode_shape *p, Decode *out) {
  g_err[0] = 0;
  if (!p) { set_error("shape is NULL"); return WKV_ERR_INVALID_ARG; }
  if (p->batch < 1) { set_error("batch must be >= 1 (got %d)", p->batch); return WKV_ERR_INVALID_ARG; }
  if (p->n_kv_heads < 1 || p->n_q_heads < 1 || p->n_q_heads % p->n_kv_heads != 0) {
    set_error("n_q_heads (%d) must be a positive multiple of n_kv_heads (%d)", p->n_q_heads, p->n_kv_heads);
    return WKV_ERR_INVALID_ARG;
  }
  if ((int64_t)p->batch * p->n_kv_heads > 65535) {
    set_error("batch * n_kv_heads exceeds 65535 (launch grid limit); split the call"); return WKV_ERR_UNSUPPORTED;
  }
  const int32_t G = p->n_q_heads / p->n_kv_heads;
  if (G > 8) { set_error("n_q_heads / n_kv_heads = %d is not supported by the decode step (at most 8)", G); return WKV_ERR_UNSUPPORTED; }
  if (p->dtype != WKV_F32 && p->dtype != WKV_BF16 && p->dtype != WKV_F16) { set_error("unknown dtype %d", p->dtype); return WKV_ERR_INVALID_ARG; }
  if (p->head_dim != 64 && p->head_dim != 128) {
    set_error("head_dim %d is not supported (64 or 128)", p->head_dim); return WKV_ERR_UNSUPPORTED;
  }
  if (!(p->scale >= 0.0f) || std::isinf(p->scale)) {
    set_error("scale must be finite and >= 0 (0 selects 1/sqrt(head_dim))"); return WKV_ERR_INVALID_ARG;
  }
  if (p->capacity < 1) { set_error("capacity must be >= 1"); return WKV_ERR_INVALID_ARG; }
  if (p->flags & ~WKV_DECODE_KEEP_COUNT) { set_error("unknown bits in flags (0x%x)", p->flags); return WKV_ERR_INVALID_ARG; }
  const int64_t vec = 16 / elem_bytes(p->dtype);
  const int64_t strides[3] = {p->cache_stride_b, p->cache_stride_h, p->cache_stride_t};
  for (int i = 0; i < 3; ++i)
    if (strides[i] < 0 || strides[i] % vec != 0) {
      set_error("cache strides must be non-negative multiples of %lld elements (16 bytes)", (long long)vec);
      return WKV_ERR_INVALID_ARG;
    }
  if (p->cache_stride_t < p->head_dim || p->cache_stride_h < p->head_dim) {
    set_error("cache token and head strides must be >= head_dim"); return WKV_ERR_INVALID_ARG;
  }
  DecodeShape &s = out->shape;
  s.B = p->batch; s.Hq = p->n_q_heads; s.Hkv = p->n_kv_heads; s.d = p->head_dim; s.G = G; s.dtype = p->dtype;
  s.capacity = p->capacity;
  s.keep_count = (p->flags & WKV_DECODE_KEEP_COUNT) ? 1 : 0;
  const double scale = p->scale > 0.0f ? (double)p->scale : 1.0 / std::sqrt((double)p->head_dim);
  s.c1 = (float)(scale * 1.4426950408889634074);
  s.sb = p->cache_stride_b; s.sh = p->cache_stride_h; s.st = p->cache_stride_t;
  s.heads_magic = division_magic(s.B * s.Hkv); s.kv_magic = division_magic(s.Hkv);
  // Key ranges: about 1536 workgroups if every cache were full (one and a half times what the device holds with 128 channels and up to four heads; n_valid is not known
  // here, and in a batch of mixed lengths a good part of them finds nothing to do), of at least 128 rows (two
  // blocks for each of four waves, or one for each of eight: with half of that the fixed cost and the merge outweigh the shorter chain),
  // multiples of 64 rows (a block for each of four waves).  us a layer of 32q/8kv heads with 1024 / 1536 / 2016 workgroups: one sequence of 20000 rows
  // 21.8 / 20.7 / 20.7, five of 3000 16.1 / 15.2 / 15.0, 16 of 4128 50.5 / 48.4 / 49.9, 64 of 4128 165.0 / 166.4 / 166.5; mixed batches, the shortest an eighth of the longest: 8 up to
  // 4000 19.3 / 15.9 / 15.9, 24 up to 4000 48.4 / 44.7 / 40.1, 64 up to 2000 65.6 / 59.3 / 59.4; 4 KV heads, 16 up to 32000 106 / 97 / 86; 32 KV heads, 8 up to 16000 244 / 185 / 164;
  // 28q/4kv, eleven 16.2 / 14.4 / 14.4.
  const int64_t rows = (int64_t)s.B * s.Hkv;
  constexpr int64_t total = 1536;
  static_assert(total * 8 * (128 + 2) * (int64_t)sizeof(float) <= WKV_DECODE_STATIC_SCRATCH_BYTES,
                "the partial results fit the static scratch array if one range per row does");
  const int64_t splits = std::min<int64_t>(std::max<int64_t>(total / rows, 1), DEC_MAX_SPLITS);
  const int64_t chunk = std::max<int64_t>(ceil_div(ceil_div(s.capacity, splits), 64) * 64, 128);
  s.chunk = (int32_t)chunk;
  s.n_splits = (int32_t)ceil_div(s.capacity, chunk);
  static_assert((int64_t)65535 * 8 * (128 + 2) * (int64_t)sizeof(float) < (int64_t)1 << 32 && total < 65535, "32-bit offsets of the partial results");
  s.stats_at = (uint32_t)(rows * s.n_splits * s.G * s.d * (int64_t)sizeof(float));
  out->ws_bytes = (size_t)rows * s.n_splits * s.G * (s.d + 2) * sizeof(float);
  return WKV_OK;
}

}  // namespace wkv

using namespace wkv;

extern "C" {

wkv_status wkv_get_dims(const wkv_problem *problem, wkv_dims *dims) {
  if (!dims) { set_error("dims is NULL"); return WKV_ERR_INVALID_ARG; }
  return validate(problem, dims);
}

size_t wkv_workspace_bytes(const wkv_problem *problem, int32_t n_groups) {
  wkv_dims dm;
  if (validate(problem, &dm) != WKV_OK) return 0;
  if (n_groups < 1 || n_groups > WKV_MAX_GROUPS) { set_error("n_groups outside [1, %d]", WKV_MAX_GROUPS); return 0; }
  Shape s; BatchParams bp;
  fill_shape(problem, dm, &s, &bp);
  ScorePlan pl = plan_score(s, bp, n_groups);
  return carve_workspace(s, pl, plan_resident(s, bp, pl, n_groups, problem->flags), n_groups, nullptr).bytes;
}

wkv_status wkv_get_workspace_layout(const wkv_problem *problem, int32_t n_groups, wkv_workspace_layout *layout) {
  if (!layout) { set_error("layout is NULL"); return WKV_ERR_INVALID_ARG; }
  wkv_dims dm;
  wkv_status st = validate(problem, &dm);
  if (st != WKV_OK) return st;
  if (n_groups < 1 || n_groups > WKV_MAX_GROUPS) { set_error("n_groups outside [1, %d]", WKV_MAX_GROUPS); return WKV_ERR_INVALID_ARG; }
  Shape s; BatchParams bp;
  fill_shape(problem, dm, &s, &bp);
  const ScorePlan pl = plan_score(s, bp, n_groups);
  const ResidentPlan rp = plan_resident(s, bp, pl, n_groups, problem->flags);
  const Workspace w = carve_workspace(s, pl, rp, n_groups, nullptr);
  layout->t_offset = w.t_offset;
  layout->s_offset = w.s_offset;
  layout->s_written = rp.pools ? 1 : 0;
  layout->t_written = rp.pools ? 0 : 1;
  return WKV_OK;
}

size_t wkv_decode_workspace_bytes(const wkv_decode_shape *shape) {
  Decode dc;
  if (validate_decode(shape, &dc) != WKV_OK) return 0;
  return dc.ws_bytes;
}

wkv_status wkv_group_budgets(double b_total, int32_t n_groups, double lambda, double *budgets_out) {
  if (!budgets_out) { set_error("budgets_out is NULL"); return WKV_ERR_INVALID_ARG; }
  if (n_groups < 1 || !(lambda > 0.0) || !(b_total >= 0.0)) {
    set_error("need n_groups >= 1, lambda > 0, b_total >= 0"); return WKV_ERR_INVALID_ARG;
  }
  const double H = (double)n_groups;
  if (n_groups == 1) { budgets_out[0] = b_total; return WKV_OK; }
  const double top = b_total / (lambda * H);          // Eq. 6, group H-1
  const double bottom = 2.0 * b_total / H - top;      // Eq. 6, group 0
  const double step = (bottom - top) / (H - 1.0);     // Eq. 7
  for (int32_t h = 0; h < n_groups; ++h) budgets_out[h] = bottom - step * (double)h;
  return WKV_OK;
}

const char *wkv_status_string(wkv_status st) {
  switch (st) {
    case WKV_OK: return "ok";
    case WKV_ERR_INVALID_ARG: return "invalid argument";
    case WKV_ERR_UNSUPPORTED: return "unsupported problem";
    case WKV_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case WKV_ERR_HIP: return "HIP error";
  }
  return "unknown status";
}

const char *wkv_last_error(void) { return g_err; }

}  // extern "C"
