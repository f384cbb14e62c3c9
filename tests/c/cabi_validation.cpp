// Drives every entry point of the C ABI through its host-side validation with valid and invalid
// arguments.  Linked against the host half of the library and the launcher stand-ins, built with
// AddressSanitizer + UndefinedBehaviorSanitizer: any out-of-bounds access, overflow or misuse in the
// validation, size and planning code aborts the program.  Device pointers are fake (never
// dereferenced: the stubs launch nothing).
#include <cstdio>
#include <cstring>
#include <vector>

#include "wkv.h"

extern "C" int wkv_stub_launches;
static int failures = 0;
#define EXPECT(cond) do { if (!(cond)) { std::printf("FAILED line %d: %s (last error: %s)\n", __LINE__, #cond, wkv_last_error()); ++failures; } } while (0)

struct Prob {
  std::vector<int32_t> L, win, p, k;
  wkv_problem pr;
  Prob(int batch, int L0, int hq, int hkv, int d, int w_obs, int w, int tp, int kk, int dtype) : L(batch), win(batch, w), p(batch, tp), k(batch, kk) {
    std::memset(&pr, 0, sizeof pr);
    int lmax = 0;
    for (int b = 0; b < batch; ++b) { L[b] = L0 - 17 * b; if (L[b] > lmax) lmax = L[b]; }
    pr.batch = batch; pr.n_q_heads = hq; pr.n_kv_heads = hkv; pr.head_dim = d; pr.w_obs = w_obs; pr.max_seq_len = lmax;
    pr.dtype = dtype; pr.seq_len = L.data(); pr.win = win.data(); pr.top_p = p.data(); pr.k_windows = k.data();
    pr.q_stride_b = (int64_t)hq * w_obs * d; pr.q_stride_h = (int64_t)w_obs * d; pr.q_stride_t = d;
    pr.kv_stride_b = (int64_t)hkv * lmax * d; pr.kv_stride_h = (int64_t)lmax * d; pr.kv_stride_t = d;
    const int64_t nk = (int64_t)kk * w + w_obs;
    pr.out_stride_b = hkv * nk * d; pr.out_stride_h = nk * d; pr.out_stride_t = d;
  }
};

int main() {
  void *dev = (void *)0x7f0000001000ull;      // "device" memory: aligned, never touched
  // ---- dims, workspace sizes and layouts over a sweep of shapes (the planning code runs for each) -------
  const int dtypes[3] = {WKV_F32, WKV_BF16, WKV_F16};
  for (int dt = 0; dt < 3; ++dt)
    for (int batch : {1, 3, 64})
      for (int L0 : {2400, 4096, 32768, 262176})
        for (int hq : {8, 32, 64})
          for (int w : {1, 8, 24, 128}) {
            if ((int64_t)(L0 - 32) / w > WKV_MAX_WINDOWS) continue;
            Prob P(batch, L0, hq, 8, 128, 32, w, (w + 1) / 2, 3, dtypes[dt]);
            wkv_dims d;
            const wkv_status st = wkv_get_dims(&P.pr, &d);
            EXPECT(st == WKV_OK);
            if (st != WKV_OK) continue;
            EXPECT(d.obs_rows == hq / 8 * 32 && d.t_stride == L0 - 32 && d.nkeep_max == 3 * w + 32);
            for (int ng : {1, 8, 64}) {
              const size_t ws = wkv_workspace_bytes(&P.pr, ng);
              wkv_workspace_layout lay;
              EXPECT(ws > 0 && ws % 256 == 0);
              EXPECT(wkv_get_workspace_layout(&P.pr, ng, &lay) == WKV_OK);
              EXPECT(lay.t_offset < lay.s_offset && lay.s_offset < ws && lay.t_written + lay.s_written == 1);
            }
          }
  // ---- every entry point: valid arguments reach the (stub) launchers, invalid ones launch nothing -----------
  Prob P(2, 4096, 32, 8, 128, 32, 8, 8, 64, WKV_BF16);
  const size_t ws1 = wkv_workspace_bytes(&P.pr, 1), ws2 = wkv_workspace_bytes(&P.pr, 2);
  const void *kl[4] = {dev, dev, dev, dev}; void *ol[4] = {dev, dev, dev, dev};
  const void *qg[2] = {dev, dev}; const float *lg[2] = {(const float *)dev, (const float *)dev};
  int32_t *idev = (int32_t *)dev; float *fdev = (float *)dev;
  int before = wkv_stub_launches;
  EXPECT(wkv_score(&P.pr, dev, dev, nullptr, fdev, dev, ws1, nullptr) == WKV_OK);
  EXPECT(wkv_window_pool(&P.pr, fdev, fdev, nullptr) == WKV_OK);
  EXPECT(wkv_topk_windows(&P.pr, fdev, idev, idev, idev, nullptr) == WKV_OK);
  EXPECT(wkv_gather_group(&P.pr, 4, kl, kl, idev, idev, ol, ol, nullptr) == WKV_OK);
  EXPECT(wkv_compress_group(&P.pr, 4, dev, nullptr, kl, kl, ol, ol, idev, idev, idev, dev, ws1, nullptr) == WKV_OK);
  EXPECT(wkv_compress_groups(&P.pr, 2, 2, qg, lg, nullptr, kl, kl, ol, ol, idev, idev, idev, dev, ws2, nullptr) == WKV_OK);
  int32_t kg[4] = {64, 10, 0, 64};
  EXPECT(wkv_compress_groups(&P.pr, 2, 2, qg, nullptr, kg, kl, kl, ol, ol, idev, idev, idev, dev, ws2, nullptr) == WKV_OK);
  EXPECT(wkv_index_jaccard(&P.pr, 4, idev, idev, fdev, nullptr) == WKV_OK);
  EXPECT(wkv_stub_launches > before);
  // ---- a short call: one launch, or by the two score passes (one launcher) where the caller asks for them -----------
  Prob Q(2, 500, 8, 2, 128, 8, 8, 8, 6, WKV_BF16);
  const size_t wsq = wkv_workspace_bytes(&Q.pr, 1);
  char *base = (char *)dev;
  const void *kq[2] = {base, base + (1 << 20)}; void *oq[2] = {base + (2 << 20), base + (3 << 20)};
  int32_t *iq = (int32_t *)(base + (4 << 20));
  auto launches = [&]() {
    const int had = wkv_stub_launches;
    EXPECT(wkv_compress_group(&Q.pr, 2, base + (5 << 20), nullptr, kq, kq, oq, oq, iq, iq, iq, base + (6 << 20), wsq, nullptr) == WKV_OK);
    return wkv_stub_launches - had;
  };
  EXPECT(launches() == 1);
  Q.pr.flags = WKV_SCORE_TWO_PASS;
  EXPECT(launches() == 2);
  // outputs in the memory of the queries or the normalisers are written when the passes have read those; beside it they are as any others
  Q.pr.flags = 0;
  const int64_t q_bytes = 2 * 8 * 8 * 128 * 2, out_bytes = 2 * 2 * 56 * 128 * 2;
  void *const v_out = oq[1];
  auto with = [&](char *q, const float *lse, char *out, char *idx) {
    oq[1] = out;
    const int had = wkv_stub_launches;
    EXPECT(wkv_compress_group(&Q.pr, 2, q, lse, kq, kq, oq, oq, iq, (int32_t *)idx, iq, base + (6 << 20), wsq, nullptr) == WKV_OK);
    oq[1] = v_out;
    return wkv_stub_launches - had;
  };
  char *const q = base + (5 << 20), *const lse = base + (7 << 20), *const apart = (char *)v_out;
  EXPECT(with(q, nullptr, q + q_bytes, (char *)iq) == 1);
  EXPECT(with(q, nullptr, q + q_bytes - 16, (char *)iq) == 2);
  EXPECT(with(q, nullptr, q - out_bytes, (char *)iq) == 1);
  EXPECT(with(q, nullptr, q - out_bytes + 16, (char *)iq) == 2);
  EXPECT(with(q, (const float *)lse, apart, (char *)iq) == 1);
  EXPECT(with(q, (const float *)lse, lse, (char *)iq) == 2);
  EXPECT(with(q, (const float *)lse, apart, lse + 2 * 8 * 8 * 4 - 4) == 2);
  EXPECT(with(q, (const float *)lse, apart, lse + 2 * 8 * 8 * 4) == 1);
  // ---- which short calls are one launch: with handed-over normalisers fewer, long windows only in short sequences ---------------
  auto one = [&](int L, int heads, int kv, int d, int w_obs, int win, int dtype, bool given) {
    Prob R(1, L, heads, kv, d, w_obs, win, win, 1, dtype);
    const int had = wkv_stub_launches;
    EXPECT(wkv_compress_group(&R.pr, 2, q, given ? (const float *)lse : nullptr, kq, kq, oq, oq, iq, iq, iq, base + (64 << 20), wkv_workspace_bytes(&R.pr, 1), nullptr) == WKV_OK);
    return wkv_stub_launches - had == 1;
  };
  const int rows_of[5] = {16, 32, 64, 128, 136};              // by one query head of two a KV head; tokens at most: all, with normalisers
  const int tokens[2][2][5][2] = {{{{1024, 1024}, {1024, 1024}, {1024, 512}, {512, 0}, {0, 0}}, {{1024, 1024}, {1024, 512}, {512, 512}, {512, 0}, {0, 0}}},
                                  {{{1024, 512}, {512, 0}, {0, 0}, {0, 0}, {0, 0}}, {{512, 0}, {0, 0}, {0, 0}, {0, 0}, {0, 0}}}};
  for (int f32 = 0; f32 < 2; ++f32)
    for (int wide = 0; wide < 2; ++wide)
      for (int r = 0; r < 5; ++r)
        for (int given = 0; given < 2; ++given)
          for (int L : {400, 512, 513, 1024, 1025})
            for (int dtype : {WKV_F32, WKV_BF16, WKV_F16})
              if ((dtype == WKV_F32) == (f32 == 1))
                EXPECT(one(L, 4, 2, wide ? 128 : 64, rows_of[r] / 2, 8, dtype, given) == (L <= tokens[f32][wide][r][given]));
  for (int given = 0; given < 2; ++given) {
    EXPECT(one(1000, 4, 2, 64, 8, 64, WKV_BF16, given));
    EXPECT(one(512 + 8, 4, 2, 64, 8, 65, WKV_BF16, given) && !one(513 + 8, 4, 2, 64, 8, 65, WKV_BF16, given));
  }
  before = wkv_stub_launches;
  EXPECT(wkv_score(&P.pr, nullptr, dev, nullptr, fdev, dev, ws1, nullptr) == WKV_ERR_INVALID_ARG);
  EXPECT(wkv_score(&P.pr, (char *)dev + 2, dev, nullptr, fdev, dev, ws1, nullptr) == WKV_ERR_INVALID_ARG);
  EXPECT(wkv_score(&P.pr, dev, dev, nullptr, fdev, nullptr, ws1, nullptr) == WKV_ERR_WORKSPACE);
  EXPECT(wkv_score(&P.pr, dev, dev, nullptr, fdev, (char *)dev + 64, ws1, nullptr) == WKV_ERR_WORKSPACE);
  EXPECT(wkv_score(&P.pr, dev, dev, nullptr, fdev, dev, ws1 - 1, nullptr) == WKV_ERR_WORKSPACE);
  EXPECT(wkv_score(nullptr, dev, dev, nullptr, fdev, dev, ws1, nullptr) == WKV_ERR_INVALID_ARG);
  EXPECT(wkv_window_pool(&P.pr, nullptr, fdev, nullptr) == WKV_ERR_INVALID_ARG);
  EXPECT(wkv_topk_windows(&P.pr, fdev, idev, nullptr, idev, nullptr) == WKV_ERR_INVALID_ARG);
  EXPECT(wkv_gather_group(&P.pr, 0, kl, kl, idev, idev, ol, ol, nullptr) == WKV_ERR_INVALID_ARG);
  EXPECT(wkv_gather_group(&P.pr, WKV_MAX_LAYERS + 1, kl, kl, idev, idev, ol, ol, nullptr) == WKV_ERR_INVALID_ARG);
  const void *kl_bad[4] = {dev, nullptr, dev, dev};
  EXPECT(wkv_gather_group(&P.pr, 4, kl_bad, kl, idev, idev, ol, ol, nullptr) == WKV_ERR_INVALID_ARG);
  EXPECT(wkv_compress_group(&P.pr, 0, dev, nullptr, kl, kl, ol, ol, idev, idev, idev, dev, ws1, nullptr) == WKV_ERR_INVALID_ARG);
  EXPECT(wkv_compress_group(&P.pr, 4, nullptr, nullptr, kl, kl, ol, ol, idev, idev, idev, dev, ws1, nullptr) == WKV_ERR_INVALID_ARG);
  EXPECT(wkv_compress_groups(&P.pr, 0, 2, qg, nullptr, nullptr, kl, kl, ol, ol, idev, idev, idev, dev, ws2, nullptr) == WKV_ERR_INVALID_ARG);
  EXPECT(wkv_compress_groups(&P.pr, 2, 64, qg, nullptr, nullptr, kl, kl, ol, ol, idev, idev, idev, dev, ws2, nullptr) == WKV_ERR_INVALID_ARG);
  EXPECT(wkv_compress_groups(&P.pr, 2, 2, qg, nullptr, nullptr, kl, kl, ol, ol, idev, idev, idev, dev, ws1, nullptr) == WKV_ERR_WORKSPACE);
  const float *lg_bad[2] = {(const float *)dev, nullptr};
  EXPECT(wkv_compress_groups(&P.pr, 2, 2, qg, lg_bad, nullptr, kl, kl, ol, ol, idev, idev, idev, dev, ws2, nullptr) == WKV_ERR_INVALID_ARG);
  int32_t kg_bad[4] = {64, 65, 0, 64};
  EXPECT(wkv_compress_groups(&P.pr, 2, 2, qg, nullptr, kg_bad, kl, kl, ol, ol, idev, idev, idev, dev, ws2, nullptr) == WKV_ERR_INVALID_ARG);
  EXPECT(wkv_index_jaccard(&P.pr, 0, idev, idev, fdev, nullptr) == WKV_ERR_INVALID_ARG);
  EXPECT(wkv_get_workspace_layout(&P.pr, 1, nullptr) == WKV_ERR_INVALID_ARG);
  EXPECT(wkv_get_dims(&P.pr, nullptr) == WKV_ERR_INVALID_ARG);
  EXPECT(wkv_workspace_bytes(&P.pr, 0) == 0);
  EXPECT(std::strlen(wkv_last_error()) > 0);
  EXPECT(wkv_stub_launches == before);
  // ---- decode -------------------------------------------------------------------------------------------------
  wkv_decode_shape ds; std::memset(&ds, 0, sizeof ds);
  ds.batch = 64; ds.n_q_heads = 32; ds.n_kv_heads = 8; ds.head_dim = 128; ds.dtype = WKV_BF16; ds.capacity = 4200;
  ds.cache_stride_b = 8LL * 4200 * 128; ds.cache_stride_h = 4200 * 128; ds.cache_stride_t = 128;
  const size_t dws = wkv_decode_workspace_bytes(&ds);
  EXPECT(dws > 0);
  EXPECT(wkv_decode_step(&ds, dev, dev, dev, dev, dev, idev, fdev, dev, dws, nullptr) == WKV_OK);
  ds.flags = WKV_DECODE_KEEP_COUNT;
  EXPECT(wkv_decode_step(&ds, dev, dev, dev, dev, dev, idev, fdev, dev, dws, nullptr) == WKV_OK);
  ds.flags = 2;
  EXPECT(wkv_decode_step(&ds, dev, dev, dev, dev, dev, idev, fdev, dev, dws, nullptr) == WKV_ERR_INVALID_ARG);
  ds.flags = 0;
  EXPECT(wkv_decode_step(&ds, dev, dev, dev, dev, dev, idev, fdev, dev, dws - 1, nullptr) == WKV_ERR_WORKSPACE);
  EXPECT(wkv_decode_step(&ds, dev, dev, dev, dev, dev, nullptr, fdev, dev, dws, nullptr) == WKV_ERR_INVALID_ARG);
  before = wkv_stub_launches;
  EXPECT(wkv_decode_step_static(&ds, dev, dev, dev, dev, dev, idev, fdev, nullptr) == WKV_OK);
  EXPECT(wkv_stub_launches == before + 1);
  EXPECT(wkv_decode_step_static(&ds, dev, dev, nullptr, dev, dev, idev, fdev, nullptr) == WKV_ERR_INVALID_ARG);
  ds.batch = 4000;                    // 32000 rows of partial results: beyond the static scratch array
  EXPECT(wkv_decode_workspace_bytes(&ds) > WKV_DECODE_STATIC_SCRATCH_BYTES);
  EXPECT(wkv_decode_step_static(&ds, dev, dev, dev, dev, dev, idev, fdev, nullptr) == WKV_ERR_WORKSPACE);
  EXPECT(wkv_stub_launches == before + 1);
  ds.batch = 64;
  ds.n_q_heads = 72;
  EXPECT(wkv_decode_workspace_bytes(&ds) == 0);
  // ---- budgets (Eq. 5-7) ----------------------------------------------------------------------------------------
  double bud[8];
  EXPECT(wkv_group_budgets(32768.0, 8, 14.0, bud) == WKV_OK);
  double sum = 0; for (double x : bud) sum += x;
  EXPECT(sum > 32767.99 && sum < 32768.01);
  EXPECT(wkv_group_budgets(1.0, 0, 14.0, bud) == WKV_ERR_INVALID_ARG);
  EXPECT(std::strcmp(wkv_status_string(WKV_ERR_HIP), "HIP error") == 0);
  std::printf("%s (%d checks failed)\n", failures ? "FAILED" : "ok", failures);
  return failures ? 1 : 0;
}
