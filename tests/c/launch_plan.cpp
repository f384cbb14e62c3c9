// The chunk lengths of the score passes against a search of every length, on batches of random and of awkward lengths.
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <random>

#include "wkv_internal.h"

using namespace wkv;

static int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Chunks as long as filling the slots a whole number of times allows, in steps of CHUNK_UNIT from 2 * CHUNK_UNIT to 8192 keys.
static int64_t searched(const BatchParams &bp, int32_t B, int64_t rows, int32_t drop, int64_t slots) {
  const int64_t lo = 2 * CHUNK_UNIT, hi = 8192;
  int64_t total = 0;
  for (int32_t b = 0; b < B; ++b) total += std::max(bp.seq[b].L - drop, 0) * rows;
  if (total == 0) return lo;
  for (int64_t rounds = 1; rounds <= 64; ++rounds) {
    int64_t c = ceil_div(ceil_div(total, slots * rounds), CHUNK_UNIT) * CHUNK_UNIT;
    if (c < lo) return lo;
    for (; c <= hi; c += CHUNK_UNIT) {
      int64_t items = 0;
      for (int32_t b = 0; b < B; ++b) items += ceil_div(std::max(bp.seq[b].L - drop, 0), c) * rows;
      if (items <= slots * rounds) return c;
    }
  }
  return hi;
}

int main() {
  std::mt19937 rng(5);
  auto upto = [&](int n) { return (int)(rng() % (unsigned)n); };
  int bad = 0, plans = 0;
  for (int i = 0; i < 4000; ++i) {
    Shape s;
    BatchParams bp;
    std::memset(&s, 0, sizeof s);
    std::memset(&bp, 0, sizeof bp);
    const int dtypes[3] = {WKV_BF16, WKV_F16, WKV_F32};
    s.B = i % 5 == 0 ? WKV_MAX_BATCH : 1 + upto(WKV_MAX_BATCH);
    s.Hkv = 1 + upto(i % 7 == 0 ? 512 : 32);
    s.w_obs = 1 + upto(64);
    s.M = 1 + upto(WKV_MAX_OBS_ROWS);
    s.d = 64 << upto(2);
    s.dtype = dtypes[upto(3)];
    const int groups = 1 + upto(i % 3 == 0 ? WKV_MAX_GROUPS : 8), longest = s.w_obs + (1 << upto(19));
    for (int b = 0; b < s.B; ++b) {
      bp.seq[b].L = i % 4 == 0 ? longest : s.w_obs + upto(longest - s.w_obs + 1);
      bp.seq[b].win = 8;
    }
    const ScorePlan pl = plan_score(s, bp, groups);
    int64_t keys = 0;
    const int64_t rows = (int64_t)s.Hkv * groups;
    for (int b = 0; b < s.B; ++b) keys += bp.seq[b].L * rows;
    const int wave_rows = s.dtype == WKV_F32 && s.d == 128 ? 64 : 128;
    const int64_t slots = (s.M + 15) / 16 * 16 <= wave_rows && keys > 256 * 1024 ? 512 : 256;
    for (int pass = 0; pass < 2; ++pass) {
      const int drop = pass ? s.w_obs : 0;
      const int64_t c = searched(bp, s.B, rows, drop, slots);
      int32_t first = 0;
      for (int b = 0; b < s.B; ++b, ++plans) {
        const int64_t L = std::max(bp.seq[b].L - drop, 1), n = ceil_div(L, c), units = ceil_div(ceil_div(L, n), CHUNK_UNIT);
        first += (int32_t)ceil_div(L, units * CHUNK_UNIT);
        if (pl.pass[pass].chunk[b] != units || pl.pass[pass].first[b + 1] != first) ++bad;
      }
    }
  }
  std::printf("%d of %d plans differ\n", bad, plans);
  return bad != 0;
}
