// The launch grid of the score passes: every workgroup of every row once and equal shares for the 8 XCDs, to which workgroup numbers are
// dealt in turn; and the argument block against the plan it is made of.
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <vector>

#include "wkv_internal.h"

using namespace wkv;

static int failures = 0;
#define EXPECT(cond, ...) do { if (!(cond)) { std::printf("FAILED line %d: %s: ", __LINE__, #cond); std::printf(__VA_ARGS__); std::printf("\n"); ++failures; } } while (0)

int main() {
  for (int rows = 1; rows <= 72; ++rows)
    for (int items = 1; items <= 130; items += items < 40 ? 1 : 7) {
      const int groups = rows % 4 == 0 && items % 2 ? 4 : rows % 3 == 0 ? 3 : 1, heads = rows / groups;
      const ScoreGrid g = score_grid(heads, groups, items);
      std::vector<int> taken(rows * items, 0), share(8, 0), xcds(rows, 0);
      int number = 0;
      for (int z = 0; z < g.z; ++z)
        for (int y = 0; y < g.y; ++y)
          for (int x = 0; x < g.x; ++x, ++number) {
            const ScoreItem it(x, y, z, g.row_bits, heads, division_magic(heads));
            const int row = it.group * heads + it.head;
            EXPECT(it.group >= 0 && it.group < groups && it.head >= 0 && it.head < heads && it.item >= 0, "%d rows of %d", rows, items);
            if (it.item >= items) continue;
            ++taken[row * items + it.item];
            ++share[number % 8];
            xcds[row] |= 1 << number % 8;
          }
      for (int n : taken) EXPECT(n == 1, "%d rows of %d", rows, items);
      EXPECT(*std::max_element(share.begin(), share.end()) == (rows * items + 7) / 8, "%d rows of %d", rows, items);
      if (g.row_bits)
        for (int m : xcds) EXPECT(__builtin_popcount(m) <= 8 >> g.row_bits, "%d rows of %d", rows, items);
    }
  EXPECT(score_grid(8, 1, 32).row_bits == 3 && score_grid(8, 8, 7).row_bits == 3 && score_grid(4, 1, 63).row_bits == 2 && score_grid(4, 3, 20).row_bits == 2, " ");
  EXPECT(score_grid(12, 1, 21).row_bits == 0 && score_grid(3, 1, 40).row_bits == 0 && score_grid(1, 2, 127).row_bits == 1, " ");
  // As many heads and groups as a call may have: within what a grid has in y and z, and the group and head of every row right.
  for (int heads : {1, 1023, 1024, 8192, 32767, 32768, 46342, 50000, 65535})
    for (int groups : {1, 2, 3, 8, 64})
      for (int items : {1, 8}) {
        const ScoreGrid g = score_grid(heads, groups, items);
        EXPECT(g.y <= 65535 && g.z <= 65535, "%d heads, %d groups", heads, groups);
        int64_t wrong = 0, seen = 0;
        std::vector<uint8_t> taken((size_t)heads * groups, 0);
        for (int z = 0; z < g.z; ++z)
          for (int y = 0; y < g.y; ++y)
            for (int x = 0; x < g.x; ++x) {
              const ScoreItem it(x, y, z, g.row_bits, heads, division_magic(heads));
              const bool in = it.group >= 0 && it.group < groups && it.head >= 0 && it.head < heads;
              if (!in) ++wrong;
              else if (it.item < items) { ++seen; ++taken[(size_t)it.group * heads + it.head]; }
            }
        for (uint8_t n : taken) wrong += n != items;
        EXPECT(wrong == 0 && seen == (int64_t)heads * groups * items, "%d heads, %d groups, %d items", heads, groups, items);
      }

  Shape s;
  BatchParams bp;
  GroupPtrs gp;
  std::memset(&s, 0, sizeof s);
  std::memset(&bp, 0, sizeof bp);
  std::memset(&gp, 0, sizeof gp);
  s.B = WKV_MAX_BATCH; s.Hkv = 3; s.w_obs = 32; s.M = 128; s.d = 128; s.dtype = WKV_BF16;
  for (int b = 0; b < s.B; ++b) bp.seq[b] = {b == 7 ? 32 : 32 + 37 * b * b, 1 + 2 * b, 1 + b, 1, division_magic(1 + 2 * b)};
  const ScorePlan pl = plan_score(s, bp, 2);
  for (int pass = 0; pass < 2; ++pass) {
    ScoreArgs a;
    ScoreGrid g;
    fill_score_args(s, bp, pl, gp, 2, pass, pass == 1, &a, &g);
    const PassPlan &pp = pl.pass[pass];
    EXPECT(a.items == pp.first[s.B] && a.fold == pass && a.m_pad == pl.m_pad, "pass %d", pass);
    for (int b = 0; b < s.B; ++b) {
      const ScoreSeq &q = a.seq[b];
      EXPECT(a.ends[b] == pp.first[b + 1] && q.first == pp.first[b] && q.last == pp.first[b + 1] - 1, "pass %d, sequence %d", pass, b);
      EXPECT(q.n_parts == pl.pass[0].first[b + 1] - pl.pass[0].first[b] && (q.packed & 0xff) == pp.chunk[b], "pass %d, sequence %d", pass, b);
      EXPECT((int)(q.packed >> 8 & 0xff) == 1 + 2 * b && (int)(q.packed >> 16) == 1 + b && q.win_magic == bp.seq[b].win_magic, "pass %d, sequence %d", pass, b);
    }
  }
  std::printf("%d checks failed\n", failures);
  return failures != 0;
}
