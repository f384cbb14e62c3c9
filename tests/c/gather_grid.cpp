// The gather's grid: every piece of a compact cache once, no workgroup without one and all but the last with two; and which
// batches take workgroups of more than one wave.
#include <cstdio>
#include <cstring>
#include <initializer_list>
#include <vector>

#include "wkv_internal.h"

using namespace wkv;

static int failures = 0;
#define EXPECT(cond, ...) do { if (!(cond)) { std::printf("FAILED line %d: %s: ", __LINE__, #cond); std::printf(__VA_ARGS__); std::printf("\n"); ++failures; } } while (0)

static int threads(std::initializer_list<int> k, int w_obs, bool keep, int d = 64) {
  Shape s;
  BatchParams bp;
  std::memset(&s, 0, sizeof s);
  std::memset(&bp, 0, sizeof bp);
  s.w_obs = w_obs;
  s.d = d;
  s.dtype = WKV_BF16;
  s.fill_padding = !keep;
  for (int n : k) {
    bp.seq[s.B].win = 1;
    bp.seq[s.B++].k = n;
    if (n + w_obs > s.nkeep_max) s.nkeep_max = n + w_obs;
  }
  return gather_threads(s, bp);
}

int main() {
  for (int apart : {1, 4, 8})
    for (int rows : {2, 4, 8, 16, 32})
      for (int nk = 1; nk < 2200; nk += nk < 300 ? 1 : 37) {
        const GatherGrid g = gather_grid(nk, rows, apart);
        const int pieces = (nk + rows - 1) / rows;
        std::vector<int> taken(pieces + 2 * apart + 2, 0);
        for (int x = 0; x < g.workgroups; ++x) {        // as the kernel numbers them
          const int first = x / apart * (2 * apart) + x % apart, step = x < g.last ? apart : g.last_apart;
          EXPECT(first < pieces, "%d rows, workgroup %d", nk, x);
          ++taken[first]; ++taken[first + step];
        }
        for (int i = 0; i < pieces; ++i) EXPECT(taken[i] == 1, "%d rows by %d, %d apart: piece %d", nk, rows, apart, i);
        EXPECT(g.workgroups == (pieces + 1) / 2, "%d rows by %d, %d apart", nk, rows, apart);
      }
  // budgets and the room for them, observation window included
  EXPECT(threads({1000}, 0, false) == 64, " "); EXPECT(threads({1000}, 0, true) == 64, " ");
  EXPECT(threads({1000, 0, 0}, 0, false) == 64, "a third"); EXPECT(threads({1000, 0, 0}, 0, true) == 128, "a third");
  EXPECT(threads({1001, 0, 0, 0}, 0, false) == 256, "a quarter"); EXPECT(threads({1000, 200, 0}, 0, true) == 64, "0.4");
  EXPECT(threads({1000, 199, 0}, 0, true) == 128, "less than 0.4"); EXPECT(threads({800, 0, 0, 0, 0}, 200, false) == 64, "0.36");
  EXPECT(threads({800, 0, 0, 0, 0}, 200, false, 128) == 256, "0.36, rows of 256 bytes"); EXPECT(threads({8, 1, 0}, 0, false, 128) == 64, "3/8");
  EXPECT(threads({0, 0}, 8, true) == 64, "observation window alone");
  std::printf("%d checks failed\n", failures);
  return failures != 0;
}
