// Which kernels the launch plan of the score passes asks for, on both sides of its lines.
#include <cstdio>
#include <cstring>

#include "wkv_internal.h"

using namespace wkv;

static ScorePlan plan(int dtype, int d, int rows, int hkv, int groups, int L, int w_obs = 16) {
  Shape s;
  BatchParams bp;
  std::memset(&s, 0, sizeof s);
  std::memset(&bp, 0, sizeof bp);
  s.B = 1; s.Hkv = hkv; s.w_obs = w_obs; s.M = rows; s.d = d; s.dtype = dtype;
  bp.seq[0].L = L;
  bp.seq[0].win = 8;
  return plan_score(s, bp, groups);
}

static int failures = 0;
#define CHECK(x) do { if (!(x)) { std::printf("FAILED line %d: %s\n", __LINE__, #x); ++failures; } } while (0)

int main() {
  for (int dtype : {WKV_BF16, WKV_F16}) {
    // two row groups: tiles of 32 rows whatever the stream (16384 tokens of 8 groups are 256 MB)
    for (int L : {512, 4096, 16381, 16384, 16385, 32768})
      for (int rows : {129, 192, 224, 256})
        for (int d : {64, 128}) CHECK(plan(dtype, d, rows, 8, 8, L).tile == 32);
    // 97 to 112 rows: 16, but 32 where little is computed
    for (int rows : {97, 100, 112}) {
      for (int L : {12000, 32768}) CHECK(plan(dtype, 128, rows, 4, 2, L).tile == 16);
      CHECK(plan(dtype, 64, rows, 4, 8, 32768).tile == 16);
      CHECK(plan(dtype, 128, rows, 4, 1, 4096).tile == 32);
      CHECK(plan(dtype, 64, rows, 4, 1, 32768).tile == 32);
    }
    CHECK(plan(dtype, 128, 96, 4, 2, 12000).tile == 32);
    CHECK(plan(dtype, 128, 113, 4, 2, 12000).tile == 32);
    // one row group of other counts: 16 only on nontemporal streams of 128 channels
    for (int rows : {8, 16, 32, 64, 96, 128}) {
      CHECK(plan(dtype, 128, rows, 8, 8, 16384).tile == 32);
      CHECK(plan(dtype, 128, rows, 8, 8, 16385).tile == 16);
      CHECK(plan(dtype, 64, rows, 32, 8, 32768).tile == 32);
    }
  }
  for (int rows : {16, 64, 112, 128, 256})
    for (int d : {64, 128}) CHECK(plan(WKV_F32, d, rows, 8, 8, 16385).tile == 16);
  for (int dtype : {WKV_BF16, WKV_F16}) {
    // two row groups: rings of their own
    for (int rows : {160, 192, 193, 256}) {
      CHECK(!plan(dtype, 128, rows, 8, 1, 4608).own_rings && plan(dtype, 128, rows, 8, 1, 4609).own_rings);        // 9 MB
      CHECK(plan(dtype, 64, rows, 8, 1, 512).own_rings);
    }
    CHECK(plan(dtype, 128, 256, 8, 7, 8192).own_rings && !plan(dtype, 128, 256, 8, 7, 8193).own_rings);          // 112 MB
    CHECK(plan(dtype, 64, 256, 8, 12, 16384).own_rings && !plan(dtype, 64, 256, 8, 12, 16385).own_rings);        // 192 MB
  }
  std::printf("%d checks failed\n", failures);
  return failures != 0;
}
