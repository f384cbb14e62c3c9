// The order in which the decode step's workgroups take the key ranges of a batch: every range once, and the rows of a
// batch of mixed lengths spread over the 8 XCDs, to which workgroups are dealt in turn.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <random>
#include <vector>

#include "wkv_internal.h"

using namespace wkv;

static int failures = 0;
#define EXPECT(cond, ...) do { if (!(cond)) { std::printf("FAILED line %d: %s: ", __LINE__, #cond); std::printf(__VA_ARGS__); std::printf("\n"); ++failures; } } while (0)

static DecodeShape shape_of(int batch, int heads, int capacity) {
  wkv_decode_shape p;
  std::memset(&p, 0, sizeof p);
  p.batch = batch; p.n_q_heads = heads; p.n_kv_heads = heads; p.head_dim = 128; p.dtype = WKV_BF16; p.capacity = capacity;
  p.cache_stride_b = (int64_t)heads * capacity * 128; p.cache_stride_h = (int64_t)capacity * 128; p.cache_stride_t = 128;
  Decode d;
  if (validate_decode(&p, &d) != WKV_OK) { EXPECT(false, "%d x %d", batch, heads); std::memset(&d, 0, sizeof d); }
  return d.shape;
}

int main() {
  for (int heads : {1, 2, 4, 5, 8, 32})
    for (int batch : {1, 2, 3, 8, 11, 24, 48, 64, 200, 2000})
      for (int capacity : {1, 100, 1000, 4352, 33024, 200000}) {
        const DecodeShape s = shape_of(batch, heads, capacity);
        const int rows = s.B * s.Hkv;
        std::vector<char> seen((size_t)rows * s.n_splits, 0);
        int missing = rows * s.n_splits;
        for (int y = 0; y < s.n_splits; ++y)
          for (int x = 0; x < rows; ++x) {
            const RangeOf it(x, y, rows, s.heads_magic);
            if (it.head < 0 || it.head >= rows || it.range < 0 || it.range >= s.n_splits) { ++missing; continue; }
            char &c = seen[(size_t)it.head * s.n_splits + it.range];
            missing -= !c;
            c = 1;
          }
        EXPECT(missing == 0, "%d x %d, capacity %d", batch, heads, capacity);
      }
  // the most rows of an XCD over the mean
  std::mt19937 rng(7);
  for (int heads : {4, 8, 32})
    for (int batch : {8, 11, 16, 24, 48, 64})
      for (int longest : {1000, 4000, 32000}) {
        const DecodeShape s = shape_of(batch, heads, longest + 256);
        double worst = 0.0;
        for (int draw = 0; draw < 20; ++draw) {
          std::vector<int> n(batch, longest);
          for (int b = 1; b < batch; ++b) n[b] = (int)(longest / 8.0 * std::exp2(3.0 * (rng() % 10000) / 10000.0));
          std::vector<double> xcd(8, 0.0);
          double all = 0.0;
          const int rows = s.B * s.Hkv;
          for (int id = 0; id < rows * s.n_splits; ++id) {
            const RangeOf it(id % rows, id / rows, rows, s.heads_magic);
            const int left = n[it.head / s.Hkv] - it.range * s.chunk, take = left < 0 ? 0 : left < s.chunk ? left : s.chunk;
            xcd[id % 8] += take;
            all += take;
          }
          for (double v : xcd) worst = std::max(worst, v / (all / 8));
        }
        std::printf("%d x %d, %d rows, %d ranges of %d: most over mean %.2f\n", batch, heads, longest, s.n_splits, s.chunk, worst);
        // a range is not divided: with 4 heads of 8 sequences, four ranges more or less on an XCD
        EXPECT(worst <= 1.3, "%d x %d, %d rows", batch, heads, longest);
      }
  std::printf("%d checks failed\n", failures);
  return failures != 0;
}
