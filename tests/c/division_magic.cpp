// Divisions by multiplication in the decode step's kernels: every workgroup gets the head and range that the division gives.
#include <cstdio>
#include <cstring>

#include "wkv_internal.h"

using namespace wkv;

int main() {
  int failures = 0;
  for (int heads : {1, 2, 3, 5, 7, 8, 32, 44, 96, 255, 511, 512, 513, 768, 1535, 1536, 1537, 4097, 32767, 65534, 65535}) {
    wkv_decode_shape p;
    std::memset(&p, 0, sizeof p);
    p.batch = 1; p.n_kv_heads = p.n_q_heads = heads; p.head_dim = 64; p.dtype = WKV_F16; p.capacity = 1 << 20;
    p.cache_stride_b = 64; p.cache_stride_h = 64; p.cache_stride_t = (int64_t)64 * heads;
    for (int batch = 1; batch <= 2 && batch * heads <= 65535; ++batch) {
      p.batch = batch;
      Decode d;
      if (validate_decode(&p, &d) != WKV_OK) { std::printf("FAILED %d x %d: %s\n", batch, heads, wkv_last_error()); ++failures; continue; }
      const int rows = batch * heads;
      for (int y = 0; y < d.shape.n_splits; ++y)
        for (int x = 0; x < rows; ++x) {
          const RangeOf it(x, y, rows, d.shape.heads_magic);
          const int head = (x + 9 * y) % rows;
          if (it.head != head || it.range != y || divide(it.head, d.shape.kv_magic) != head / heads) {
            if (++failures < 10) std::printf("FAILED %d of %d, range %d: head %d, %d\n", x, rows, y, head, it.head);
          }
        }
    }
  }
  std::printf("%d checks failed\n", failures);
  return failures != 0;
}
