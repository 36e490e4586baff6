// Every order the no-allocation entry point takes has a tile on every device, within its buffers.
#include <cstdio>

#include "../../paper_1101_0265_amd/csrc/direct_tiles.h"

int main() {
  using namespace snf;
  const int64_t max_n = 896, max_ld = 912;
  int other = 0;
  for (int cus = 1; cus <= 320; ++cus)
    for (int64_t n = 1; n <= max_n; ++n) {
      const int t = noalloc_tile(n, cus, max_ld), own = direct_tile(n, cus);
      const int64_t nt = t ? (n + t - 1) / t : 0, ld = t ? direct_stride(n, t) : 0;
      if (!t || ld > max_ld || ld < nt * t || ld % 16 || nt * (nt + 1) / 2 > kDirectThreads ||
          (cus >= kDirectThreads && t != own)) {
        std::printf("n = %lld on %d units: tile %d, stride %lld\n", (long long)n, cus, t,
                    (long long)ld);
        return 1;
      }
      other += t != own;
    }
  std::printf("ok %d\n", other);
  return 0;
}
