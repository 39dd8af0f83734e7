// The segment length of the marching kernels (lor_common.hpp) is that of a search
// over every length, and is found in little time whatever the number of layers.
#include <chrono>
#include <cstdio>

#include "../../paper_2210_12253_amd/csrc/lor_common.hpp"

static int64_t exhaustive(int64_t layers, int64_t tiles, int64_t slots, int64_t extra, int64_t* steps) {
  int64_t seglen = layers, best = -1;
  for (int64_t len = 1; len <= layers; ++len) {
    const int64_t ns = (layers + len - 1) / len;
    if (ns > 65535) continue;
    const int64_t cost = (tiles * ns + slots - 1) / slots * (len + (ns > 1 ? extra : 0));
    if (best < 0 || cost < best) {
      best = cost;
      seglen = len;
    }
  }
  *steps = best;
  return seglen;
}

int main() {
  const int64_t tiles[] = {1, 3, 16, 49, 500, 4099, 1000003}, slots[] = {256, 1024, 2048, 4096};
  const int64_t many[] = {1000, 4096, 65535, 65536, 99991, 131071, 200000};
  for (int i = 1; i <= 300 + 7; ++i) {
    const int64_t layers = i <= 300 ? i : many[i - 301];
    for (int64_t t : tiles)
      for (int64_t s : slots)
        for (int64_t extra = 0; extra < 2; ++extra) {
          int64_t a, b;
          const int64_t la = lor::march_segment(layers, t, s, extra, &a), lb = exhaustive(layers, t, s, extra, &b);
          if (la != lb || a != b) {
            std::printf("layers %lld tiles %lld slots %lld extra %lld: %lld (%lld), not %lld (%lld)\n", (long long)layers,
                        (long long)t, (long long)s, (long long)extra, (long long)la, (long long)a, (long long)lb,
                        (long long)b);
            return 1;
          }
        }
  }
  const auto t0 = std::chrono::steady_clock::now();
  const int64_t len = lor::march_segment(500000000, 1, 2048, 1);
  const double s = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
  std::printf("500,000,000 layers: length %lld in %.6f s\n", (long long)len, s);
  return s < 0.1 ? 0 : 1;
}
