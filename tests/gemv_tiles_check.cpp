// Host check of gemv_tiles.h: the workgroups of every owner visit each of its
// tiles once and stop, up to 2^31 - 1 tiles; a split covers every row and leaves a
// launch that fills the device as it is.
#include <cstdint>
#include <cstdio>
#include <vector>

#include "gemv_tiles.h"

int main() {
  using namespace ebag;
  int bad = 0, cases = 0;
  const int64_t most = 0x7fffffff;
  // few tiles: every tile, counted
  for (int64_t n : {(int64_t)1, (int64_t)2, (int64_t)7, (int64_t)64, (int64_t)1000})
    for (int R : {1, 2, 3, 8, 16})
      for (int64_t P : {(int64_t)1, (int64_t)3, (int64_t)64, n}) {
        if (P > n) continue;
        ++cases;
        TileOwners o;
        make_owners(n, R, (int32_t)P, &o);
        std::vector<int> seen(n, 0);
        for (int q = 0; q < R; ++q)
          for (uint32_t p = 0; p < P; ++p)
            for (uint32_t i = first_tile(o, q, p, (uint32_t)P); i < o.own[q + 1]; i += (uint32_t)P) {
              if (i % (uint32_t)P != p) ++bad;
              ++seen[i];
            }
        for (int s : seen) bad += s != 1;
      }
  // many: walks of few steps, from the first tile to past the last
  for (int64_t n : {most, most - 1, most - 1000})
    for (int R : {1, 2, 16})
      for (int64_t P : {n, n - 1, n / 2 + 1, n / 5}) {
        TileOwners o;
        make_owners(n, R, (int32_t)P, &o);
        if (o.own[0] != 0 || o.own[R] != (uint64_t)n) ++bad;
        for (int q = 0; q < R; ++q)
          for (int64_t p : {(int64_t)0, (int64_t)1, P / 2, P - 1}) {
            ++cases;
            int64_t want = (int64_t)o.own[q] + ((p - (int64_t)o.own[q]) % P + P) % P;
            uint32_t i = first_tile(o, q, (uint32_t)p, (uint32_t)P);
            int steps = 0;
            for (; i < o.own[q + 1] && steps < 10; i += (uint32_t)P, want += P, ++steps)
              if ((int64_t)i != want) ++bad;
            if (steps >= 10 || want < (int64_t)o.own[q + 1]) ++bad;
          }
      }
  for (int64_t wgs : {(int64_t)1, (int64_t)8, (int64_t)51, (int64_t)1024, (int64_t)2048, (int64_t)16777216, most})
    for (int W : {1, 2, 4, 16})
      for (int TM : {1, 63, 64, 128, 4096})
        for (int64_t bytes : {(int64_t)16, (int64_t)1024, (int64_t)65536}) {
          ++cases;
          int32_t sub = 0;
          const int32_t split = split_for(wgs, W, TM, bytes, &sub);
          if (split < 1 || sub < 1 || (int64_t)split * sub < TM || (int64_t)(split - 1) * sub >= TM) ++bad;
          if (split > 1 && wgs * W * split > 2 * kTargetWaves) ++bad;
        }
  std::printf("cases=%d bad=%d\n", cases, bad);
  return bad != 0;
}
