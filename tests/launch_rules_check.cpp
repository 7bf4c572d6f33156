// Host check of the launch rules in common.h that size and index device
// memory: spread slice counters stay inside their allocation; division by a
// launch constant is exact; the kernels' run decoding (run_at on a RunOrder)
// is the one on the SliceOrder.
#include <cstdint>
#include <cstdio>

#include "common.h"

int main() {
  using namespace ebag;
  int bad = 0, cases = 0;
  for (int64_t capacity : {(int64_t)65536, (int64_t)1 << 24})
    for (int64_t n : {(int64_t)1, (int64_t)8, (int64_t)1023, (int64_t)1024, (int64_t)1025, (int64_t)2048, (int64_t)32769,
                      (int64_t)65536, (int64_t)262144, (int64_t)262145, (int64_t)1 << 24, (int64_t)1 << 30})
      for (bool per_table : {false, true}) {
        ++cases;
        const int32_t s = counter_shift_for(n, capacity, per_table);
        if (s < 0 || s > 6 || (per_table && s != 0)) ++bad;
        if (s > 0 && (n << s) > capacity) ++bad;                               // beyond the allocation
        if (!per_table && s < 6 && (n << (s + 1)) <= capacity) ++bad;          // spread as far as it fits
      }
  const uint32_t edges[] = {0, 1, 2, 3, 25, 26, 63, 64, 65, 127, 128, 1000, 65535, 65536, 65537, 6700417,
                            0x3fffffff, 0x40000000, 0x40000001, 0x7ffffffe, 0x7fffffff};
  for (uint32_t d : edges) {
    if (d == 0) continue;
    const Divisor v = make_divisor(d);
    for (uint32_t n : edges)
      for (int64_t m : {(int64_t)n - 1, (int64_t)n, (int64_t)n + 1, (int64_t)n * d - 1, (int64_t)n * d, (int64_t)n * d + 1,
                        (int64_t)0x7fffffff / d * d - 1, (int64_t)0x7fffffff / d * d}) {
        if (m < 0 || m > 0x7fffffff) continue;
        ++cases;
        if (divide_by(v, (uint32_t)m) != (uint32_t)m / d) ++bad;
      }
  }
  for (int64_t d : {(int64_t)0, (int64_t)1 << 31, (int64_t)1 << 32, (int64_t)1 << 40})  // refused launches
    if (make_divisor(d).d < 1) ++bad;
  for (int G : {0, 1, 2, 8})
    for (int T : {1, 3, 8, 24, 40})
      for (int J : {1, 2, 5})
        for (int n : {1, 2, 7, 64}) {
          if (G > 1 && T % G) continue;
          const SliceOrder o{n, 1, 0, 0, G};
          const RunOrder r = make_run_order(o, T, J);
          for (int64_t q = 0; q < (int64_t)n * T * J; ++q) {
            ++cases;
            int64_t gs;
            int32_t tp, j;
            uint32_t gs2, tp2, j2;
            run_at(o, T, J, q, &gs, &tp, &j);
            run_at(r, (uint32_t)q, &gs2, &tp2, &j2);
            if (gs2 != gs || (int32_t)tp2 != tp || (int32_t)j2 != j) ++bad;
          }
        }
  std::printf("cases=%d bad=%d\n", cases, bad);
  return bad != 0;
}
