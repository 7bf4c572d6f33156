// Host check of the launch rules in common.h that size and index device
// memory: spread slice counters stay inside their allocation.
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
  std::printf("cases=%d bad=%d\n", cases, bad);
  return bad != 0;
}
