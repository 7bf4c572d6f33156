// Host check of the launch rules in common.h that size and index device
// memory: spread slice counters stay inside their allocation; division by a
// launch constant is exact; the kernels' run decoding (run_at on a RunOrder)
// is the one on the SliceOrder; which pooling kernel and which loads a plan's
// tables get; pooling workgroups' LDS leaves a CU the workgroups that their
// registers allow, and a weighted backward's keep to their bounds.
#include <cstdint>
#include <cstdio>

#include "backward.h"
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
  struct Want { int64_t rows; int64_t bytes; int check; PoolKind kind; bool streams; };
  for (const Want& w : {Want{1000, 512, 0, POOL_FAST, true}, Want{1000, 16, 0, POOL_FAST, true}, Want{1000, 512, 1, POOL_NARROW, true},
                        Want{1000, 64, 1, POOL_NARROW, false}, Want{1000, 640, 0, POOL_WIDE, true}, Want{1000, 192, 0, POOL_NARROW, false},
                        Want{1000, 2080, 0, POOL_WIDE, false}, Want{1000, 1280, 0, POOL_WIDE, true},
                        Want{10000000, 512, 0, POOL_NARROW, true}, Want{300000000, 16, 0, POOL_NARROW, false}}) {
    ebag_a2a_opts_t o{};
    o.check_indices = w.check;
    o.rows_in_flight = 8;
    TabMeta m[2] = {};
    m[0].rows = 10, m[0].row_bytes = 128, m[0].vecs = 8, m[0].vshift = 3;
    m[1].rows = w.rows, m[1].row_bytes = w.bytes, m[1].vecs = (int32_t)(w.bytes / 16), m[1].vshift = -1;
    for (int s = 0; s <= 6; ++s)
      if (m[1].vecs == 1 << s) m[1].vshift = s;
    PoolSetup ps{};
    ps.o = &o;
    ps.meta = m;
    ps.T = 2;
    for (int streams : {0, 1}) {
      ++cases;
      o.stream_rows = streams;
      const PoolVariant k = pool_variant(ps, true, false);
      if (k.kind != w.kind || k.stream_rows != (streams && w.streams)) ++bad;
    }
  }
  // a run's tile: within 16 KiB, in the general kernels five workgroups of four waves
  // (twenty of one) a CU with it
  for (PoolKind kind : {POOL_FAST, POOL_NARROW, POOL_WIDE})
    for (int waves : {1, 2, 4, 8, 16})
      for (int dim : {4, 12, 128, 256, 512, 5000}) {
        ++cases;
        const int vecs_dim = dim > 512 ? 0 : dim;  // wider rows bypass the tile
        const int bags = pool_tile_bags(kind, waves, dim, vecs_dim);
        if (bags < 1 || (bags > 1 && bags * dim > 4096)) ++bad;
        if (kind != POOL_FAST && bags > 1 && pool_lds_bytes(true, true, waves, bags * vecs_dim) * 20 > (size_t)waves * 160 * 1024) ++bad;
      }
  // workgroups that fit a CU's 160 KiB: (any, weighted, waves, tile floats) -> at least
  struct Fit { bool any, weighted; int waves, floats, at_least; };
  for (const Fit& f : {Fit{false, true, 16, 2048, 2}, Fit{false, true, 8, 1024, 4}, Fit{false, true, 4, 4096, 4},
                       Fit{false, false, 4, 4096, 6}, Fit{false, false, 16, 4096, 2}, Fit{true, true, 4, 4096, 5},
                       Fit{true, false, 4, 4096, 6}, Fit{true, true, 16, 4096 + 1024, 1}}) {
    ++cases;
    if ((int64_t)pool_lds_bytes(f.any, f.weighted, f.waves, f.floats) * f.at_least > 160 * 1024) ++bad;
  }
  // a weighted backward's run stays within 64 KiB, and its weights leave a CU its
  // 32 waves (or what the rows alone leave it)
  for (int waves : {1, 2, 4, 8, 16})
    for (int64_t rows_lds : {(int64_t)64, (int64_t)2088, (int64_t)16424, (int64_t)57464, (int64_t)65536}) {
      ++cases;
      const int64_t lds = rows_lds + 4 * (int64_t)backward_weight_slots(rows_lds, waves);
      if (lds > 65536 || (lds > rows_lds && lds * 32 > (int64_t)waves * 160 * 1024)) ++bad;
      if (waves == 16 && rows_lds < 57344 && lds != rows_lds + 8192) ++bad;
    }
  std::printf("cases=%d bad=%d\n", cases, bad);
  return bad != 0;
}
