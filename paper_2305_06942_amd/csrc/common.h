// Internal definitions shared by the host plan code and the kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ebag_a2a.h"

namespace ebag {

// Per-table constants, resident in device memory for the plan's lifetime.
struct TabMeta {
  int64_t rows;      // number of rows
  int64_t row_bytes; // D * elt (multiple of 16)
  int32_t dim;       // D
  int32_t col_off;   // first column of this table in a send-buffer row
  int32_t vecs;      // 16-byte vectors per row (= row_bytes / 16)
  int32_t vshift;    // log2(vecs) when vecs is a power of two <= 64, else -1
};

// Order in which slices are produced and drained.  order 0: natural; order
// 1: slices of destination `self` last, so slices bound for other
// destinations are finished (and can be shipped) first (Sec. III-A,
// communication-aware scheduling).  table_groups 0: runs go slice by slice,
// table positions fastest; G >= 1: table by table, slices (in the order
// above) inside a table, with run q taken by table group q mod G -- with G
// the number of XCDs, every XCD works through its own tables one at a time.
struct SliceOrder {
  int64_t n_chunks;    // B / C
  int64_t per_rank;    // (B / R) / C
  int64_t self;        // destination kept local
  int32_t order;
  int32_t table_groups;
};

__host__ __device__ inline int64_t slice_at(const SliceOrder& o, int64_t x) {
  if (o.order == 0) return x;
  const int64_t lo = o.self * o.per_rank;
  const int64_t others = o.n_chunks - o.per_rank;
  if (x < lo) return x;
  if (x < others) return x + o.per_rank;
  return lo + (x - others);
}

// Run q of a launch over n_chunks slices x T table positions x J runs per
// (slice, table) pair -> slice position gs (for slice_at), table position
// tpos, run j inside the pair.  Every q in [0, n_chunks * T * J) maps to a
// distinct triple; with table_groups G > 1, T is a multiple of G.
__host__ __device__ inline void run_at(const SliceOrder& o, int32_t T, int32_t J, int64_t q, int64_t* gs,
                                       int32_t* tpos, int32_t* j) {
  if (o.table_groups == 0) {
    const int64_t per_slice = (int64_t)T * J;
    *gs = q / per_slice;
    const int64_t rem = q - *gs * per_slice;
    *tpos = (int32_t)(rem % T);
    *j = (int32_t)(rem / T);
    return;
  }
  const int64_t G = o.table_groups;
  const int64_t per_table = o.n_chunks * J;
  const int64_t x = q % G, i = q / G;
  const int64_t k = i / per_table, r = i - k * per_table;
  *tpos = (int32_t)(k * G + x);
  *gs = r / J;
  *j = (int32_t)(r - *gs * J);
}

// Division by a launch constant d in [1, 2^31) of numbers below 2^31, as a
// multiplication (Granlund and Montgomery's round-up method: mul =
// floor(2^32 (2^shift - d) / d) + 1 with 2^shift >= d).  A division by a
// variable is a sequence of over twenty vector instructions on this GPU, over a
// hundred in 64 bits, and would stand at the head of every workgroup's chain
// of dependent steps; this is three scalar ones.
struct Divisor {
  uint32_t d, mul, shift;
};

// Out-of-range d (of launches that are refused for their run count) is clamped.
inline Divisor make_divisor(int64_t d) {
  Divisor v;
  v.d = d < 1 ? 1u : d > 0x7fffffff ? 0x7fffffffu : (uint32_t)d;
  v.shift = 0;
  while (((uint64_t)1 << v.shift) < v.d) ++v.shift;
  v.mul = (uint32_t)(((((uint64_t)1 << v.shift) - v.d) << 32) / v.d + 1);
  return v;
}

__host__ __device__ inline uint32_t divide_by(const Divisor& v, uint32_t n) {
  return (uint32_t)(((uint64_t)n * v.mul >> 32) + n) >> v.shift;
}

// run_at for launches of fewer than 2^31 runs, with the order's divisors
// prepared on the host.
struct RunOrder {
  Divisor first;   // slice-major: T * J; table-major: table_groups
  Divisor second;  // slice-major: T; table-major: n_chunks * J
  Divisor third;   // table-major: J
  int32_t table_groups;
};

inline RunOrder make_run_order(const SliceOrder& o, int32_t T, int32_t J) {
  RunOrder r;
  r.table_groups = o.table_groups;
  r.first = make_divisor(o.table_groups ? o.table_groups : (int64_t)T * J);
  r.second = make_divisor(o.table_groups ? o.n_chunks * J : T);
  r.third = make_divisor(J);
  return r;
}

__host__ __device__ inline void run_at(const RunOrder& o, uint32_t q, uint32_t* gs, uint32_t* tpos, uint32_t* j) {
  const uint32_t a = divide_by(o.first, q), x = q - a * o.first.d;
  if (o.table_groups == 0) {  // a: slice, x: (j, table) inside it
    *gs = a;
    *j = divide_by(o.second, x);
    *tpos = x - *j * o.second.d;
    return;
  }
  const uint32_t k = divide_by(o.second, a), r = a - k * o.second.d;  // x: table group, a: run inside it
  *tpos = k * o.first.d + x;
  *gs = divide_by(o.third, r);
  *j = r - *gs * o.third.d;
}

struct PoolArgs {
  const void* const* tables;  // [T] table base pointers
  const TabMeta* meta;        // [T]
  const int32_t* tperm;       // [T] position within a slice -> table
  const int32_t* indices;
  const int64_t* offsets;
  const float* weights;       // nullptr for plain sum
  float* out;                 // fused: send buffer; unfused: [T][B][D_t] scratch
  uint32_t* counters;         // bags finished per flag's slice (self-resetting), flag f's at f << counter_shift
  uint32_t* flags;            // [n_flags] epoch flags
  int32_t* status;            // plan status word
  uint64_t* trace_release;    // [n_flags] or nullptr
  uint32_t* ticket;           // [2] persistent grid: next run, workgroups done (self-resetting)
  int64_t B;
  int64_t nruns;
  int64_t suppress;           // flag index never released (-1: none)
  SliceOrder so;
  RunOrder ro;
  Divisor by_waves;           // waves
  int32_t T;
  int32_t C;
  int32_t K;                  // bags per run
  int32_t sum_dim;
  int32_t check;              // check offsets / indices
  int32_t release_mode;       // 0 agent-scope release fence, 1 device-scope stores + completion wait
  int32_t waves;              // wavefronts per workgroup (blockDim.x / 64)
  int32_t out_floats;         // LDS tile of the run's pooled rows: K x the widest of <= 64 vectors (mean: and K lengths)
  int32_t mean;               // 1: mean pooling (sum / bag length)
  int32_t per_table;          // 1: one flag / counter per (slice, table), index g * T + t
  int32_t counter_shift;
};

// Host-side description of the plan behind a pooling launch: a plan from
// ebag_a2a_create, or one assembled per call by the plan-free forward.
struct PoolSetup {
  const ebag_a2a_opts_t* o;
  const TabMeta* meta;          // [T], host copy
  int32_t T;
  int32_t C;
  int32_t sum_dim;
  int32_t dtype;
  int32_t num_cus;
  int32_t table_groups;         // SliceOrder::table_groups under these options
  const void* const* d_tables;  // device arrays the kernels read and write
  const TabMeta* d_meta;
  const int32_t* d_tperm;
  uint32_t* d_counters;
  int32_t counter_shift;
  int32_t* d_status;
  uint64_t* d_trace_release;    // nullptr: no trace
  uint32_t* d_ticket;
};

// Which of the pooling kernels a launch takes.  POOL_FAST: every table below 4
// GiB (32-bit offsets) with rows of 2^k <= 64 sixteen-byte vectors, no index
// report; its kernel needs fewer registers (fp32: 59 instead of 69 and 82) and
// reads such tables faster (26 tables x 16384 bags of 0 to 3 rows of 512 bytes: 110
// us, against 143 us by the general one).  POOL_NARROW, POOL_WIDE: the general
// kernel for any tables and for index reports, without and with rows of more than
// 32 vectors, whose code costs the others registers.
enum PoolKind { POOL_FAST = 0, POOL_NARROW = 1, POOL_WIDE = 2 };
struct PoolVariant {
  int dtype;
  int rows_in_flight;
  bool weighted, fused, stream_rows;
  PoolKind kind;
};
typedef void (*pool_fn)(const PoolArgs);
pool_fn pick_pool_f32(const PoolVariant& k);
pool_fn pick_pool_f16(const PoolVariant& k);
pool_fn pick_pool_bf16(const PoolVariant& k);
pool_fn pick_pool_wide_f32(const PoolVariant& k);
pool_fn pick_pool_wide_f16(const PoolVariant& k);
pool_fn pick_pool_wide_bf16(const PoolVariant& k);

// stream_rows: the general kernel takes it only where every table's rows are
// whole 128-byte lines.  A line that two rows share is read again soon, and loaded
// non-temporally it is gone by then: 8 tables of 2080-byte rows that fit the
// caches, bags of 32: 260 us non-temporal, 171 us cached; of 192-byte rows that do
// not, bags of 1 to 100: 117 us and 102 us.  Rows of whole lines that do not fit
// the caches are up to 4% faster non-temporal (640 bytes, bags of 32: 178 us and
// 185 us).
inline PoolVariant pool_variant(const PoolSetup& s, bool fused, bool weighted) {
  PoolVariant k;
  k.dtype = s.dtype;
  k.rows_in_flight = s.o->rows_in_flight;
  k.weighted = weighted;
  k.fused = fused;
  bool any = s.o->check_indices != 0, wide = false, whole_lines = true;
  for (int32_t t = 0; t < s.T; ++t) {
    const TabMeta& m = s.meta[t];
    if (m.vshift < 0 || m.rows * m.row_bytes > (int64_t)0xFFFFFFFFll) any = true;
    if (m.vecs > 32) wide = true;
    if (m.row_bytes % 128) whole_lines = false;
  }
  k.kind = !any ? POOL_FAST : wide ? POOL_WIDE : POOL_NARROW;
  k.stream_rows = s.o->stream_rows && (!any || whole_lines);
  return k;
}

// Most bags of a run whose pooled rows fit its LDS tile: 16 KiB, and in the
// general kernels 4.5 KiB a wave, so that with its staging slot a wave stays below
// the 8 KiB that the 20 waves their registers allow leave it.
inline int32_t pool_tile_bags(PoolKind kind, int32_t waves, int32_t max_dim, int32_t tile_dim) {
  int32_t bags = 16384 / (4 * max_dim);
  if (kind != POOL_FAST && tile_dim > 0) {
    const int32_t fit = (4608 * waves - 272) / (4 * tile_dim);
    if (fit < bags) bags = fit;
  }
  return bags < 1 ? 1 : bags;
}

// Host helpers shared by the plan and the plan-free forward (plan.hip).
constexpr int kMaxXcd = 64;

// Words between the slice counters of two flags, as a power of two, for n
// counters in `capacity` words.  Every run adds to its slice's counter, and
// atomics on one cache line are served one after the other, about 6 ns each,
// so with packed counters the runs of all whole slices in flight queue on one
// line: those get 256 bytes each where they fit.  Measured at 26 tables x
// 16384 bags of 0 to 3 rows of 512 bytes (26,624 runs, 104 to a counter): 227
// us packed, 189 us spread.  A per-table counter takes only its pair's few
// runs; there are T times as many, and spreading them gains nothing (132 us
// either way on the same bags) but touches T times the lines.
inline int32_t counter_shift_for(int64_t n, int64_t capacity, bool per_table) {
  int32_t s = per_table ? 0 : 6;
  while (s > 0 && (n << s) > capacity) --s;
  return s;
}
int check_opts(const ebag_a2a_opts_t& o);
int xcd_count(int num_cus);
int32_t table_groups_for(const ebag_a2a_opts_t& o, int32_t T, int n_xcd);
void table_order(const int64_t* row_bytes, int32_t T, int n_xcd, int32_t* perm, int32_t* work, int64_t* load);
void fill_pool_args(const PoolSetup& s, const int32_t* indices, const int64_t* offsets, const float* weights,
                    int64_t B, const SliceOrder& so, float* out, uint32_t* flags, PoolArgs* a);
int pool_grid(const PoolSetup& s, int64_t nruns, const PoolVariant& k, int block, int out_floats);

// Status word layout (int32[4]) and its initial value.
enum { ST_TIMED_OUT = 0, ST_FIRST_MISSING = 1, ST_OVERSHOOT = 2, ST_FIRST_BAD_BAG = 3 };
constexpr int32_t kStatusInit[4] = {0, 0x7fffffff, 0, 0x7fffffff};

// Error reporting shared by every entry point (thread-local message).
int fail(int code, const char* fmt, ...);
void clear_error();

// Lookups a pooling wave stages in LDS at once.  With weights the general
// kernel takes fewer, so that four waves' slots and a run's tile of 16 KiB fit
// five times into a CU's 160 KiB, as its registers do: 8 fp16 tables of 1008-byte
// rows that fit the caches, weighted bags of 1 to 100: 231 us with four workgroups
// a CU, 190 us with five.
constexpr int pool_staged(bool any, bool weighted) { return any && weighted ? 448 : 512; }
// Words behind the last slot: a row group may read up to 63 entries past the
// last index (what it reads there is not used), in the other slots the next
// wave's.  A tail in each slot left no room for a second workgroup of 16 waves
// with weights and a tile of 8 KiB: 77 us against 49 us, 8 fp32 tables of 512-byte
// rows, bags of 0 to 3.
constexpr int kPoolSlotTail = 64;

// LDS of a pooling workgroup: the run-arrival counter and the ticket's
// broadcast slot (16 bytes), a staging slot per wave, the tail, the run's tile.
constexpr size_t pool_lds_bytes(bool any, bool weighted, int waves, int out_floats) {
  return 16 + (size_t)waves * pool_staged(any, weighted) * (weighted ? 8 : 4) + (size_t)(kPoolSlotTail + out_floats) * 4;
}

hipError_t launch_pool(const PoolVariant& k, const PoolArgs& a, int grid, int block, hipStream_t stream);
int pool_max_wgs_per_cu(const PoolVariant& k, int block, int out_floats);

}  // namespace ebag
