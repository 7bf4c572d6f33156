// Embedding-bag pooling kernels for gfx950.  Templates over the storage type;
// each type's kernels are instantiated in source files of their own (pool_f32.hip,
// pool_wide_f32.hip, ...), which compile side by side.
//
// One wavefront pools whole bags (the paper's "logical workgroup" of the
// EmbeddingBag kernel, Sec. III-A), a contiguous block of them.  A workgroup
// takes a *run* of up to K consecutive samples of one table inside one slice and
// its waves share the run's bags; after the run the workgroup bumps that slice's counter once,
// and the arrival that completes the slice releases the slice's flag
// (Sec. III-A, "Book-keeping Flags").
//
// Gather: a row of D_t elements is V = D_t*elt/16 sixteen-byte vectors.  For
// V a power of two <= 64 the 64 lanes form G = 64/V row groups, lane (g, v)
// loads vector v of rows g, g+G, g+2G, ... so one wave instruction fetches G
// whole rows (1 KiB) with fully coalesced 16-byte loads; every wave keeps U
// such loads in flight.  A wave's block of bags has its index run staged in
// LDS with coalesced loads and read back by broadcast.  Partial sums of the G
// groups are combined across lanes.
//
// The U loads in flight are the next ones of the wave's whole block, of one bag
// or of several (gather_bags); each pooled row goes to an LDS tile of the run;
// the last wave of the workgroup to finish writes the whole run to its
// destination slots with contiguous 16-byte stores, waits for them and updates
// the slice counter -- no workgroup barrier, and no store queued ahead of a
// gather load.  Tables below 4 GiB with V = 2^k and no index report take the
// fast kernel (FastTable).  Any others take the general one: V <= 32 G = 64/V
// rounded down (AnyTable), wider rows 64 vectors at a time, a row a load
// (WideTable), V > 64 stored directly; its waves store their own bags, from the
// tile where V <= 64.
// Long bags are bound by the memory system (512-byte rows arrive at the rate of
// a random-row read probe); short ones by the waves in flight and by
// instructions issued per bag, which is why the run's decoding divides by
// multiplication, the kernel's arguments are re-read instead of kept
// (late_args) and groups combine without LDS.  Measured at 26 tables x 16384
// bags of 0 to 3 rows of 512 bytes (547 MB): 188 us with one bag at a time and
// 81 vector registers (5 waves per SIMD), 112 us with 59 (8 waves), 4.9 TB/s;
// 24 to 64 rows a bag are level (within 0.5% on the same buffers).  Vector
// registers at U = 8, plain and weighted: fp32 59 and 68, fp16 65 and 72, bf16 64
// and 71 (8 waves up to 64, 7 up to 72; above 96 scalar registers 7); general, narrow:
// 69 and 77, 78 and 86, 77 and 82; wide: 82 and 89, 86 and 91, 85 and 91.
//
// Run order (run_at): by default runs are numbered slice-major (all runs of
// slice 0, then slice 1 ...), tables fastest inside a slice, so slices
// complete progressively and a consumer can drain them while later slices
// are still being pooled.  Table-major order pools one table at a time, on
// each XCD separately (table_major = 1: the table's hot rows stay in that
// XCD's L2) or on the whole device (table_major = 2: the table shares the
// Infinity Cache); with per-table slices those still complete progressively.
#pragma once

#include "common.h"

namespace ebag {
namespace {

typedef uint32_t u4v __attribute__((ext_vector_type(4)));

struct EF32 { static constexpr int EPV = 4; };
struct EF16 { static constexpr int EPV = 8; };
struct EBF16 { static constexpr int EPV = 8; };

template <class E> struct Widen;

template <> struct Widen<EF32> {
  template <bool WT>
  static __device__ __forceinline__ void add(float* acc, const u4v& r, float w) {
    const float x[4] = {__uint_as_float(r.x), __uint_as_float(r.y), __uint_as_float(r.z), __uint_as_float(r.w)};
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] = WT ? __builtin_fmaf(w, x[e], acc[e]) : acc[e] + x[e];
  }
};

__device__ __forceinline__ float h2f(uint32_t bits16) {
  return (float)__builtin_bit_cast(_Float16, (uint16_t)bits16);
}

// fp16 rows: every element goes through one fma(w, widen(h), acc), also
// without weights.  There the caller's w is 1 for a row it loaded and 0 for a
// slot it left empty (whose row bits are zero), a value the compiler cannot
// fold, so it emits one mixed-precision FMA per element (the fp16 operand is
// widened inside the instruction) instead of a convert and an add.  Since
// 1 * x and 0 * (+0) are exact, the single rounding gives the bits acc + x and
// acc + 0 would: the result does not change, only the instruction count.
template <> struct Widen<EF16> {
  template <bool WT>
  static __device__ __forceinline__ void add(float* acc, const u4v& r, float w) {
    const uint32_t u[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float lo = h2f(u[e] & 0xffffu), hi = h2f(u[e] >> 16);
      acc[2 * e] = __builtin_fmaf(w, lo, acc[2 * e]);
      acc[2 * e + 1] = __builtin_fmaf(w, hi, acc[2 * e + 1]);
    }
  }
};

template <> struct Widen<EBF16> {
  template <bool WT>
  static __device__ __forceinline__ void add(float* acc, const u4v& r, float w) {
    const uint32_t u[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float lo = __uint_as_float(u[e] << 16), hi = __uint_as_float(u[e] & 0xffff0000u);
      acc[2 * e] = WT ? __builtin_fmaf(w, lo, acc[2 * e]) : acc[2 * e] + lo;
      acc[2 * e + 1] = WT ? __builtin_fmaf(w, hi, acc[2 * e + 1]) : acc[2 * e + 1] + hi;
    }
  }
};

// LDS written by some lanes of a wave and read by others: keep the compiler
// from reordering across this point and wait for the LDS writes.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Table rows live in global memory; say so, so the loads are global_load
// (vmcnt only) rather than flat loads that would also hold up LDS reads.
typedef __attribute__((address_space(1))) const u4v gu4v;
constexpr int kBufferWord3 = 0x00020000;  // raw buffer, 32-bit data format

// Output stores go through a buffer descriptor spanning exactly the pooled rows
// stored (out-of-range lanes are dropped by the hardware).  sc1 = 1 gives
// device-scope stores: they complete at device scope, so a release needs no
// L2 writeback for them; sc1 = 0 gives plain write-back stores.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(float* row, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(row, 0, bytes, kBufferWord3);
}

__device__ __forceinline__ void store16(__amdgpu_buffer_rsrc_t r, int off, float a, float b, float c, float d,
                                        bool sc1) {
  const u4v x = {__float_as_uint(a), __float_as_uint(b), __float_as_uint(c), __float_as_uint(d)};
  if (sc1)
    __builtin_amdgcn_raw_buffer_store_b128(x, r, off, 0, 16);
  else
    __builtin_amdgcn_raw_buffer_store_b128(x, r, off, 0, 0);
}

// Read-only inputs read with wave-uniform addresses (table order, table
// constants and pointers, CSR offsets) go through the scalar data cache:
// their latency then does not queue behind the row gathers in the vector
// memory pipeline.  Nothing the kernel writes is read this way.
template <class T>
__device__ __forceinline__ T sload(const T* p, int64_t i) {
  return ((const __attribute__((address_space(4))) T*)p)[i];
}

__device__ __forceinline__ TabMeta load_meta(const TabMeta* p) {
  TabMeta m;
  m.rows = sload(&p->rows, 0);
  m.row_bytes = sload(&p->row_bytes, 0);
  m.dim = sload(&p->dim, 0);
  m.col_off = sload(&p->col_off, 0);
  m.vecs = sload(&p->vecs, 0);
  m.vshift = sload(&p->vshift, 0);
  return m;
}

// Combine the G = 64 >> vs row groups of a wave: every lane of group 0 ends
// with the sum over the groups, added pairwise from the farthest (lane xor 32)
// to the nearest.  Lane moves inside the vector unit (row swaps and rotations)
// instead of LDS permutes: after the first two steps all rows of 16 lanes hold
// the same values, and after a rotation by 8 (4, 2, 1) they repeat with that
// period, so each rotation fetches the value of lane xor 8 (4, 2, 1).
template <int EPV>
__device__ __forceinline__ void reduce_groups(float* acc, int vs) {
  if (vs > 5) return;
#pragma unroll
  for (int e = 0; e < EPV; ++e) {
    const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[e]), __float_as_uint(acc[e]), false, false);
    acc[e] = __uint_as_float(p[0]) + __uint_as_float(p[1]);
  }
  if (vs > 4) return;
#pragma unroll
  for (int e = 0; e < EPV; ++e) {
    const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(acc[e]), __float_as_uint(acc[e]), false, false);
    acc[e] = __uint_as_float(p[0]) + __uint_as_float(p[1]);
  }
  if (vs > 3) return;
#pragma unroll
  for (int e = 0; e < EPV; ++e)
    acc[e] += __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(acc[e]), 0x128, 0xf, 0xf, true));  // row_ror:8
  if (vs > 2) return;
#pragma unroll
  for (int e = 0; e < EPV; ++e)
    acc[e] += __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(acc[e]), 0x124, 0xf, 0xf, true));  // row_ror:4
  if (vs > 1) return;
#pragma unroll
  for (int e = 0; e < EPV; ++e)
    acc[e] += __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(acc[e]), 0x122, 0xf, 0xf, true));  // row_ror:2
  if (vs > 0) return;
#pragma unroll
  for (int e = 0; e < EPV; ++e)
    acc[e] += __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(acc[e]), 0x121, 0xf, 0xf, true));  // row_ror:1
}

// Stage indices (and weights, S words behind them) [base, base + n) into this
// wave's LDS slot, n <= S, 64 at a time through buffer descriptors: the
// tail's range check costs no instruction, so a block of a few lookups is one
// load and one LDS write.
template <bool WT, int S>
__device__ __forceinline__ void stage_block(const int32_t* idx, const float* wts, int64_t base, int n, int lane,
                                            int32_t* slot) {
  const __amdgpu_buffer_rsrc_t ri =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(idx + base), 0, n * 4, kBufferWord3);
  const __amdgpu_buffer_rsrc_t rw =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(WT ? wts + base : nullptr), 0, WT ? n * 4 : 0, kBufferWord3);
  for (int i0 = 0; i0 < n; i0 += 256) {
    uint32_t x[4], y[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (u > 0 && i0 + 64 * u >= n) continue;
      x[u] = __builtin_amdgcn_raw_buffer_load_b32(ri, (i0 + 64 * u + lane) * 4, 0, 0);
      if (WT) y[u] = __builtin_amdgcn_raw_buffer_load_b32(rw, (i0 + 64 * u + lane) * 4, 0, 0);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (u > 0 && i0 + 64 * u >= n) continue;
      slot[i0 + 64 * u + lane] = (int32_t)x[u];
      if (WT) slot[S + i0 + 64 * u + lane] = (int32_t)y[u];
    }
  }
}

// The kernel's arguments, read again from the kernel argument segment wherever
// this is called.  The compiler otherwise loads all of them at the top and
// keeps them (over fifty scalar registers, beyond what the kernel has left),
// spilling scalars into the vector registers that bound the waves per SIMD.
__device__ __forceinline__ const PoolArgs& late_args() {
  typedef const __attribute__((address_space(4))) PoolArgs KernArgs;
  KernArgs* p = (KernArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const PoolArgs*)p;
}

// This lane's part of a pooled row, into the run's LDS tile.
template <int EPV>
__device__ __forceinline__ void put_tile(float* lrow, const float* acc) {
  float4* d = reinterpret_cast<float4*>(lrow);
#pragma unroll
  for (int h = 0; h < EPV / 4; ++h) d[h] = make_float4(acc[4 * h], acc[4 * h + 1], acc[4 * h + 2], acc[4 * h + 3]);
}

// One table's rows as the lanes of a wave read them: lane (g, v) takes vector v
// of a row of group g, G = 64 / V groups (rounded down; the lanes left over read
// nothing).  A pooled row leaves through emit(): to the run's LDS tile (lrow:
// this lane's vector of the next bag's row), or where a row has more than 64
// vectors and takes several column blocks, straight to its destination.
//
// Fast tables (below 4 GiB, rows of 2^k <= 64 vectors, no index report): loads
// go through a buffer descriptor covering exactly the table.  32-bit offsets
// keep one address register per load instead of two, and the hardware range
// check turns any offset past the table into zeros, so even invalid indices
// cannot read outside it.  NT: non-temporal (streaming) loads -- rows that will
// not be read again do not displace reusable lines (such as the pooled output
// being written) from L2 and the Infinity Cache.
template <int EPV, bool NT>
struct FastTable {
  static constexpr bool CHECKS = false, WIDE = false;
  __amdgpu_buffer_rsrc_t rs;
  uint32_t col;  // byte offset of this lane's 16-byte vector inside a row
  int vs;        // log2 of the vectors per row
  int g;
  float* lrow;
  int dim;
  __device__ __forceinline__ void init(const void* tab, const TabMeta& m, int, int lane) {
    rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(tab), 0, (int)(uint32_t)(m.rows * m.row_bytes),
                                           kBufferWord3);
    vs = m.vshift;
    g = lane >> vs;
    col = (uint32_t)(lane & ((1 << vs) - 1)) * 16u;
    dim = m.dim;
  }
  __device__ __forceinline__ int groups() const { return 64 >> vs; }
  __device__ __forceinline__ int vector(int lane) const { return lane & ((1 << vs) - 1); }
  __device__ __forceinline__ int few() const { return 0; }
  __device__ __forceinline__ int slot_lane() const { return g; }
  // Zeros, and no memory access, in lanes past the bag's end: their offset is
  // past any table.
  __device__ __forceinline__ u4v load(int32_t r, int left, bool*) const {
    return __builtin_amdgcn_raw_buffer_load_b128(rs, g < left ? ((uint32_t)r << (vs + 4)) + col : 0xFFFFFFF0u, 0,
                                                 NT ? 2 : 0);
  }
  __device__ __forceinline__ void emit(float* acc) {
    reduce_groups<EPV>(acc, vs);
    if (g == 0) put_tile<EPV>(lrow, acc);
    lrow += dim;
  }
};

// Where the general kernel's pooled rows go that bypass the run's tile: straight
// to their destination, a column block of vb vectors from `first` at a time.
template <int EPV, bool FUSED>
struct DirectRows {
  int first, dim, t;  // first vector, floats of a row, table
  int64_t bag;        // the next bag's sample
  const float* len;   // and, mean pooling, its length
  // acc: vector v of the row, in the lanes that hold one (on).
  __device__ __forceinline__ void store(float* acc, int v, bool on) {
    const PoolArgs& a = late_args();
    if (a.mean) {
      const float d = *len;
#pragma unroll
      for (int e = 0; e < EPV; ++e) acc[e] = d > 0.f ? acc[e] / d : acc[e];
    }
    const int col_off = sload(&a.meta[t].col_off, 0);
    float* row = a.out + (FUSED ? bag * a.sum_dim + col_off : a.B * col_off + bag * dim);
    if (on) {
      const __amdgpu_buffer_rsrc_t rs = row_rsrc(row, dim * 4);
#pragma unroll
      for (int h = 0; h < EPV / 4; ++h)
        store16(rs, ((first + v) * EPV + 4 * h) * 4, acc[4 * h], acc[4 * h + 1], acc[4 * h + 2], acc[4 * h + 3],
                FUSED && a.release_mode == 1);
    }
    ++bag;
    ++len;
  }
};

// Rows of at most 32 vectors of any table, or (WITH_WIDE: not of a narrow plan)
// the last column block, of at most 32 vectors, of wider ones: any width, 64-bit
// addresses, indices checked against the table (a row out of range is skipped, and
// reported by the caller when the plan asks for it).  Measured on 24 fp16 tables of
// 96 to 640-byte rows, bags of 1 to 40 (0.94 GB): 292 us with one row a load and
// one bag at a time, 236 us like this -- its rows touch 8.7 M cache lines, which
// random reads return in about 175 us; reading tables below 4 GiB through a buffer
// descriptor here too left it at 236 us.  Four fp32 tables of 5.1 GB, mean of 1 to
// 40 rows of 512 bytes (0.72 GB): 156 us before, 141 us.
template <int EPV, bool NT, bool FUSED, bool WITH_WIDE>
struct AnyTable {
  static constexpr bool CHECKS = true, WIDE = false;
  const char* colp;   // this lane's vector of row 0
  uint32_t rows, rb;
  int vb, G, g, v;    // g: beyond any bag in the lanes left over
  int few_rows;
  bool tile;          // a whole row: leaves through the LDS tile
  float* lrow;
  int dim;
  DirectRows<EPV, FUSED> direct;
  __device__ __forceinline__ void init(const void* tab, const TabMeta& m, int block, int lane) {
    rows = (uint32_t)m.rows;
    rb = (uint32_t)m.row_bytes;
    dim = m.dim;
    vb = m.vecs - block;
    G = (int)(64u / (unsigned)vb);
    g = (int)((unsigned)lane / (unsigned)vb);
    v = lane - g * vb;
    if (g >= G) g = 1 << 20;
    colp = static_cast<const char*>(tab) + (int64_t)(block + v) * 16;
    tile = block == 0;
    few_rows = m.vshift < 0 ? 7 : 0;
  }
  __device__ __forceinline__ int groups() const { return G; }
  __device__ __forceinline__ int vector(int) const { return v; }
  // Weighted bags of fewer lookups are added row after row in every column block
  // of a row that is no power of two of vectors: every product is rounded by
  // itself when rows go side by side, once with its sum when they follow each
  // other.  In units of one product's rounding variance, side by side over six
  // groups or more against in sequence: 4 and 3 for 2 rows, 22 and 21 for 6, 27 and
  // 28 for 7.  With fewer groups it is level sooner (2 groups at 4 rows, 3 at
  // 5); 7 holds for every width.  Bags of 1 to 3 lookups: 3.3e-8 off the sum in 64
  // bits in sequence, 3.9e-8 side by side.  Rows of 2^k vectors go side by side
  // whatever the kernel.
  __device__ __forceinline__ int few() const { return few_rows; }
  __device__ __forceinline__ int slot_lane() const { return g < G ? g : 0; }
  __device__ __forceinline__ u4v load(int32_t r, int left, bool* bad) const {
    const bool in = (uint32_t)r < rows;
    *bad = g < left && !in;
    u4v x = {0u, 0u, 0u, 0u};
    if (g < left && in) {
      gu4v* p = (gu4v*)(colp + (uint64_t)(uint32_t)r * rb);
      x = NT ? __builtin_nontemporal_load(p) : *p;
    }
    return x;
  }
  __device__ __forceinline__ void emit(float* acc) {
    for (int s = 32; s > 0; s >>= 1) {  // group g < s takes in group g + s, farthest first
      if (s >= G) continue;
      const bool take = g < s && g + s < G;
#pragma unroll
      for (int e = 0; e < EPV; ++e) {
        const float x = __shfl(acc[e], (int)(threadIdx.x & 63) + s * vb);
        acc[e] = take ? acc[e] + x : acc[e];
      }
    }
    if (WITH_WIDE && !tile) {
      direct.store(acc, v, g == 0);
      return;
    }
    if (g == 0) put_tile<EPV>(lrow, acc);
    lrow += dim;
  }
};

// Rows of more than 32 vectors of any table, 64 at a time: a row (a column block
// of it) takes the whole wave, so a load is one lookup (gather_rows).
template <int EPV, bool NT, bool FUSED>
struct WideTable {
  static constexpr bool CHECKS = true, WIDE = true;
  const char* colp;   // this lane's vector of row 0
  uint32_t rows, rb;
  int vb, v;
  bool tile;          // a whole row: leaves through the LDS tile
  float* lrow;
  DirectRows<EPV, FUSED> direct;
  __device__ __forceinline__ void init(const void* tab, const TabMeta& m, int block, int lane) {
    rows = (uint32_t)m.rows;
    rb = (uint32_t)m.row_bytes;
    vb = min(64, m.vecs - block);
    v = lane;
    tile = m.vecs <= 64;
    colp = static_cast<const char*>(tab) + (int64_t)(block + lane) * 16;
  }
  __device__ __forceinline__ int vector(int) const { return v; }
  __device__ __forceinline__ bool active() const { return v < vb; }  // lanes that hold a vector
  __device__ __forceinline__ u4v load(uint32_t r) const {
    gu4v* p = (gu4v*)(colp + (uint64_t)r * rb);
    return NT ? __builtin_nontemporal_load(p) : *p;
  }
  __device__ __forceinline__ void emit(float* acc) {
    if (tile) {
      put_tile<EPV>(lrow, acc);
      lrow += direct.dim;
    } else {
      direct.store(acc, v, true);
    }
  }
};

// Gather the bags of one staged block: lane i < c <= 63 holds bag i as first
// staged lookup << 16 | lookups (0 in lanes >= c).  Lane (g, v) takes vector v
// of rows g, g + G, ... of each bag; G consecutive rows of one bag are one load
// instruction.  The wave walks these groups of all its bags in order, U at a
// time, whatever bags they belong to: all U loads are in flight before the
// first is added, so bags shorter than U * G rows do not leave the wave with a
// load or two in flight and a round trip to memory per bag.  The bookkeeping
// is wave-uniform (scalar registers); a lane past its bag's end loads nothing
// and adds zeros.  A bag's rows are added in the order of its own lookups, so
// the result does not depend on how bags share a wave.  After a bag's last
// group its row is emitted; closes = false: the block is a piece of one long
// bag, which goes on.  A bag with an index out of range reports itself: bad
// carries over the pieces of one bag, report is the first bag's number (or
// nullptr status).
template <class E, int U, bool WT, int S, class Table>
__device__ __forceinline__ void gather_bags(Table& tb, int c, uint32_t bags, const int32_t* slot, int lane,
                                            bool closes, float* acc, int32_t* status, int64_t report, bool* carry) {
  constexpr int EPV = E::EPV;
  const int G = tb.groups();
  const int g = tb.g;
  const int few = WT && Table::CHECKS ? tb.few() : 0;
  const int32_t* lg = slot + tb.slot_lane();
  // fp16 rows are widened inside a multiply-add by one; the compiler must not
  // see that it is one, or it would widen and add in two instructions.
  float one = 1.f;
  asm("" : "+v"(one));
  int bag = 0;
  uint32_t b = __builtin_amdgcn_readlane(bags, 0);
  int pos = b >> 16, n = b & 0xffff;  // next staged lookup of the bag, lookups left
  int step = n < few ? 1 : G;         // rows of this bag per load
  while (bag < c) {
    int32_t r[U];
    float wv[U];
    int cnt[U];
    uint32_t ends = 0, bads = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      cnt[u] = few ? min(n, step) : n;
      r[u] = lg[pos];
      wv[u] = WT ? (g < cnt[u] ? __int_as_float(lg[S + pos]) : 0.f) : one;
      pos += step;
      n -= step;
      if (n <= 0) {
        ends |= bag < c ? 1u << u : 0u;
        ++bag;
        b = __builtin_amdgcn_readlane(bags, min(bag, 63));  // lane 63 holds no bag
        pos = b >> 16;
        n = b & 0xffff;
        step = n < few ? 1 : G;
      }
    }
    u4v raw[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      raw[u] = u4v{0u, 0u, 0u, 0u};
      if (cnt[u] > 0) {  // empty bags and the block's end skip
        bool bad = false;
        raw[u] = tb.load(r[u], cnt[u], &bad);
        if (Table::CHECKS && WT) wv[u] = bad ? 0.f : wv[u];  // left out, whatever its weight
        if (Table::CHECKS && status) bads |= __any(bad) ? 1u << u : 0u;
      }
    }
    if (!closes) ends = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      Widen<E>::template add<WT>(acc, raw[u], wv[u]);
      if (Table::CHECKS) *carry |= bads >> u & 1u;
      if (ends >> u & 1u) {
        tb.emit(acc);
#pragma unroll
        for (int e = 0; e < EPV; ++e) acc[e] = 0.f;
        if (Table::CHECKS) {
          if (*carry && lane == 0) atomicMin(&status[ST_FIRST_BAD_BAG], (int32_t)report);
          *carry = false;
          ++report;
        }
      }
    }
  }
}

// gather_bags where a row takes the whole wave: a load is one staged lookup, so
// a block's loads are its lookups in order, whatever bags they belong to, and
// need none of the bookkeeping of groups.  A chunk of U lookups whose rows are all
// in the table is checked once, by its largest index.  Rows that come from the
// caches are bound by the instructions issued per row: 8 fp32 tables of 1008-byte
// rows that fit them, weighted bags of 1 to 100, 209 us in gather_bags and 135 us
// here (138 us one bag at a time without any check); that do not, 489 us and 494
// us (514 us).
template <class E, int U, bool WT, int S, class Table>
__device__ __forceinline__ void gather_rows(Table& tb, int c, uint32_t bags, const int32_t* slot, int lane,
                                            bool closes, float* acc, int32_t* status, int64_t report, bool* carry) {
  const uint32_t ends = (bags >> 16) + (bags & 0xffff);
  const int total = __builtin_amdgcn_readlane(ends, c - 1);
  float one = 1.f;  // as in gather_bags
  asm("" : "+v"(one));
  int bag = closes ? 0 : c;
  int end = __builtin_amdgcn_readlane(ends, 0);  // lookups up to the bag's last
  // With k lookups added: the bags that end there.
  const auto close = [&](int k) __attribute__((always_inline)) {
    while (bag < c && end <= k) {
      if (tb.active()) tb.emit(acc);
#pragma unroll
      for (int e = 0; e < E::EPV; ++e) acc[e] = 0.f;
      if (*carry && lane == 0) atomicMin(&status[ST_FIRST_BAD_BAG], (int32_t)(report + bag));
      *carry = false;
      ++bag;
      end = __builtin_amdgcn_readlane(ends, min(bag, 63));
    }
  };
  close(0);
  for (int k0 = 0; k0 < total; k0 += U) {
    uint32_t r[U], most = 0;
    float wv[U];
    uint32_t bads = 0;
#pragma unroll
    for (int u = 0; u < U; u += 4) {
      const u4v x = *reinterpret_cast<const u4v*>(slot + k0 + u);
      r[u] = x.x, r[u + 1] = x.y, r[u + 2] = x.z, r[u + 3] = x.w;
      const u4v y = WT ? *reinterpret_cast<const u4v*>(slot + S + k0 + u) : u4v{0u, 0u, 0u, 0u};
      wv[u] = WT ? __uint_as_float(y.x) : one, wv[u + 1] = WT ? __uint_as_float(y.y) : one;
      wv[u + 2] = WT ? __uint_as_float(y.z) : one, wv[u + 3] = WT ? __uint_as_float(y.w) : one;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) most = max(most, r[u]);
    u4v raw[U];
    if (k0 + U <= total && (uint32_t)__builtin_amdgcn_readfirstlane(most) < tb.rows) {
      if (tb.active()) {
#pragma unroll
        for (int u = 0; u < U; ++u) raw[u] = tb.load(r[u]);
      }
    } else {  // the block's end, or a row out of range, which is left out whatever its weight
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const bool on = k0 + u < total, in = on && r[u] < tb.rows;
        raw[u] = u4v{0u, 0u, 0u, 0u};
        if (in && tb.active()) raw[u] = tb.load(r[u]);
        if (WT) wv[u] = in ? wv[u] : 0.f;
        if (status) bads |= __any(on && !in) ? 1u << u : 0u;
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      Widen<E>::template add<WT>(acc, raw[u], wv[u]);
      *carry |= bads >> u & 1u;
      close(k0 + u + 1);
    }
  }
}

// Write nb pooled rows of dim floats from LDS to global rows base + i * stride:
// 64 lanes x 16 bytes per instruction, each row contiguous; a lane steps its
// (row, vector) by 64 vectors; P2: dim is a power of two.  len:
// mean pooling in the general kernel -- row i is divided by len[i] (an IEEE
// division) on the way, once per stored value rather than at each bag's end in
// the gather loop.
template <bool P2>
__device__ __forceinline__ void store_rows(const float* lds, const float* len, int nb, float* base, int64_t stride,
                                           int dim, int lane, bool sc1) {
  const unsigned n4 = (unsigned)dim >> 2;
  const int64_t span = ((int64_t)(nb - 1) * stride + dim) * 4;
  const __amdgpu_buffer_rsrc_t rs = row_rsrc(base, (int)span);
  const float4* l4 = reinterpret_cast<const float4*>(lds);
  const int total = nb * (int)n4;
  const int s4 = P2 ? __builtin_ctz(n4) : 0;
  const int dr = (int)(P2 ? 64u >> s4 : 64u / n4), dc = (int)(64u - dr * n4);
  int i = (int)(P2 ? (unsigned)lane >> s4 : (unsigned)lane / n4), c4 = lane - i * (int)n4;
  for (int e = lane; e < total; e += 64) {
    float4 x = l4[e];
    if (len) {
      const float d = len[i];
      if (d > 0.f) x = make_float4(x.x / d, x.y / d, x.z / d, x.w / d);
    }
    store16(rs, (int)((uint32_t)i * (uint32_t)(stride * 4)) + c4 * 16, x.x, x.y, x.z, x.w, sc1);
    i += dr;
    c4 += dc;
    if (c4 >= (int)n4) {
      c4 -= (int)n4;
      ++i;
    }
  }
}

// Completion of one run (fused only).  release_mode 0: the workgroup's
// stores are published by an agent-scope release on the slice counter (an L2
// writeback on every run).  release_mode 1: the pooled vectors were stored
// with device-scope stores, and the waves that stored them waited for them to
// complete at device scope (vmcnt 0) before this, so the counter update needs no
// cache writeback.  The arrival that completes the slice re-arms the counter and
// increments the slice flag.
__device__ __forceinline__ void release_slice(uint32_t* counters, uint32_t* flags, int64_t g, uint32_t n,
                                              uint32_t target, int64_t suppress, uint64_t* trace, int mode,
                                              int counter_shift) {
  uint32_t* counter = counters + (g << counter_shift);
  uint32_t old;
  if (mode == 0)
    old = __hip_atomic_fetch_add(counter, n, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
  else
    old = __hip_atomic_fetch_add(counter, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (old + n == target) {
    if (mode == 0) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (trace) trace[g] = wall_clock64();
    if (g != suppress) {
      if (mode == 0)
        __hip_atomic_fetch_add(&flags[g], 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
      else
        __hip_atomic_fetch_add(&flags[g], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// s_waitcnt vmcnt(0): every vector memory operation of this wave, stores
// included, has completed (for device-scope stores: at device scope).
__device__ __forceinline__ void wait_stores_complete() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// Persistent grid: workgroups claim runs in production order from an atomic
// ticket (ticket[0]).  The leading barrier makes sure every wave is done with
// the previous run (its LDS tile and the broadcast slot) before the slot is
// rewritten.
__device__ __forceinline__ int64_t draw_run(uint32_t* ticket, uint32_t* s_tick) {
  __syncthreads();
  if (threadIdx.x == 0) *s_tick = __hip_atomic_fetch_add(&ticket[0], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  return (int64_t)__builtin_amdgcn_readfirstlane(*s_tick);
}

// A workgroup whose draw came back past the last run counts itself out in
// ticket[1]; the last one re-arms both words for the next launch.  Every
// workgroup's final draw has returned (its value decided the exit) before it
// counts itself out, so no draw of this launch can follow the re-arm.
__device__ __forceinline__ void leave_runs(uint32_t* ticket) {
  if (threadIdx.x == 0 &&
      __hip_atomic_fetch_add(&ticket[1], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1) {
    __hip_atomic_store(&ticket[0], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&ticket[1], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Mean pooling in the fast kernel: nb pooled rows of dim = 2^k floats in the
// tile, row i divided by len[i] (an IEEE division, so an exact fp32 sum gives the
// correctly rounded mean), by the wave that pooled them.  Left to the wave that
// stores the run, while the others have gone, it held up the run's end: 8 fp16
// tables of 512-byte rows, bags of 1 to 40, 111 us, 109 us like this; of 0 to 3, 32
// us and 28 us.
__device__ __forceinline__ void divide_rows(float* lds, const float* len, int nb, int dim, int lane) {
  const int s4 = __builtin_ctz(dim) - 2;
  float4* l4 = reinterpret_cast<float4*>(lds);
  asm volatile("" : "+v"(lane));  // no register held for this through the gather
  for (int e = lane; e < nb << s4; e += 64) {
    const float d = len[e >> s4];
    const float4 x = l4[e];
    if (d > 0.f) l4[e] = make_float4(x.x / d, x.y / d, x.z / d, x.w / d);
  }
}

// A wave's bags [wid * per, ...) of a run, in blocks of at most 63: reads the
// block's CSR offsets (one lane each), stages the block's whole index segment
// into the wave's LDS slot when it fits (else bag by bag, S at a time), then
// gathers vectors [first, last) of every bag.  Where one staged block was all of
// the wave's bags, that is returned and *bags is what gather_bags takes for it; a
// call for other vectors of the same bags is then passed both and reads nothing
// again.
template <class E, int U, bool WT, class Table>
__device__ __forceinline__ bool pool_blocks(const PoolArgs& a, const TabMeta& m, const void* tab, int t, int64_t b0,
                                            int nb, int per, int wid, int lane, int32_t* slot, float* lds_out,
                                            int first, int last, bool staged, uint32_t* kept) {
  constexpr int EPV = E::EPV;
  constexpr int S = pool_staged(Table::CHECKS, WT);
  const int64_t bag0 = (int64_t)t * a.B + b0;  // the run's first bag
  const int64_t* offs = a.offsets + bag0;
  float* lens = lds_out + a.out_floats - ((a.K + 3) & ~3);  // mean pooling
  const int end = min((wid + 1) * per, nb);
  float acc[EPV];
#pragma unroll
  for (int e = 0; e < EPV; ++e) acc[e] = 0.f;
  bool whole = false;
  for (int blk = wid * per; blk < end; blk += 63) {
    const int c = min(63, end - blk);
    // Offsets are clamped into [0, nnz] and each bag into the block's
    // segment, so malformed CSR input can never drive a read outside the
    // index array (results are then meaningless but memory-safe).  With
    // index checks a bag of invalid offsets is empty and reported, and its
    // block goes bag by bag, which leaves the valid bags beside it whole.
    int64_t seg_lo = 0, seg_hi = 0;
    bool all = true;  // the block's lookups fit the staging slot
    uint64_t invalid = 0;
    uint32_t packed = *kept;
    if (!staged) {
      const int64_t off = offs[blk + min(lane, c)];
      const int64_t nnz = sload(a.offsets, (int64_t)a.T * a.B);
      seg_lo = min(max(sload(offs, blk), (int64_t)0), nnz);
      seg_hi = min(max(sload(offs, blk + c), seg_lo), nnz);
      all = seg_hi - seg_lo <= S;
      if (Table::CHECKS && a.check) {
        const int64_t next = __shfl_down(off, 1);
        const bool ok = off >= 0 && off <= next && next <= nnz;
        invalid = __ballot(lane < c && !ok);
        if (lane < c && !ok) atomicMin(&a.status[ST_FIRST_BAD_BAG], (int32_t)(bag0 + blk + lane));
        if (invalid) all = false;
      }
      if (all) stage_block<WT, S>(a.indices, a.weights, seg_lo, (int)(seg_hi - seg_lo), lane, slot);
      const int64_t rel = min(max(off, seg_lo), seg_hi) - seg_lo;
      const int64_t len = max((int64_t)__shfl_down(rel, 1) - rel, (int64_t)0);
      if (a.mean && lane < c) lens[blk + lane] = (float)(int)len;
      packed = all && lane < c ? (uint32_t)rel << 16 | (uint32_t)len : 0u;
    }
    for (int col = first; col < last; col += 64) {
      Table tb;
      tb.init(tab, m, col, lane);
      tb.lrow = lds_out + blk * m.dim + tb.vector(lane) * EPV;
      if constexpr (Table::CHECKS) tb.direct = {col, m.dim, t, b0 + blk, lens + blk};
      bool carry = false;
      int64_t lo = 0, hi = 0;
      for (int i = 0; i < c;) {
        bool closes = true;
        uint32_t bags = packed;
        if (!all) {  // bag by bag, S lookups at a time
          if (lo == hi) {
            lo = sload(offs, blk + i);
            hi = sload(offs, blk + i + 1);
            if (!Table::CHECKS || !a.check) {
              lo = min(max(lo, seg_lo), seg_hi);
              hi = min(max(hi, lo), seg_hi);
            } else if (invalid >> i & 1u) {
              lo = hi = 0;
            }
            if (Table::CHECKS && a.mean && lane == 0) lens[blk + i] = (float)(int)(hi - lo);
          }
          const int n = (int)min((int64_t)S, hi - lo);
          stage_block<WT, S>(a.indices, a.weights, lo, n, lane, slot);
          bags = lane == 0 ? n : 0;
          lo += n;
          closes = lo == hi;
        }
        int32_t* status = Table::CHECKS && a.check ? a.status : nullptr;
        wave_lds_sync();
        if constexpr (Table::WIDE)
          gather_rows<E, U, WT, S>(tb, all ? c : 1, bags, slot, lane, closes, acc, status, bag0 + blk + i, &carry);
        else
          gather_bags<E, U, WT, S>(tb, all ? c : 1, bags, slot, lane, closes, acc, status, bag0 + blk + i, &carry);
        wave_lds_sync();
        if (closes) i += all ? c : 1;
      }
    }
    if constexpr (!Table::CHECKS) {
      const PoolArgs& l = late_args();  // nothing of it held through the gather either
      if (l.mean)
        divide_rows(lds_out + blk * m.dim, lds_out + l.out_floats - ((l.K + 3) & ~3) + blk, c, m.dim, lane);
    }
    whole = all && c == end - wid * per;
    *kept = packed;
  }
  return whole;
}

// One workgroup per run of up to K consecutive samples of one table inside one
// slice.  The counter it feeds is the slice's (target C * T bags)
// or, with per-table slices, the (slice, table) pair's (target C bags).  Wave
// w pools a contiguous block of the run's bags (pool_blocks).
template <class E, int U, bool WT, bool NT, bool FUSED, int KIND>
__device__ __forceinline__ void pool_body() {
  constexpr int EPV = E::EPV;
  extern __shared__ int32_t s_dyn[];
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int W = late_args().waves;
  // LDS: the run's arrival counter and the ticket's broadcast slot, a staging
  // slot per wave (and one for the weights), the run's pooled rows (K x max
  // dim floats), with mean pooling their K bag lengths.
  int32_t* s_arrive = s_dyn;
  uint32_t* s_tick = reinterpret_cast<uint32_t*>(s_dyn + 1);
  constexpr int slot_words = pool_staged(KIND != POOL_FAST, WT) * (WT ? 2 : 1);
  int32_t* slot = s_dyn + 4 + wid * slot_words;
  float* lds_out = reinterpret_cast<float*>(s_dyn + 4 + W * slot_words + kPoolSlotTail);
  if (threadIdx.x == 0) *s_arrive = 0;
  __syncthreads();
  // One-shot grid: workgroup i pools run i.  Persistent grid (fewer
  // workgroups than runs): runs are claimed from the ticket.
  const bool persistent = gridDim.x < late_args().nruns;
  for (uint32_t q = persistent ? draw_run(late_args().ticket, s_tick) : blockIdx.x; q < late_args().nruns;
       q = persistent ? draw_run(late_args().ticket, s_tick) : 0x7fffffffu) {
    uint32_t gs, tpos, j;
    int t, nb, per;
    int64_t g, b0;
    {
      const PoolArgs& a = late_args();
      run_at(a.ro, q, &gs, &tpos, &j);
      t = sload(a.tperm, tpos);
      g = slice_at(a.so, gs);
      b0 = g * a.C + (int64_t)j * a.K;
      nb = min(a.K, a.C - (int)j * a.K);
      per = (int)divide_by(a.by_waves, (uint32_t)(nb + W - 1));
    }
    {
      const PoolArgs& a = late_args();
      const TabMeta m = load_meta(a.meta + t);
      const void* tab = sload(a.tables, t);
      if constexpr (KIND == POOL_FAST) {
        uint32_t kept = 0;
        pool_blocks<E, U, WT, FastTable<EPV, NT>>(a, m, tab, t, b0, nb, per, wid, lane, slot, lds_out, 0, 1, false,
                                                  &kept);
      } else {
        // the row's last column block of at most 32 vectors (the whole of a narrow row)
        const int rest = KIND == POOL_NARROW ? m.vecs : (m.vecs & 63) <= 32 ? m.vecs & 63 : 0;
        bool staged = false;
        uint32_t kept = 0;
        if constexpr (KIND == POOL_WIDE)
          if (m.vecs > rest)
            staged = pool_blocks<E, U, WT, WideTable<EPV, NT, FUSED>>(a, m, tab, t, b0, nb, per, wid, lane, slot, lds_out,
                                                                      0, m.vecs - rest, false, &kept);
        if (rest)
          pool_blocks<E, U, WT, AnyTable<EPV, NT, FUSED, KIND == POOL_WIDE>>(a, m, tab, t, b0, nb, per, wid, lane, slot,
                                                                             lds_out, m.vecs - rest, m.vecs, staged, &kept);
      }
    }
    // General kernels: a wave stores its own rows, and they are complete before it
    // arrives.
    if constexpr (KIND != POOL_FAST) {
      const PoolArgs& a = late_args();
      const int dim = sload(&a.meta[t].dim, 0), col_off = sload(&a.meta[t].col_off, 0);
      const int64_t stride = FUSED ? a.sum_dim : dim;
      const int i0 = wid * per, n = min(per, nb - i0);
      if (n > 0 && (KIND == POOL_NARROW || sload(&a.meta[t].vecs, 0) <= 64))
        store_rows<false>(lds_out + i0 * dim, a.mean ? lds_out + a.out_floats - ((a.K + 3) & ~3) + i0 : nullptr, n,
                          a.out + (FUSED ? col_off : a.B * col_off) + (b0 + i0) * stride, stride, dim, lane,
                          FUSED && a.release_mode == 1);
      wait_stores_complete();
    }
    // The last wave to finish its bags (fast kernel) writes the whole run from LDS
    // to global memory and (fused) completes the run for the slice; the other
    // waves leave at once.  No workgroup barrier, and no store ever sits in
    // front of a gather load of the same wave.
    int old = 0;
    if (lane == 0) old = __hip_atomic_fetch_add(s_arrive, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP);
    old = __builtin_amdgcn_readfirstlane(old);
    if (old == W - 1) {
      const PoolArgs& a = late_args();
      if (lane == 0) __hip_atomic_store(s_arrive, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      if constexpr (KIND == POOL_FAST) {
        const int dim = sload(&a.meta[t].dim, 0), col_off = sload(&a.meta[t].col_off, 0);
        const int64_t stride = FUSED ? a.sum_dim : dim;
        store_rows<true>(lds_out, nullptr, nb, a.out + (FUSED ? col_off : a.B * col_off) + b0 * stride, stride, dim,
                         lane, FUSED && a.release_mode == 1);
      }
      if (FUSED) {
        if (a.release_mode == 1) wait_stores_complete();
        if (lane == 0)
          release_slice(a.counters, a.flags, a.per_table ? g * a.T + t : g, (uint32_t)nb,
                        a.per_table ? (uint32_t)a.C : (uint32_t)a.C * (uint32_t)a.T, a.suppress, a.trace_release,
                        a.release_mode, a.counter_shift);
      }
    }
  }
  if (persistent) leave_runs(late_args().ticket);
}

// Fused operator: pooled vectors go straight to the send layout and slices
// are released as they complete.
template <class E, int U, bool WT, bool NT, int KIND>
__global__ __launch_bounds__(1024) void fused_pool_kernel(const PoolArgs a) {
  pool_body<E, U, WT, NT, true, KIND>();
}

// Unfused baseline, first kernel: plain per-table EmbeddingBag output.
template <class E, int U, bool WT, bool NT, int KIND>
__global__ __launch_bounds__(1024) void unfused_pool_kernel(const PoolArgs a) {
  pool_body<E, U, WT, NT, false, KIND>();
}

template <class E, int U, bool WT, bool NT, int KIND>
pool_fn pick_f(const PoolVariant& k) {
  return k.fused ? &fused_pool_kernel<E, U, WT, NT, KIND> : &unfused_pool_kernel<E, U, WT, NT, KIND>;
}

template <class E, int U, bool WT, int KIND>
pool_fn pick_n(const PoolVariant& k) {
  return k.stream_rows ? pick_f<E, U, WT, true, KIND>(k) : pick_f<E, U, WT, false, KIND>(k);
}

template <class E, int U, int KIND>
pool_fn pick_w(const PoolVariant& k) {
  return k.weighted ? pick_n<E, U, true, KIND>(k) : pick_n<E, U, false, KIND>(k);
}

template <class E, int KIND>
pool_fn pick_u(const PoolVariant& k) {
  switch (k.rows_in_flight) {
    case 4: return pick_w<E, 4, KIND>(k);
    case 16: return pick_w<E, 16, KIND>(k);
    default: return pick_w<E, 8, KIND>(k);
  }
}

}  // namespace
}  // namespace ebag
