// Embedding-bag pooling kernels for gfx950.
//
// One wavefront pools one bag at a time (the paper's "logical workgroup" of
// the EmbeddingBag kernel, Sec. III-A).  A workgroup takes a *run* of up to K
// consecutive samples of one table inside one slice and its waves share the
// run's bags; after the run the workgroup bumps that slice's counter once,
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
// Fast path (tables < 4 GiB, V = 2^k, no index checks): the U loads in flight
// are the next ones of the wave's whole block, of one bag or of several
// (gather_bags); each pooled row goes to an LDS tile of the run; the last wave
// of the workgroup to finish writes the whole run to its destination slots
// with contiguous 16-byte stores, waits for them and updates the slice counter
// -- no workgroup barrier, and no store queued ahead of a gather load.
// Long bags are bound by the memory system (512-byte rows arrive at the rate of
// a random-row read probe); short ones by the waves in flight and by
// instructions issued per bag, which is why the run's decoding divides by
// multiplication, the kernel's arguments are re-read instead of kept
// (late_args) and groups combine without LDS.  Measured at 26 tables x 16384
// bags of 0 to 3 rows of 512 bytes (547 MB): 188 us with one bag at a time and
// 81 vector registers (5 waves per SIMD), 112 us with 56 (8 waves), 4.9 TB/s;
// 24 to 64 rows a bag are level within the 2% that buffer placement moves them.
// General path (any width, index checks): per-bag staging, rows stored
// directly, a barrier before the counter update.
//
// Run order (run_at): by default runs are numbered slice-major (all runs of
// slice 0, then slice 1 ...), tables fastest inside a slice, so slices
// complete progressively and a consumer can drain them while later slices
// are still being pooled.  Table-major order pools one table at a time, on
// each XCD separately (table_major = 1: the table's hot rows stay in that
// XCD's L2) or on the whole device (table_major = 2: the table shares the
// Infinity Cache); with per-table slices those still complete progressively.
#include "common.h"

namespace ebag {
namespace {

constexpr int SEG = 128;       // indices staged in LDS per wave per step (general kernels)
constexpr int SEGW = 512;      // indices a wave stages at once for a block of bags (fast kernels)
constexpr int SLOTW = SEGW + 64;  // its LDS slot: a row group may read up to 63 entries past the last index

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

// Mean pooling: divide the bag's pooled sum by its length (div > 0; an IEEE
// division, so an exact fp32 sum gives the correctly rounded mean).
template <int EPV>
__device__ __forceinline__ void divide(float* acc, int div) {
  if (div > 0) {
    const float d = (float)div;
#pragma unroll
    for (int e = 0; e < EPV; ++e) acc[e] = acc[e] / d;
  }
}

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
typedef __attribute__((address_space(1))) const int32_t gint;
typedef __attribute__((address_space(1))) const float gfloat;

__device__ __forceinline__ u4v ld_row(const char* colp, int32_t r, uint32_t row_bytes) {
  return *(gu4v*)(colp + (uint64_t)(uint32_t)r * row_bytes);
}

constexpr int kBufferWord3 = 0x00020000;  // raw buffer, 32-bit data format

// Row loads through a buffer descriptor covering exactly one table (tables
// below 4 GiB): 32-bit offsets keep one address register per load instead
// of two, and the hardware range check turns any offset past the table into
// zeros, so even invalid indices cannot read outside the table.
// NT: non-temporal (streaming) loads -- rows that will not be read again do
// not displace reusable lines (such as the pooled output being written) from
// L2 and the Infinity Cache.
struct BufRows {
  __amdgpu_buffer_rsrc_t rs;
  uint32_t col;  // byte offset of this lane's 16-byte vector inside a row
  int shift;     // log2 of the row bytes
  // Zeros, and no memory access, where !ok: the offset is past any table.
  template <bool NT>
  __device__ __forceinline__ u4v load(int32_t r, bool ok) const {
    return __builtin_amdgcn_raw_buffer_load_b128(rs, ok ? ((uint32_t)r << shift) + col : 0xFFFFFFF0u, 0, NT ? 2 : 0);
  }
};

// Plain 64-bit addressed row loads (any table size).
struct GlobalRows {
  const char* colp;
  uint32_t rb;
  __device__ __forceinline__ u4v load(int32_t r) const { return ld_row(colp, r, rb); }
};

// Output stores go through a buffer descriptor spanning exactly one pooled
// row (out-of-range lanes are dropped by the hardware).  sc1 = 1 gives
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

// Stage indices (and weights) [base, base + n) into this wave's LDS slot
// with coalesced loads.
template <bool WT>
__device__ __forceinline__ void stage(const int32_t* __restrict__ idx, const float* __restrict__ wts, int64_t base,
                                      int n, int lane, int32_t* lds_i, float* lds_w) {
  // Four 64-index loads in flight before the first LDS write.
  for (int i0 = 0; i0 < n; i0 += 256) {
    int32_t x[4];
    float y[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = i0 + 64 * u + lane;
      x[u] = i < n ? ((gint*)idx)[base + i] : 0;
      y[u] = (WT && i < n) ? ((gfloat*)wts)[base + i] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = i0 + 64 * u + lane;
      if (i < n) {
        lds_i[i] = x[u];
        if (WT) lds_w[i] = y[u];
      }
    }
  }
}

// Gather and accumulate n staged rows whose width is V = 2^vs <= 64 vectors:
// lane (g, v) with g = lane >> vs takes vector v of rows g, g + G, ... (G = 64
// / V); U index reads from LDS first (clamped into the staged run, no
// branches), then U predicated 16-byte row loads, then the accumulation.
// Returns true in lanes that met an out-of-range index (CHECK only; such rows
// are skipped).
template <class E, int U, bool WT, bool CHECK, class Rows>
__device__ __forceinline__ bool gather_p2(const Rows& rows_ld, int vs, int64_t rows, const int32_t* li,
                                          const float* lw, int n, int lane, float* acc) {
  const int G = 64 >> vs;
  const int g = lane >> vs;
  bool bad = false;
  for (int k0 = 0; k0 < n; k0 += G * U) {
    int32_t r[U];
    float wv[U];
    bool ok[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = k0 + u * G + g;
      ok[u] = k < n;
      const int kc = ok[u] ? k : n - 1;
      r[u] = li[kc];
      wv[u] = WT ? lw[kc] : 1.f;
    }
    if (CHECK) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const bool in = r[u] >= 0 && (int64_t)r[u] < rows;
        bad |= ok[u] && !in;
        ok[u] = ok[u] && in;
      }
    }
    u4v raw[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      raw[u] = u4v{0u, 0u, 0u, 0u};
      if (ok[u]) raw[u] = rows_ld.load(r[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) Widen<E>::template add<WT>(acc, raw[u], ok[u] ? wv[u] : 0.f);
  }
  return bad;
}

// Any row width: 64-vector column blocks, one row per wave step, indices
// staged SEG at a time.  Used for widths that are not 2^k <= 64 vectors.
template <class E, int U, bool WT>
__device__ __forceinline__ bool pool_bag_generic(const char* __restrict__ tab, const TabMeta& m,
                                                 const int32_t* __restrict__ idx, const float* __restrict__ wts,
                                                 int64_t lo, int L, int32_t* lds_i, float* lds_w, int lane,
                                                 int check, float* __restrict__ orow, bool sc1, int div) {
  constexpr int EPV = E::EPV;
  bool bad = false;
  for (int cb = 0; cb < m.vecs; cb += 64) {
    const int vv = cb + lane;
    const bool act = vv < m.vecs;
    const char* colp = tab + (int64_t)vv * 16;
    float acc[EPV];
#pragma unroll
    for (int e = 0; e < EPV; ++e) acc[e] = 0.f;
    for (int s0 = 0; s0 < L; s0 += SEG) {
      const int n = min(SEG, L - s0);
      stage<WT>(idx, wts, lo + s0, n, lane, lds_i, lds_w);
      wave_lds_sync();
      for (int k0 = 0; k0 < n; k0 += U) {
        int32_t r[U];
        float wv[U];
        bool ok[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int k = k0 + u;
          ok[u] = k < n && act;
          const int kc = k < n ? k : n - 1;
          r[u] = lds_i[kc];
          wv[u] = WT ? lds_w[kc] : 1.f;
        }
        if (check) {
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const bool in = r[u] >= 0 && (int64_t)r[u] < m.rows;
            bad |= ok[u] && !in;
            ok[u] = ok[u] && in;
          }
        }
        u4v raw[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          raw[u] = u4v{0u, 0u, 0u, 0u};
          if (ok[u]) raw[u] = ld_row(colp, r[u], (uint32_t)m.row_bytes);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) Widen<E>::template add<WT>(acc, raw[u], ok[u] ? wv[u] : 0.f);
      }
      wave_lds_sync();
    }
    divide<EPV>(acc, div);
    if (act) {
      const __amdgpu_buffer_rsrc_t rs = row_rsrc(orow, m.dim * 4);
#pragma unroll
      for (int h = 0; h < EPV / 4; ++h)
        store16(rs, (vv * EPV + 4 * h) * 4, acc[4 * h], acc[4 * h + 1], acc[4 * h + 2], acc[4 * h + 3], sc1);
    }
  }
  return bad;
}

// Combine the G row groups (lane bits vs..5) with xor shuffles, then store
// the row with 16-byte stores laid out so that one instruction covers the row
// contiguously: fp32 tables -- lane v of group 0 writes floats [4v, 4v + 4);
// 16-bit tables (8 values per lane) -- groups 0 and 1 write the two halves
// of lane v's 32 bytes (every lane holds the total after the xor butterfly).
template <int EPV>
__device__ __forceinline__ void reduce_store(float* acc, int vs, int lane, float* __restrict__ orow, int dim,
                                             bool sc1, int div) {
  const int V = 1 << vs;
  for (int msk = 32; msk >= V; msk >>= 1) {
#pragma unroll
    for (int e = 0; e < EPV; ++e) acc[e] += __shfl_xor(acc[e], msk);
  }
  divide<EPV>(acc, div);
  const int g = lane >> vs;
  const int v = lane & (V - 1);
  const __amdgpu_buffer_rsrc_t rs = row_rsrc(orow, dim * 4);
  if (EPV == 4) {
    if (g == 0) store16(rs, 16 * v, acc[0], acc[1], acc[2], acc[3], sc1);
  } else if (vs <= 5) {
    if (g < 2) {
      const bool hi = g == 1;
      store16(rs, 32 * v + 16 * g, hi ? acc[4] : acc[0], hi ? acc[5] : acc[1], hi ? acc[6] : acc[2],
              hi ? acc[7] : acc[3], sc1);
    }
  } else {
    store16(rs, 32 * v, acc[0], acc[1], acc[2], acc[3], sc1);
    store16(rs, 32 * v + 16, acc[4], acc[5], acc[6], acc[7], sc1);
  }
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

// Stage indices (and weights, SLOTW words behind them) [base, base + n) into
// this wave's LDS slot, n <= SEGW, 64 at a time through buffer descriptors: the
// tail's range check costs no instruction, so a block of a few lookups is one
// load and one LDS write.
template <bool WT>
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
      if (WT) slot[SLOTW + i0 + 64 * u + lane] = (int32_t)y[u];
    }
  }
}

// Gather the bags of one staged block (rows of V = 2^vs <= 64 vectors): lane i
// < c <= 63 holds bag i as first staged lookup << 16 | lookups (0 in lanes >=
// c).  Lane (g, v) with g = lane >> vs takes vector v of rows g, g + G, ... of
// each bag (G = 64 / V); G consecutive rows of one bag are one load
// instruction.  The wave walks these groups of all its bags in order, U at a
// time, whatever bags they belong to: all U loads are in flight before the
// first is added, so bags shorter than U * G rows do not leave the wave with a
// load or two in flight and a round trip to memory per bag.  The bookkeeping
// is wave-uniform (scalar registers); a lane past its bag's end loads nothing
// and adds zeros.  A bag's rows are added in the order of its own lookups, so
// the result does not depend on how bags share a wave.  After a bag's last
// group the groups are combined and the row is written to lrow (this lane's
// vector of it), one row of dim floats per bag; closes = false: the block is a
// piece of one long bag, which goes on.
template <class E, int U, bool WT, bool NT>
__device__ __forceinline__ void gather_bags(const BufRows& rows_ld, int vs, int c, uint32_t bags, const int32_t* slot,
                                            int lane, bool closes, float* acc, float* lrow, int dim) {
  constexpr int EPV = E::EPV;
  const int G = 64 >> vs;
  const int g = lane >> vs;
  const int32_t* lg = slot + g;
  // fp16 rows are widened inside a multiply-add by one; the compiler must not
  // see that it is one, or it would widen and add in two instructions.
  float one = 1.f;
  asm("" : "+v"(one));
  int bag = 0;
  uint32_t b = __builtin_amdgcn_readlane(bags, 0);
  int pos = b >> 16, n = b & 0xffff;  // next staged lookup of the bag, lookups left
  while (bag < c) {
    int32_t r[U];
    float wv[U];
    int cnt[U];
    uint32_t ends = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      cnt[u] = n;
      r[u] = lg[pos];
      wv[u] = WT ? (g < n ? __int_as_float(lg[SLOTW + pos]) : 0.f) : one;
      pos += G;
      n -= G;
      if (n <= 0) {
        ends |= bag < c ? 1u << u : 0u;
        ++bag;
        b = __builtin_amdgcn_readlane(bags, min(bag, 63));  // lane 63 holds no bag
        pos = b >> 16;
        n = b & 0xffff;
      }
    }
    u4v raw[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      raw[u] = u4v{0u, 0u, 0u, 0u};
      if (cnt[u] > 0) raw[u] = rows_ld.template load<NT>(r[u], g < cnt[u]);  // empty bags and the block's end skip
    }
    if (!closes) ends = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      Widen<E>::template add<WT>(acc, raw[u], wv[u]);
      if (ends >> u & 1u) {
        reduce_groups<EPV>(acc, vs);
        if (g == 0) {
          float4* d = reinterpret_cast<float4*>(lrow);
#pragma unroll
          for (int h = 0; h < EPV / 4; ++h)
            d[h] = make_float4(acc[4 * h], acc[4 * h + 1], acc[4 * h + 2], acc[4 * h + 3]);
        }
        lrow += dim;
#pragma unroll
        for (int e = 0; e < EPV; ++e) acc[e] = 0.f;
      }
    }
  }
}

// Write nb pooled rows of dim floats (dim / 4 = 2^s4 float4s each) from LDS
// to global rows base + i * stride: 64 lanes x 16 bytes per instruction,
// each row contiguous.  len: mean pooling -- row i is divided by len[i] (an
// IEEE division, so an exact fp32 sum gives the correctly rounded mean), once
// per stored value rather than at each bag's end in the gather loop.
__device__ __forceinline__ void store_rows(const float* lds, const float* len, int nb, int s4, float* base,
                                           int64_t stride, int dim, int lane, bool sc1) {
  const int n4 = 1 << s4;
  const int64_t span = ((int64_t)(nb - 1) * stride + dim) * 4;
  const __amdgpu_buffer_rsrc_t rs = row_rsrc(base, (int)span);
  const float4* l4 = reinterpret_cast<const float4*>(lds);
  for (int e = lane; e < (nb << s4); e += 64) {
    const int i = e >> s4;
    const int c4 = e & (n4 - 1);
    float4 x = l4[e];
    if (len) {
      const float d = len[i];
      if (d > 0.f) x = make_float4(x.x / d, x.y / d, x.z / d, x.w / d);
    }
    store16(rs, (int)((uint32_t)i * (uint32_t)(stride * 4)) + c4 * 16, x.x, x.y, x.z, x.w, sc1);
  }
}

// Completion of one run (fused only).  release_mode 0: the workgroup's
// stores are published by an agent-scope release on the slice counter (an L2
// writeback on every run).  release_mode 1: the pooled vectors were stored
// with device-scope stores, each wave waited for them to complete at device
// scope (vmcnt 0) before the barrier, so the counter update needs no cache
// writeback.  The arrival that completes the slice re-arms the counter and
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

// Fast path: one workgroup per run of up to K consecutive samples of one table
// inside one slice.  The counter it feeds is the slice's (target C * T bags)
// or, with per-table slices, the (slice, table) pair's (target C bags).  Wave
// w pools a contiguous block of the run's bags: it reads the block's CSR
// offsets (one lane each), stages the block's whole index segment into its
// LDS slot when it fits (else bag by bag, SEGW at a time), then gathers every
// bag into the run's LDS tile.
template <class E, int U, bool WT, bool NT, bool FUSED>
__device__ __forceinline__ void pool_fast() {
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
  int32_t* slot = s_dyn + 4 + wid * SLOTW * (WT ? 2 : 1);
  float* lds_out = reinterpret_cast<float*>(s_dyn + 4 + W * SLOTW * (WT ? 2 : 1));
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
      BufRows rows_ld;
      rows_ld.rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(sload(a.tables, t)), 0,
                                                     (int)(uint32_t)(m.rows * m.row_bytes), kBufferWord3);
      rows_ld.col = (uint32_t)(lane & ((1 << m.vshift) - 1)) * 16u;
      rows_ld.shift = m.vshift + 4;
      const int64_t nnz = sload(a.offsets, (int64_t)a.T * a.B);
      const int64_t* offs = a.offsets + ((int64_t)t * a.B + b0);  // the run's bags
      const int end = min((wid + 1) * per, nb);
      float* lrow = lds_out + (lane & ((1 << m.vshift) - 1)) * EPV;
      float acc[EPV];
#pragma unroll
      for (int e = 0; e < EPV; ++e) acc[e] = 0.f;
      for (int blk = wid * per; blk < end; blk += 63) {
        const int c = min(63, end - blk);
        // Offsets are clamped into [0, nnz] and each bag into the block's
        // segment, so malformed CSR input can never drive a read outside the
        // index array (results are then meaningless but memory-safe).
        const int64_t off = offs[blk + min(lane, c)];
        const int64_t seg_lo = min(max(sload(offs, blk), (int64_t)0), nnz);
        const int64_t seg_hi = min(max(sload(offs, blk + c), seg_lo), nnz);
        const bool all = seg_hi - seg_lo <= SEGW;  // the block's lookups fit the staging slot
        if (all) stage_block<WT>(a.indices, a.weights, seg_lo, (int)(seg_hi - seg_lo), lane, slot);
        const int64_t rel = min(max(off, seg_lo), seg_hi) - seg_lo;
        const int64_t len = max((int64_t)__shfl_down(rel, 1) - rel, (int64_t)0);
        if (a.mean && lane < c) (lds_out + a.out_floats - ((a.K + 3) & ~3))[blk + lane] = (float)(int)len;
        uint32_t bags = all && lane < c ? (uint32_t)rel << 16 | (uint32_t)len : 0u;
        int64_t lo = 0, hi = 0;
        for (int i = 0; i < c;) {
          bool closes = true;
          if (!all) {  // bag by bag, SEGW lookups at a time
            if (lo == hi) {
              lo = min(max(sload(offs, blk + i), seg_lo), seg_hi);
              hi = min(max(sload(offs, blk + i + 1), lo), seg_hi);
            }
            const int n = (int)min((int64_t)SEGW, hi - lo);
            stage_block<WT>(a.indices, a.weights, lo, n, lane, slot);
            bags = lane == 0 ? n : 0;
            lo += n;
            closes = lo == hi;
          }
          wave_lds_sync();
          gather_bags<E, U, WT, NT>(rows_ld, m.vshift, all ? c : 1, bags, slot, lane, closes, acc,
                                    lrow + (blk + i) * m.dim, m.dim);
          wave_lds_sync();
          if (closes) i += all ? c : 1;
        }
      }
    }
    // The last wave to finish its bags writes the whole run from LDS to
    // global memory and (fused) completes the run for the slice; the other
    // waves leave at once.  No workgroup barrier, and no store ever sits in
    // front of a gather load of the same wave.
    int old = 0;
    if (lane == 0) old = __hip_atomic_fetch_add(s_arrive, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP);
    old = __builtin_amdgcn_readfirstlane(old);
    if (old == W - 1) {
      const PoolArgs& a = late_args();
      if (lane == 0) __hip_atomic_store(s_arrive, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      const int dim = sload(&a.meta[t].dim, 0), col_off = sload(&a.meta[t].col_off, 0);
      const int s4 = sload(&a.meta[t].vshift, 0) + (EPV == 8 ? 1 : 0);
      const int64_t stride = FUSED ? a.sum_dim : dim;
      float* base = a.out + (FUSED ? col_off : a.B * col_off) + b0 * stride;
      store_rows(lds_out, a.mean ? lds_out + a.out_floats - ((a.K + 3) & ~3) : nullptr, nb, s4, base, stride, dim, lane,
                 FUSED && a.release_mode == 1);
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

// General path: any row width, 64-bit addresses, index checks; per-bag
// staging, rows stored directly, a barrier before the counter update.
template <class E, int U, bool WT, bool FUSED>
__device__ __forceinline__ void pool_safe(const PoolArgs& a) {
  constexpr int EPV = E::EPV;
  extern __shared__ int32_t s_dyn[];
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int W = a.waves;
  int32_t* lds_i = s_dyn + wid * SEG;
  float* lds_w = WT ? reinterpret_cast<float*>(s_dyn + W * SEG) + wid * SEG : nullptr;
  const bool sc1 = FUSED && a.release_mode == 1;
  const int64_t nnz = a.check ? sload(a.offsets, (int64_t)a.T * a.B) : 0;
  const bool persistent = gridDim.x < a.nruns;
  uint32_t* s_tick = reinterpret_cast<uint32_t*>(s_dyn + W * SEG * (WT ? 2 : 1));
  for (int64_t q = persistent ? draw_run(a.ticket, s_tick) : (int64_t)blockIdx.x; q < a.nruns;
       q = persistent ? draw_run(a.ticket, s_tick) : a.nruns) {
    uint32_t gs, tpos, j;
    run_at(a.ro, (uint32_t)q, &gs, &tpos, &j);
    const int t = sload(a.tperm, tpos);
    const int64_t g = slice_at(a.so, gs);
    const int64_t b0 = g * a.C + (int64_t)j * a.K;
    const int64_t b1 = min(b0 + (int64_t)a.K, (g + 1) * (int64_t)a.C);
    const TabMeta m = load_meta(a.meta + t);
    const char* tab = static_cast<const char*>(sload(a.tables, t));
    const int64_t nb = b1 - b0;
    const int64_t per = (nb + W - 1) / W;
    const int64_t bb = b0 + wid * per;
    const int64_t be = min(bb + per, b1);
    const int64_t obase = (int64_t)t * a.B;
    const float* outbase = FUSED ? a.out + m.col_off : a.out + a.B * m.col_off;
    const int64_t ostride = FUSED ? a.sum_dim : m.dim;
    for (int64_t b = bb; b < be; ++b) {
      int64_t lo = a.offsets[obase + b];
      int64_t hi = a.offsets[obase + b + 1];
      bool bad = false;
      if (a.check && !(lo >= 0 && lo <= hi && hi <= nnz)) {
        bad = true;
        lo = hi = 0;
      }
      const int L = (int)(hi - lo);
      float* orow = const_cast<float*>(outbase) + b * ostride;
      if (m.vshift >= 0) {
        GlobalRows rl;
        rl.colp = tab + (lane & ((1 << m.vshift) - 1)) * 16;
        rl.rb = (uint32_t)m.row_bytes;
        float acc[EPV];
#pragma unroll
        for (int e = 0; e < EPV; ++e) acc[e] = 0.f;
        for (int s0 = 0; s0 < L; s0 += SEG) {
          const int n = min(SEG, L - s0);
          stage<WT>(a.indices, a.weights, lo + s0, n, lane, lds_i, lds_w);
          wave_lds_sync();
          bad |= a.check ? gather_p2<E, U, WT, true>(rl, m.vshift, m.rows, lds_i, lds_w, n, lane, acc)
                         : gather_p2<E, U, WT, false>(rl, m.vshift, m.rows, lds_i, lds_w, n, lane, acc);
          wave_lds_sync();
        }
        reduce_store<EPV>(acc, m.vshift, lane, orow, m.dim, sc1, a.mean ? L : 0);
      } else {
        bad |= pool_bag_generic<E, U, WT>(tab, m, a.indices, a.weights, lo, L, lds_i, lds_w, lane, a.check, orow,
                                          sc1, a.mean ? L : 0);
      }
      if (a.check && __any(bad) && lane == 0) atomicMin(&a.status[ST_FIRST_BAD_BAG], (int32_t)(obase + b));
    }
    if (FUSED) {
      if (a.release_mode == 1) wait_stores_complete();
      __syncthreads();
      if (threadIdx.x == 0)
        release_slice(a.counters, a.flags, a.per_table ? g * a.T + t : g, (uint32_t)nb,
                      a.per_table ? (uint32_t)a.C : (uint32_t)a.C * (uint32_t)a.T, a.suppress, a.trace_release,
                      a.release_mode, a.counter_shift);
    }
  }
  if (persistent) leave_runs(a.ticket);
}

// How a launch reads table rows: through one buffer descriptor per table with
// non-temporal or cached loads (the fast path), or by the general path.
enum { ROWS_STREAMED = 0, ROWS_CACHED = 1, ROWS_GENERAL = 2 };

// Fused operator: pooled vectors go straight to the send layout and slices
// are released as they complete.
template <class E, int U, bool WT, int ROWS>
__global__ __launch_bounds__(1024) void fused_pool_kernel(const PoolArgs a) {
  if constexpr (ROWS == ROWS_GENERAL)
    pool_safe<E, U, WT, true>(a);
  else
    pool_fast<E, U, WT, ROWS == ROWS_STREAMED, true>();
}

// Unfused baseline, first kernel: plain per-table EmbeddingBag output.
template <class E, int U, bool WT, int ROWS>
__global__ __launch_bounds__(1024) void unfused_pool_kernel(const PoolArgs a) {
  if constexpr (ROWS == ROWS_GENERAL)
    pool_safe<E, U, WT, false>(a);
  else
    pool_fast<E, U, WT, ROWS == ROWS_STREAMED, false>();
}

typedef void (*pool_fn)(const PoolArgs);

template <class E, int U, bool WT>
pool_fn pick_r(int rows, bool fused) {
  switch (rows) {
    case ROWS_STREAMED:
      return fused ? &fused_pool_kernel<E, U, WT, ROWS_STREAMED> : &unfused_pool_kernel<E, U, WT, ROWS_STREAMED>;
    case ROWS_CACHED:
      return fused ? &fused_pool_kernel<E, U, WT, ROWS_CACHED> : &unfused_pool_kernel<E, U, WT, ROWS_CACHED>;
    default:
      return fused ? &fused_pool_kernel<E, U, WT, ROWS_GENERAL> : &unfused_pool_kernel<E, U, WT, ROWS_GENERAL>;
  }
}

template <class E>
pool_fn pick_u(int u, bool weighted, int rows, bool fused) {
  switch (u) {
    case 4: return weighted ? pick_r<E, 4, true>(rows, fused) : pick_r<E, 4, false>(rows, fused);
    case 16: return weighted ? pick_r<E, 16, true>(rows, fused) : pick_r<E, 16, false>(rows, fused);
    default: return weighted ? pick_r<E, 8, true>(rows, fused) : pick_r<E, 8, false>(rows, fused);
  }
}

pool_fn pick(int dtype, int u, bool weighted, bool fused, bool safe, bool stream_rows) {
  const int rows = safe ? ROWS_GENERAL : stream_rows ? ROWS_STREAMED : ROWS_CACHED;
  switch (dtype) {
    case 1: return pick_u<EF16>(u, weighted, rows, fused);
    case 2: return pick_u<EBF16>(u, weighted, rows, fused);
    default: return pick_u<EF32>(u, weighted, rows, fused);
  }
}

size_t lds_bytes(bool safe, bool weighted, int block, int out_floats) {
  // + 16 bytes: the run-arrival counter and the ticket broadcast slot
  const size_t staging = (size_t)(block / 64) * (safe ? SEG : SLOTW) * (weighted ? 8 : 4);
  return safe ? staging + 16 : staging + (size_t)out_floats * 4 + 16;
}

}  // namespace

hipError_t launch_pool(int dtype, int rows_in_flight, bool weighted, bool fused, bool safe, const PoolArgs& a,
                       int grid, int block, hipStream_t stream) {
  pool_fn f = pick(dtype, rows_in_flight, weighted, fused, safe, a.stream_rows);
  hipLaunchKernelGGL(f, dim3(grid), dim3(block), lds_bytes(safe, weighted, block, a.out_floats), stream, a);
  return hipGetLastError();
}

int pool_max_wgs_per_cu(int dtype, int rows_in_flight, bool weighted, bool fused, bool safe, bool stream_rows,
                        int block, int out_floats) {
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, pick(dtype, rows_in_flight, weighted, fused, safe, stream_rows), block,
                                                   lds_bytes(safe, weighted, block, out_floats)) != hipSuccess)
    return 0;
  return n;
}

}  // namespace ebag
