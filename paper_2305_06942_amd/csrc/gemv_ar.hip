// Fused GEMV + AllReduce (Sec. III-B) for gfx950, and its bulk-synchronous
// baseline; the C ABI is declared in include/gemv_ar.h.
//
// GEMV: a wave computes rows of its tile; for a row, lane l takes the 16-byte
// vectors l, l + 64, ... of the row (coalesced non-temporal loads -- the
// matrix is read once) and the matching vectors of x.  Sixteen loads are in
// flight per lane, spread over RPI rows and UJ = 16 / RPI vectors of each:
// rows of at most 64 (128, 256) vectors take 16 (8, 4) rows at once and keep
// the lane's vectors of x in registers; rows of at most 32 vectors share a
// wave's lanes between two or more rows; longer ones stage the rank's x in the
// workgroup's LDS.  Products are accumulated in fp32 per lane and combined
// with xor shuffles; the shape changes no sum's order.
//
// Where R * P workgroups do not fill the device, each (r, p) is `split` into
// several that share every tile's rows (split_for).
//
// AllReduce (fused), two-phase direct: workgroup (r, p) stores its partial
// tiles for owner q into the reduction slots part[r][rows] with device-scope
// stores and waits for them to complete.  Then either
//  - owner-waits mode (the paper's scheme, cooperative launch): it sets peer
//    flag (q, r, p) to the forward's epoch, and owner workgroup (q, p) polls
//    the flags of (s, p) for every s != q before reducing; or
//  - last-arriver mode (default): it counts itself in on counter (q, p), and
//    the workgroup completing the count reduces.
// The reduction sums part[0..R-1][rows] in rank order with device-scope loads
// and stores the result into every rank's output.
#include <climits>
#include <cstring>
#include <new>
#include <vector>

#include "common.h"
#include "device_guard.h"
#include "gemv_ar.h"
#include "gemv_tiles.h"

namespace ebag {
namespace {

constexpr int kBufferWord3 = 0x00020000;  // raw buffer, 32-bit data format
constexpr int kInFlight = 16;      // 16-byte loads in flight per lane
constexpr int kBf16Rows = -8;      // eight rows at once, one vector of each (bf16)
constexpr int kWholeRows = -4;     // four rows at once, all four vectors of each (fp16)
constexpr int kMaxXBytes = 64 * 1024;

typedef uint32_t u4v __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) const u4v gu4v;

struct GemvArgs {
  const char* A[kMaxRanks];
  const char* x[kMaxRanks];
  float* y[kMaxRanks];
  int64_t K[kMaxRanks];
  float* part;           // [R][M] partial vectors (the owners' reduction slots)
  uint32_t* peer;        // [R owner][R source][P] epoch flags (owner-waits mode)
  uint32_t* cnt;         // [R owner][P] arrival counters (last-arriver mode, self-resetting)
  uint32_t* out_flags;   // [R][P] or nullptr
  int32_t* status;       // [2]: timed out, first missing peer flag
  int64_t M;
  int64_t n_tiles;
  int64_t suppress;
  uint64_t timeout_ticks;
  uint32_t epoch;
  int32_t R;
  int32_t P;
  int32_t TM;
  int32_t comm_aware;
  int32_t split;         // workgroups per (r, p), each taking sub_rows rows of every tile
  int32_t sub_rows;
  int32_t lanes;         // lanes per row: 64, or less where all rows are shorter
  TileOwners tiles;
};

// 16-byte vector of the storage type -> fp32 values.
template <int DT> struct Vec;
template <> struct Vec<0> {  // fp32
  static constexpr int N = 4;
  static __device__ __forceinline__ void widen(const u4v& r, float* f) {
    f[0] = __uint_as_float(r.x); f[1] = __uint_as_float(r.y); f[2] = __uint_as_float(r.z); f[3] = __uint_as_float(r.w);
  }
};
template <> struct Vec<1> {  // fp16
  static constexpr int N = 8;
  static __device__ __forceinline__ void widen(const u4v& r, float* f) {
    const uint32_t u[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      f[2 * e] = (float)__builtin_bit_cast(_Float16, (uint16_t)(u[e] & 0xffffu));
      f[2 * e + 1] = (float)__builtin_bit_cast(_Float16, (uint16_t)(u[e] >> 16));
    }
  }
};
template <> struct Vec<2> {  // bf16
  static constexpr int N = 8;
  static __device__ __forceinline__ void widen(const u4v& r, float* f) {
    const uint32_t u[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      f[2 * e] = __uint_as_float(u[e] << 16);
      f[2 * e + 1] = __uint_as_float(u[e] & 0xffff0000u);
    }
  }
};

template <int DT>
__device__ __forceinline__ float dot16(const u4v& a, const u4v& x) {
  float fa[Vec<DT>::N], fx[Vec<DT>::N];
  Vec<DT>::widen(a, fa);
  Vec<DT>::widen(x, fx);
  float s = 0.f;
#pragma unroll
  for (int e = 0; e < Vec<DT>::N; ++e) s = __builtin_fmaf(fa[e], fx[e], s);
  return s;
}

__device__ __forceinline__ void store_f32(float* p, float v, bool device_scope) {
  if (device_scope)
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else
    *p = v;
}

__device__ __forceinline__ float load_f32_device(const float* p) {
  return __hip_atomic_load(const_cast<float*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// s_waitcnt vmcnt(0): every memory operation of this wave has completed.
__device__ __forceinline__ void wait_all_memory() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// How a launch shapes the GEMV: RPI rows at once, the lane's vectors of x in
// registers (XREG: rows of at most 64 * UJ vectors) or in LDS.
template <int RPI_, bool XREG_, int UJ_ = kInFlight / RPI_, bool TRIM_ = !XREG_ || RPI_ == 4>
struct Shape {
  static constexpr bool TRIM = TRIM_;  // steps of 64 vectors past the row's end are skipped
  static constexpr int RPI = RPI_;
  static constexpr int UJ = UJ_;
  static constexpr bool XREG = XREG_;
};

// The rank's x, as its lanes use it.
template <class S>
struct XVec {
  u4v reg[S::XREG ? S::UJ : 1];
  const u4v* lds;

  __device__ __forceinline__ void load(const char* x, int V, int lanes, u4v* lds_x) {
    lds = lds_x;
    if (S::XREG) {
      const int l = threadIdx.x & (lanes - 1);
#pragma unroll
      for (int u = 0; u < S::UJ; ++u) {
        reg[u] = u4v{0u, 0u, 0u, 0u};
        if (u * 64 + l < V) reg[u] = *(gu4v*)(x + (int64_t)(u * 64 + l) * 16);
      }
      return;
    }
    // eight loads in flight per thread
    for (int v0 = threadIdx.x; v0 < V; v0 += 8 * blockDim.x) {
      u4v t[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int v = v0 + u * blockDim.x;
        t[u] = *(gu4v*)(x + (int64_t)(v < V ? v : v0) * 16);
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (v0 + u * blockDim.x < V) lds_x[v0 + u * blockDim.x] = t[u];
    }
    __syncthreads();
  }
  __device__ __forceinline__ u4v at(int u, int v) const { return S::XREG ? reg[u] : lds[v]; }
};

// Partial product of rank r for rows [lo, hi) of tile `tile`, stored into
// part[r][rows] (device-scope stores when `device_scope`).
template <int DT, class S>
__device__ void partial_tile(const GemvArgs& a, int r, int64_t tile, int lo, int hi, const XVec<S>& x,
                             bool device_scope) {
  constexpr int RPI = S::RPI, UJ = S::UJ;
  // TRIM, where a pass takes four or more of a row: 1 x 35253 x 2320 fp32 63.5 us
  // without, 62.0 us; 2 x 30000 x 3000 bf16 66.0 and 64.5; and with four whole steps,
  // 4 x 65536 x 2048, bf16 172 to 175 and 167 to 172, but fp16 166.5 and 170, so not
  // there.
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int W = blockDim.x >> 6;
  const int64_t row0 = tile * a.TM;
  const int nrows = (int)min((int64_t)hi, a.M - row0) - lo;
  const int per = (int)((unsigned)(nrows > 0 ? nrows + W - 1 : 0) / (unsigned)W);
  const int r0 = lo + wid * per;
  const int r1 = min(r0 + per, lo + nrows);
  const int64_t row_bytes = a.K[r] * (DT == 0 ? 4 : 2);
  const int V = (int)(row_bytes / 16);
  const char* Ar = a.A[r];
  float* out = a.part + (int64_t)r * a.M + row0;
  const int L = S::RPI == kInFlight ? a.lanes : 64;  // lanes per row, G rows per load
  const int G = S::RPI == kInFlight ? 64 / L : 1;
  const int g = lane / L, l = lane & (L - 1);
  for (int base = r0; base < r1; base += 64) {  // results of up to 64 rows per store
    float res = 0.f;
    const int nb = min(64, r1 - base);
    for (int k = 0; k < nb; k += RPI * G) {
      // The step's rows are contiguous: one descriptor over what is left of
      // them, so loads past the last row return zeros.
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<char*>(Ar + (row0 + base + k) * row_bytes), 0, (nb - k) * (int)row_bytes, kBufferWord3);
      float acc[RPI];
#pragma unroll
      for (int j = 0; j < RPI; ++j) acc[j] = 0.f;
      for (int v0 = 0; v0 < V; v0 += 64 * UJ) {
        u4v ra[RPI][UJ];
#pragma unroll
        for (int u = 0; u < UJ; ++u) {
          const int v = v0 + u * 64 + l;
          if (S::TRIM && v0 + u * 64 >= V) continue;  // no lane has one
          const uint32_t off = v < V ? (uint32_t)(v * 16 + g * (int)row_bytes) : 0x80000000u;  // past any row
#pragma unroll
          for (int j = 0; j < RPI; ++j)
            ra[j][u] = __builtin_amdgcn_raw_buffer_load_b128(rs, off + (uint32_t)(j * G * (int)row_bytes), 0, 2);
        }
#pragma unroll
        for (int u = 0; u < UJ; ++u) {
          const int v = v0 + u * 64 + l;
          if (S::XREG ? !S::TRIM || v0 + u * 64 < V : v < V) {
            u4v xv = x.at(u, v);
            // widened here, not kept widened (twice the registers: fp16, 1 x 35253 x
            // 1160, 28.9 us kept, 23.1 us like this)
            if (DT == 2 || (DT == 1 && S::XREG && S::TRIM)) asm volatile("" : "+v"(xv));
#pragma unroll
            for (int j = 0; j < RPI; ++j) acc[j] += dot16<DT>(ra[j][u], xv);
          }
        }
      }
      // Lanes past the row hold zeros, so rows that share a wave leave out the
      // levels that would only add those.
#pragma unroll
      for (int m = 32; m >= 1; m >>= 1) {
        if (S::RPI == kInFlight && m >= L) continue;
#pragma unroll
        for (int j = 0; j < RPI; ++j) acc[j] += __shfl_xor(acc[j], m);
      }
      if (G == 1) {
#pragma unroll
        for (int j = 0; j < RPI; ++j)
          if (lane == k + j) res = acc[j];
      } else {
#pragma unroll
        for (int j = 0; j < RPI; ++j)
          if (k + j * G + g < nb && l == 0) store_f32(out + base + k + j * G + g, acc[j], device_scope);
      }
    }
    if (G == 1 && lane < nb) store_f32(out + base + lane, res, device_scope);
  }
}

// Sum the R partials of owner q's tiles handled by workgroup p (rank order,
// device-scope loads) and store the result into every rank's output.
__device__ void reduce_owned(const GemvArgs& a, int q, int p) {
  for (uint32_t i = first_tile(a.tiles, q, p, a.P); i < a.tiles.own[q + 1]; i += a.P) {
    const int64_t row0 = (int64_t)i * a.TM;
    const int nrows = (int)min((int64_t)a.TM, a.M - row0);
    for (int k = threadIdx.x; k < nrows; k += blockDim.x) {
      // every rank's partial in flight before the first is added
      float part[kMaxRanks];
#pragma unroll
      for (int s = 0; s < kMaxRanks; ++s)
        if (s < a.R) part[s] = load_f32_device(a.part + (int64_t)s * a.M + row0 + k);
      float sum = 0.f;
#pragma unroll
      for (int s = 0; s < kMaxRanks; ++s)
        if (s < a.R) sum += part[s];
      for (int r = 0; r < a.R; ++r) store_f32(a.y[r] + row0 + k, sum, true);
    }
  }
}

// Fused kernel, last-arriver reduction (default): workgroup (r, p) computes
// its partial tiles owner by owner; after each owner's tiles are stored it
// counts itself in on that owner's counter (q, p), and the workgroup that
// completes the count -- the last of the R ranks' (and their splits') to
// deliver -- reduces and broadcasts the owner's tiles, then re-arms the
// counter.  Nobody waits, so the grid needs no co-residency and launches
// normally.
template <int DT, class S>
__global__ __launch_bounds__(1024) void gemv_ar_last_arriver_kernel(const GemvArgs a) {
  extern __shared__ u4v lds_x[];
  __shared__ uint32_t s_old;
  const int split = a.split;
  const int wg = (int)(blockIdx.x / (unsigned)split), part = (int)blockIdx.x - wg * split;
  const int r = (int)((unsigned)wg / (unsigned)a.P);
  const int p = wg - r * a.P;
  const int lo = part * a.sub_rows, hi = min(lo + a.sub_rows, a.TM);
  XVec<S> x;
  x.load(a.x[r], (int)(a.K[r] * (DT == 0 ? 4 : 2) / 16), a.lanes, lds_x);
  for (int qi = 0; qi < a.R; ++qi) {
    int q = a.comm_aware ? r + 1 + qi : qi;
    if (q >= a.R) q -= a.R;
    const uint32_t i0 = first_tile(a.tiles, q, p, a.P), t1 = a.tiles.own[q + 1];
    if (i0 >= t1) {
      // No tile of owner q for workgroup p (on every rank alike): the owner's
      // own workgroup advances the output flag, which has nothing to cover.
      if (q == r && a.out_flags && threadIdx.x == 0 && part == 0)
        __hip_atomic_fetch_add(&a.out_flags[(int64_t)q * a.P + p], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      continue;
    }
    for (uint32_t i = i0; i < t1; i += a.P) partial_tile<DT, S>(a, r, i, lo, hi, x, true);
    // every wave's partial stores complete (device scope) before counting in
    wait_all_memory();
    __syncthreads();
    uint32_t* c = &a.cnt[(int64_t)q * a.P + p];
    if (threadIdx.x == 0) s_old = __hip_atomic_fetch_add(c, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (s_old == (uint32_t)(a.R * split) - 1) {
      reduce_owned(a, q, p);
      wait_all_memory();
      __syncthreads();
      if (threadIdx.x == 0) {
        __hip_atomic_store(c, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (a.out_flags)
          __hip_atomic_fetch_add(&a.out_flags[(int64_t)q * a.P + p], 1u, __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    __syncthreads();  // s_old is rewritten for the next owner
  }
}

template <int DT, class S>
__global__ __launch_bounds__(1024) void gemv_ar_fused_kernel(const GemvArgs a) {
  extern __shared__ u4v lds_x[];
  __shared__ int s_bad;
  const int r = (int)(blockIdx.x / (unsigned)a.P);
  const int p = (int)blockIdx.x - r * a.P;
  XVec<S> x;
  x.load(a.x[r], (int)(a.K[r] * (DT == 0 ? 4 : 2) / 16), a.lanes, lds_x);
  if (threadIdx.x == 0) s_bad = 0;
  __syncthreads();
  // Phase 1: partial tiles, other owners first (comm-aware) or in owner order.
  for (int qi = 0; qi < a.R; ++qi) {
    int q = a.comm_aware ? r + 1 + qi : qi;
    if (q >= a.R) q -= a.R;
    const uint32_t t1 = a.tiles.own[q + 1];
    for (uint32_t i = first_tile(a.tiles, q, p, a.P); i < t1; i += a.P) partial_tile<DT, S>(a, r, i, 0, a.TM, x, true);
    if (q != r) {
      // every wave's partial stores done (device scope) before the flag
      wait_all_memory();
      __syncthreads();
      const int64_t f = ((int64_t)q * a.R + r) * a.P + p;
      if (threadIdx.x == 0 && f != a.suppress)
        __hip_atomic_store(&a.peer[f], a.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  wait_all_memory();
  __syncthreads();
  // Phase 2: as owner, wait for the partials of workgroup p of every rank.
  if (threadIdx.x == 0) {
    const uint64_t t0 = wall_clock64();
    for (int s = 0; s < a.R && !s_bad; ++s) {
      if (s == r) continue;
      const int64_t f = ((int64_t)r * a.R + s) * a.P + p;
      while (__hip_atomic_load(&a.peer[f], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != a.epoch) {
        if (wall_clock64() - t0 > a.timeout_ticks) {
          __hip_atomic_store(&a.status[0], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          atomicMin(&a.status[1], (int32_t)f);
          s_bad = 1;
          break;
        }
        __builtin_amdgcn_s_sleep(2);
      }
    }
  }
  __syncthreads();
  if (s_bad) return;
  // Reduce the owned tiles in rank order and store them to every rank.
  reduce_owned(a, r, p);
  if (a.out_flags) {
    wait_all_memory();
    __syncthreads();
    if (threadIdx.x == 0)
      __hip_atomic_fetch_add(&a.out_flags[(int64_t)r * a.P + p], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Baseline, first kernel: `split` workgroups per (rank, tile).
template <int DT, class S>
__global__ __launch_bounds__(1024) void gemv_partial_kernel(const GemvArgs a) {
  extern __shared__ u4v lds_x[];
  const int wg = (int)(blockIdx.x / (unsigned)a.split), part = (int)blockIdx.x - wg * a.split;
  const int r = (int)((unsigned)wg / (unsigned)a.n_tiles);
  const int tile = wg - r * (int)a.n_tiles;
  const int lo = part * a.sub_rows, hi = min(lo + a.sub_rows, a.TM);
  XVec<S> x;
  x.load(a.x[r], (int)(a.K[r] * (DT == 0 ? 4 : 2) / 16), a.lanes, lds_x);
  partial_tile<DT, S>(a, r, tile, lo, hi, x, false);
}

// Baseline, second kernel: the AllReduce after the kernel boundary -- every
// output row is the rank-order sum of the partials, stored to every rank.
__global__ __launch_bounds__(256) void allreduce_kernel(const GemvArgs a) {
  const int64_t row = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (row >= a.M) return;
  float sum = 0.f;
  for (int s = 0; s < a.R; ++s) sum += a.part[(int64_t)s * a.M + row];
  for (int q = 0; q < a.R; ++q) a.y[q][row] = sum;
}

__global__ __launch_bounds__(256) void bump_flags_kernel(uint32_t* flags, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) __hip_atomic_fetch_add(&flags[i], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

typedef void (*gemv_fn)(const GemvArgs);

enum { GEMV_LAST_ARRIVER = 0, GEMV_OWNER_WAITS = 1, GEMV_PARTIAL = 2 };

template <int DT, class S>
gemv_fn pick_kernel(int which) {
  return which == GEMV_LAST_ARRIVER ? gemv_ar_last_arriver_kernel<DT, S>
         : which == GEMV_OWNER_WAITS ? gemv_ar_fused_kernel<DT, S> : gemv_partial_kernel<DT, S>;
}

template <int DT>
gemv_fn pick_shape(int which, int rpi, bool xreg) {
  if (xreg) {
    if constexpr (DT == 1)
      if (rpi == kWholeRows) return pick_kernel<DT, Shape<4, true, 4, false>>(which);
    if constexpr (DT == 2)
      if (rpi == kBf16Rows) return pick_kernel<DT, Shape<8, true, 1>>(which);
    switch (rpi) {
      case 16: return pick_kernel<DT, Shape<16, true>>(which);
      case 8: return pick_kernel<DT, Shape<8, true>>(which);
      default: return pick_kernel<DT, Shape<4, true>>(which);
    }
  }
  switch (rpi) {
    case 1: return pick_kernel<DT, Shape<1, false>>(which);
    case 2: return pick_kernel<DT, Shape<2, false>>(which);
    default: return pick_kernel<DT, Shape<4, false>>(which);
  }
}

gemv_fn pick(int dt, int which, int rpi, bool xreg) {
  return dt == 0 ? pick_shape<0>(which, rpi, xreg)
                 : dt == 1 ? pick_shape<1>(which, rpi, xreg) : pick_shape<2>(which, rpi, xreg);
}

}  // namespace
}  // namespace ebag

using namespace ebag;

struct gemv_ar_plan {
  int device = 0;
  int32_t R = 0;
  int64_t M = 0;
  int dtype = 0;
  int elt = 4;
  int64_t K[kMaxRanks] = {};
  int64_t max_x_bytes = 0;
  int num_cus = 0;
  double ticks_per_us = 100.0;
  gemv_ar_opts_t opts{};
  int64_t n_tiles = 0;
  int32_t P = 0;
  int32_t block = 0;
  int32_t resident = 0;  // workgroups the device holds at once for the fused kernel
  int32_t split = 1;      // workgroups per (r, p) of the last-arriver kernel
  int32_t sub_rows = 0;
  int32_t lanes = 64;
  int rpi = 4;
  bool xreg = false;
  uint32_t epoch = 0;
  // The last forward's completion, for refusing a forward on another stream
  // while it still runs (the reduction slots and counters are shared).
  hipEvent_t fwd_done = nullptr;
  hipStream_t fwd_stream = nullptr;
  bool fwd_pending = false;
  size_t lds_bytes() const { return xreg ? 0 : (size_t)max_x_bytes; }
  float* d_part = nullptr;
  uint32_t* d_peer = nullptr;
  uint32_t* d_cnt = nullptr;
  int32_t* d_status = nullptr;
};

namespace {

const int32_t kGemvStatusInit[2] = {0, INT_MAX};

void free_gemv(gemv_ar_plan* h) {
  if (!h) return;
  if (h->fwd_done) (void)hipEventDestroy(h->fwd_done);
  (void)hipFree(h->d_part);
  (void)hipFree(h->d_peer);
  (void)hipFree(h->d_cnt);
  (void)hipFree(h->d_status);
  delete h;
}

int hipf(hipError_t e, const char* what) { return fail(EBAG_EHIP, "%s: %s", what, hipGetErrorString(e)); }

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

bool capturing(hipStream_t stream) {
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  return hipStreamIsCapturing(stream, &cs) == hipSuccess && cs != hipStreamCaptureStatusNone;
}

// One forward in flight per plan: a forward on another stream than the last
// one, while the last one has not completed, would share its reduction slots
// and arrival counters.
int check_busy(gemv_ar_plan* h, hipStream_t stream) {
  if (!h->fwd_pending || stream == h->fwd_stream || capturing(stream)) return EBAG_OK;
  const hipError_t e = hipEventQuery(h->fwd_done);
  if (e == hipErrorNotReady)
    return fail(EBAG_EBUSY, "a forward of this plan is still running on another stream (the reduction slots and "
                            "counters are shared): order the forwards on one stream or wait for it");
  if (e != hipSuccess) return hipf(e, "query the last forward");
  h->fwd_pending = false;
  return EBAG_OK;
}

// Remember the forward just enqueued on `stream` (not under graph capture).
int note_forward(gemv_ar_plan* h, hipStream_t stream) {
  if (capturing(stream)) {
    h->fwd_pending = false;
    return EBAG_OK;
  }
  const hipError_t e = hipEventRecord(h->fwd_done, stream);
  if (e != hipSuccess) return hipf(e, "record the forward's completion");
  h->fwd_stream = stream;
  h->fwd_pending = true;
  return EBAG_OK;
}

// Rows at once, and where x lies, by the longest rank's row of V vectors: the
// rows that fill the loads in flight, so that a wave of short rows does not run
// with a few lanes or a few loads of the sixteen.  Measured, before (4 rows x 4
// vectors, x in LDS) and now: 4 ranks x 30000 x 96 bf16 32.8 us and 20.7 us; 8
// x 8192 x 1024 fp16 33.5 and 28.9; 4 x 65536 x 2048 fp16 (4 rows x 4 vectors
// still, x in registers) 165.9 and 164.8, 6.5 TB/s, the streaming read ceiling.
// bf16 rows of 33 to 64 vectors go eight at once, one vector a lane of each: sixteen
// take 117 registers for them and their sums (1 x 60000 x 512: 21.1 us, 16.8 us like
// this, 20.0 us four rows at once with x in LDS).
void launch_shape(gemv_ar_plan* h) {
  const int64_t V = h->max_x_bytes / 16;
  h->xreg = V <= 256;
  h->rpi = V <= 64 ? 16 : V <= 128 ? 8 : 4;
  if (h->dtype == EBAG_BF16 && V > 32 && V <= 64) h->rpi = kBf16Rows;
  if (h->dtype == EBAG_F16 && V == 256) h->rpi = kWholeRows;
  h->lanes = 64;
  while (h->lanes > 1 && V <= h->lanes / 2) h->lanes /= 2;
  // Long rows, fewer than four of them for each of 2048 waves: fewer rows at
  // once, more of each.
  if (!h->xreg)
    while (h->rpi > 1 && (int64_t)h->R * h->M < (int64_t)h->rpi * 2048) h->rpi /= 2;
}

int fill_args(gemv_ar_plan* h, const void* const* A, const void* const* x, float* const* y, uint32_t* out_flags,
              GemvArgs* a) {
  if (!h) return fail(EBAG_EINVAL, "null plan");
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev != h->device)
    return fail(EBAG_EINVAL, "the plan belongs to device %d, but device %d is current", h->device, dev);
  if (!A || !x || !y) return fail(EBAG_EINVAL, "null A, x or y pointer array");
  std::memset(a, 0, sizeof *a);
  for (int r = 0; r < h->R; ++r) {
    if (!A[r] || !x[r] || !y[r]) return fail(EBAG_EINVAL, "null A, x or y for rank %d", r);
    if (!aligned16(A[r]) || !aligned16(x[r])) return fail(EBAG_EINVAL, "A or x of rank %d not 16-byte aligned", r);
    a->A[r] = static_cast<const char*>(A[r]);
    a->x[r] = static_cast<const char*>(x[r]);
    a->y[r] = y[r];
    a->K[r] = h->K[r];
  }
  a->part = h->d_part;
  a->peer = h->d_peer;
  a->cnt = h->d_cnt;
  a->out_flags = out_flags;
  a->status = h->d_status;
  a->M = h->M;
  a->n_tiles = h->n_tiles;
  a->suppress = h->opts.debug_suppress_flag;
  a->timeout_ticks = (uint64_t)((double)h->opts.timeout_us * h->ticks_per_us);
  a->R = h->R;
  a->P = h->P;
  a->TM = h->opts.tile_rows;
  a->comm_aware = h->opts.comm_aware;
  a->split = 1;
  a->sub_rows = a->TM;
  a->lanes = h->lanes;
  make_owners(h->n_tiles, h->R, h->P, &a->tiles);
  return EBAG_OK;
}

}  // namespace

extern "C" {

int gemv_ar_default_opts(gemv_ar_opts_t* o) {
  if (!o) return fail(EBAG_EINVAL, "null opts");
  std::memset(o, 0, sizeof *o);
  o->tile_rows = 0;
  o->wgs_per_rank = 0;
  o->waves_per_wg = 2;
  o->comm_aware = 1;
  o->debug_suppress_flag = -1;
  o->reduce_mode = 0;
  o->timeout_us = 5000000;
  return EBAG_OK;
}

int gemv_ar_create(gemv_ar_t* out, int32_t R, int64_t M, const int64_t* K, int32_t dtype,
                   const gemv_ar_opts_t* opts) {
  if (!out) return fail(EBAG_EINVAL, "null output handle");
  *out = nullptr;
  if (R < 1 || R > kMaxRanks) return fail(EBAG_EINVAL, "R=%d outside [1, %d]", R, kMaxRanks);
  if (M < 1 || M > INT_MAX) return fail(EBAG_EINVAL, "M=%lld outside [1, 2^31)", (long long)M);
  if (!K) return fail(EBAG_EINVAL, "null K array");
  if (dtype != EBAG_F32 && dtype != EBAG_F16 && dtype != EBAG_BF16) return fail(EBAG_EINVAL, "bad dtype %d", (int)dtype);
  gemv_ar_opts_t o;
  if (opts) o = *opts; else gemv_ar_default_opts(&o);
  if (o.tile_rows < 0 || o.tile_rows > 4096) return fail(EBAG_EINVAL, "tile_rows must be 0 (auto) or in [1, 4096]");
  if (o.tile_rows == 0) {
    // 128-row tiles, halved (down to 64) until the R ranks hold at least
    // 2048 tiles: with about 1024 workgroups (below), each then computes two
    // or more tiles, and the reduction that follows its first tile overlaps
    // the GEMV of its next one instead of all waiting at the kernel's end.
    o.tile_rows = 128;
    while (o.tile_rows > 64 && (int64_t)R * ((M + o.tile_rows - 1) / o.tile_rows) < 2048) o.tile_rows /= 2;
  }
  if (o.waves_per_wg < 1 || o.waves_per_wg > 16) return fail(EBAG_EINVAL, "waves_per_wg must be in [1, 16]");
  if (o.wgs_per_rank < 0) return fail(EBAG_EINVAL, "wgs_per_rank must be >= 0");
  if (o.comm_aware != 0 && o.comm_aware != 1) return fail(EBAG_EINVAL, "comm_aware must be 0 or 1");
  if (o.reduce_mode != 0 && o.reduce_mode != 1) return fail(EBAG_EINVAL, "reduce_mode must be 0 or 1");
  if (o.timeout_us < 1) return fail(EBAG_EINVAL, "timeout_us must be >= 1");
  const int elt = dtype == EBAG_F32 ? 4 : 2;
  int64_t max_x = 0;
  for (int r = 0; r < R; ++r) {
    if (K[r] < 1) return fail(EBAG_EINVAL, "K[%d]=%lld must be positive", r, (long long)K[r]);
    if ((K[r] * elt) % 16) return fail(EBAG_EINVAL, "K[%d] * element size is not a multiple of 16 bytes", r);
    if (K[r] * elt > kMaxXBytes)
      return fail(EBAG_EUNSUPPORTED, "K[%d] * element size above %d bytes (x is staged in LDS)", r, kMaxXBytes);
    if (K[r] * elt > max_x) max_x = K[r] * elt;
  }
  gemv_ar_plan* h = new (std::nothrow) gemv_ar_plan();
  if (!h) return fail(EBAG_ENOMEM, "host allocation failed");
  h->R = R;
  h->M = M;
  h->dtype = (int)dtype;
  h->elt = elt;
  for (int r = 0; r < R; ++r) h->K[r] = K[r];
  h->max_x_bytes = max_x;
  h->opts = o;
  h->n_tiles = (M + o.tile_rows - 1) / o.tile_rows;
  h->block = 64 * o.waves_per_wg;
  hipError_t e = hipGetDevice(&h->device);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&h->num_cus, hipDeviceAttributeMultiprocessorCount, h->device);
  int khz = 0;
  if (e == hipSuccess && hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, h->device) == hipSuccess &&
      khz > 0)
    h->ticks_per_us = khz / 1000.0;
  const bool owner_mode = o.reduce_mode == 1;
  launch_shape(h);
  int per_cu = 0;
  if (e == hipSuccess)
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &per_cu, pick(h->dtype, owner_mode ? GEMV_OWNER_WAITS : GEMV_LAST_ARRIVER, h->rpi, h->xreg), h->block,
        h->lds_bytes());
  if (e != hipSuccess) {
    free_gemv(h);
    return hipf(e, "query device");
  }
  h->resident = per_cu * h->num_cus;
  // Owner-waits mode needs every workgroup resident (cooperative launch);
  // the last-arriver mode does not and defaults to about 1024 workgroups in
  // all (at most one tile each): one resident wave on 256 CUs.
  int64_t P = o.wgs_per_rank > 0 ? o.wgs_per_rank : owner_mode ? h->resident / R : (1024 + R - 1) / R;
  if (P > h->n_tiles) P = h->n_tiles;
  if (P * R > INT_MAX) P = INT_MAX / R;
  if (P < 1 || (owner_mode && P * R > h->resident)) {
    const int rc = fail(EBAG_EUNSUPPORTED, "%lld workgroups per rank x %d ranks cannot all be resident (%d fit)",
                        (long long)P, R, h->resident);
    free_gemv(h);
    return rc;
  }
  h->P = (int32_t)P;
  h->split = split_for((int64_t)R * P, o.waves_per_wg, o.tile_rows, max_x, &h->sub_rows);
#define GEMV_TRY(call, what)        \
  do {                              \
    hipError_t e_ = (call);         \
    if (e_ != hipSuccess) {         \
      const int r_ = hipf(e_, what); \
      free_gemv(h);                 \
      return r_;                    \
    }                               \
  } while (0)
  GEMV_TRY(hipMalloc((void**)&h->d_part, sizeof(float) * (size_t)R * (size_t)M), "alloc reduction slots");
  GEMV_TRY(hipMalloc((void**)&h->d_peer, sizeof(uint32_t) * (size_t)R * R * P), "alloc peer flags");
  GEMV_TRY(hipMemset(h->d_peer, 0, sizeof(uint32_t) * (size_t)R * R * P), "zero peer flags");
  GEMV_TRY(hipMalloc((void**)&h->d_cnt, sizeof(uint32_t) * (size_t)R * P), "alloc arrival counters");
  GEMV_TRY(hipMemset(h->d_cnt, 0, sizeof(uint32_t) * (size_t)R * P), "zero arrival counters");
  GEMV_TRY(hipMalloc((void**)&h->d_status, sizeof(kGemvStatusInit)), "alloc status");
  GEMV_TRY(hipMemcpy(h->d_status, kGemvStatusInit, sizeof(kGemvStatusInit), hipMemcpyHostToDevice), "init status");
  GEMV_TRY(hipEventCreateWithFlags(&h->fwd_done, hipEventDisableTiming), "create forward event");
#undef GEMV_TRY
  *out = h;
  clear_error();
  return EBAG_OK;
}

int gemv_ar_forward(gemv_ar_t h, const void* const* A, const void* const* x, float* const* y, uint32_t* out_flags,
                    hipStream_t stream) {
  GemvArgs a;
  int rc = fill_args(h, A, x, y, out_flags, &a);
  if (rc) return rc;
  // The peer flags carry this call's epoch, fixed at capture: a graph replay
  // would see the previous replay's flags and not wait.
  if (h->opts.reduce_mode == 1 && capturing(stream))
    return fail(EBAG_EUNSUPPORTED, "reduce_mode 1 cannot be captured into a graph (use reduce_mode 0)");
  rc = check_busy(h, stream);
  if (rc) return rc;
  // A fresh epoch per forward: peer flags of earlier forwards never match.
  // Epoch 0 is the value the flags start from, so it is skipped.
  if (++h->epoch == 0) ++h->epoch;
  a.epoch = h->epoch;
  if (h->opts.reduce_mode == 0) {
    a.split = h->split;
    a.sub_rows = h->sub_rows;
    hipLaunchKernelGGL(pick(h->dtype, GEMV_LAST_ARRIVER, h->rpi, h->xreg), dim3((unsigned)(h->R * h->P * h->split)),
                       dim3(h->block), h->lds_bytes(), stream, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hipf(e, "launch the fused GEMV + AllReduce kernel");
    return note_forward(h, stream);
  }
  void* args[] = {&a};
  const hipError_t e = hipLaunchCooperativeKernel(
      reinterpret_cast<const void*>(pick(h->dtype, GEMV_OWNER_WAITS, h->rpi, h->xreg)), dim3((unsigned)(h->R * h->P)),
      dim3(h->block), args, (unsigned)h->lds_bytes(), stream);
  if (e != hipSuccess) return hipf(e, "cooperative launch of the fused GEMV + AllReduce kernel");
  return note_forward(h, stream);
}

int gemv_ar_unfused_forward(gemv_ar_t h, const void* const* A, const void* const* x, float* const* y,
                            uint32_t* out_flags, hipStream_t stream) {
  GemvArgs a;
  int rc = fill_args(h, A, x, y, out_flags, &a);
  if (rc) return rc;
  rc = check_busy(h, stream);
  if (rc) return rc;
  const int64_t g1 = (int64_t)h->R * h->n_tiles;
  if (g1 > INT_MAX) return fail(EBAG_EINVAL, "too many tiles for one launch");
  a.split = split_for(g1, h->opts.waves_per_wg, a.TM, h->max_x_bytes, &a.sub_rows);
  hipLaunchKernelGGL(pick(h->dtype, GEMV_PARTIAL, h->rpi, h->xreg), dim3((unsigned)(g1 * a.split)), dim3(h->block),
                     h->lds_bytes(), stream, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hipf(e, "launch GEMV kernel");
  hipLaunchKernelGGL(allreduce_kernel, dim3((unsigned)((h->M + 255) / 256)), dim3(256), 0, stream, a);
  e = hipGetLastError();
  if (e != hipSuccess) return hipf(e, "launch AllReduce kernel");
  if (out_flags) {
    const int64_t n = (int64_t)h->R * h->P;
    hipLaunchKernelGGL(bump_flags_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, out_flags, n);
    e = hipGetLastError();
    if (e != hipSuccess) return hipf(e, "launch flag kernel");
  }
  return note_forward(h, stream);
}

int gemv_ar_status(gemv_ar_t h, int32_t out[2]) {
  if (!h || !out) return fail(EBAG_EINVAL, "null plan or output");
  const DeviceGuard dg(h->device);
  if (dg.error() != hipSuccess) return hipf(dg.error(), "make the plan's device current");
  hipError_t e = hipDeviceSynchronize();
  if (e != hipSuccess) return hipf(e, "synchronize");
  int32_t s[2];
  e = hipMemcpy(s, h->d_status, sizeof s, hipMemcpyDeviceToHost);
  if (e != hipSuccess) return hipf(e, "read status");
  out[0] = s[0];
  out[1] = s[1] == INT_MAX ? -1 : s[1];
  return s[0] ? EBAG_ETIMEOUT : EBAG_OK;
}

int gemv_ar_reset(gemv_ar_t h) {
  if (!h) return fail(EBAG_EINVAL, "null plan");
  const DeviceGuard dg(h->device);
  if (dg.error() != hipSuccess) return hipf(dg.error(), "make the plan's device current");
  hipError_t e = hipDeviceSynchronize();
  if (e == hipSuccess) e = hipMemcpy(h->d_status, kGemvStatusInit, sizeof(kGemvStatusInit), hipMemcpyHostToDevice);
  if (e != hipSuccess) return hipf(e, "reset status");
  return EBAG_OK;
}

int gemv_ar_launch_info(gemv_ar_t h, int32_t out[5]) {
  if (!h || !out) return fail(EBAG_EINVAL, "null plan or output");
  out[0] = h->P;
  out[1] = h->block;
  out[2] = (int32_t)(h->n_tiles > INT_MAX ? INT_MAX : h->n_tiles);
  out[3] = h->resident;
  out[4] = h->opts.tile_rows;
  return EBAG_OK;
}

void gemv_ar_destroy(gemv_ar_t h) { free_gemv(h); }

}  // extern "C"
