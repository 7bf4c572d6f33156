// Embedding backward fused with the arrival of the gradient All-to-All, and
// the one-GPU stand-in for that arrival (the deliver kernel).
//
// The table owner receives the gradient of every pooled vector in the
// destination-partitioned layout grad[R][S][sum D] (= [B][sum D]), slice by
// slice.  The gradient of lookup k of bag (t, b) is w_k * grad[b][off_t ..
// off_t + D_t) (sum mode; w_k = 1 without weights) or grad[b][...] / L (mean
// mode).  Output: per table, in lookup order, nnz_t rows of D_t fp32 values;
// table blocks follow each other in table order.
//
// Runs are the forward's: up to K consecutive samples of one table inside
// one slice, numbered slice-major.  With flags, a workgroup waits for its
// slice's flag before touching the gradient, so slices are expanded as they
// arrive.  The workgroup scales its K gradient rows once into LDS (the
// mean's division happens there, once per element); the run's output rows
// are contiguous (consecutive bags' lookups follow each other), so the whole
// workgroup writes them as one block with 16-byte non-temporal stores,
// balanced however the bag lengths vary.
#include "backward.h"

namespace ebag {
namespace {

typedef uint32_t u4v __attribute__((ext_vector_type(4)));
typedef float f4v __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void wait_all_memory() { __builtin_amdgcn_s_waitcnt(0x0F70); }

template <class T>
__device__ __forceinline__ T sld(const T* p, int64_t i) {
  return ((const __attribute__((address_space(4))) T*)p)[i];
}

// First float of every table's output block: base[t] = sum over t' < t of
// nnz_t' * D_t', base[T] the total.  One workgroup of 256 threads: the
// tables' sizes are loaded 256 at a time (independent loads, one memory
// latency per 256 tables) and prefix-summed in LDS.
__global__ __launch_bounds__(256) void value_base_kernel(const int64_t* offsets, const TabMeta* meta, int32_t T,
                                                         int64_t B, int64_t* base) {
  __shared__ int64_t s_scan[256];
  const int tid = threadIdx.x;
  int64_t carry = 0;
  for (int32_t c0 = 0; c0 < T; c0 += 256) {
    const int32_t t = c0 + tid;
    const int64_t v = t < T ? (offsets[(int64_t)(t + 1) * B] - offsets[(int64_t)t * B]) * meta[t].dim : 0;
    s_scan[tid] = v;
    __syncthreads();
    for (int d = 1; d < 256; d <<= 1) {  // inclusive Hillis-Steele scan
      const int64_t add = tid >= d ? s_scan[tid - d] : 0;
      __syncthreads();
      s_scan[tid] += add;
      __syncthreads();
    }
    if (t < T) base[t] = carry + s_scan[tid] - v;
    carry += s_scan[255];
    __syncthreads();
  }
  if (tid == 0) base[T] = carry;
}

// Streams a run's output block, n = rows x V float4s, to out: element e is
// vector e mod V of lookup e / V, the row of the lookup's bag times its weight.
// Each thread walks elements tid, tid + step, ... keeping its (lookup, vector)
// position incrementally (no division on the way) and the end of its current
// bag in a register (LDS is read only when a bag boundary is crossed).
//
// The weights lie in LDS (LDSW) wherever the run's fit its slots.  Loads and
// stores are counted by one counter on this GPU, in order, so a weight loaded
// from memory on the way cannot be waited for without the stores before it.
template <class I, bool WT, bool LDSW>
struct BlockStream {
  const f4v* rows_lds;
  const int64_t* s_off;
  const float* w;
  f4v* out;
  I n, k, bag_end;
  int V, step, dk, dc, c, bag;

  // UB elements from e0 on: their LDS rows and weights are all requested before
  // the first store.
  template <int UB>
  __device__ __forceinline__ void pass(I e0) {
    f4v x[UB];
    float wv[UB];
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      const bool in = e0 + (I)u * step < n;
      // k < rows = s_off[nb] for every element in range, so the walk stops
      // at a bag below nb.
      if (in)
        while (k >= bag_end) bag_end = (I)s_off[++bag + 1];
      x[u] = rows_lds[bag * V + c];
      wv[u] = WT ? (LDSW ? w[in ? k : 0] : in ? w[k] : 1.f) : 1.f;
      k += dk;
      c += dc;
      if (c >= V) {
        c -= V;
        ++k;
      }
    }
#pragma unroll
    for (int u = 0; u < UB; ++u)
      if (e0 + (I)u * step < n) __builtin_nontemporal_store(WT ? wv[u] * x[u] : x[u], out + e0 + (I)u * step);
  }

  // Eight elements a thread at a time while more than four are left, then as
  // few as hold the rest.  Measured, 4 at a time always and like this: 48 tables
  // of 32 to 256 floats, weighted bags of 1 to 100 (9.8 GB) 1768 us and 1706 us;
  // 32 x 128 floats, bags of 40 (10.9 GB) 1918 and 1844; bags of 32 at 4 a run,
  // four elements a thread, 340 and 345 (level within its runs overlapped with
  // the delivery).  Eight-element passes over a rest of three or four made the
  // weighted ones 15% slower.
  __device__ __forceinline__ void run() {
    dk = (int)((unsigned)step / (unsigned)V);
    dc = step - dk * V;
    k = (I)((unsigned)threadIdx.x / (unsigned)V);
    c = (int)threadIdx.x - (int)k * V;
    bag = 0;
    bag_end = (I)s_off[1];
    for (I e = 0; e < n;) {
      const I left = n - e;
      if (left > (I)4 * step) {
        pass<8>(e + (I)threadIdx.x);
        e += (I)8 * step;
      } else {
        if (left > (I)2 * step)
          pass<4>(e + (I)threadIdx.x);
        else if (left > step)
          pass<2>(e + (I)threadIdx.x);
        else
          pass<1>(e + (I)threadIdx.x);
        break;
      }
    }
  }
};

template <bool WT>
__global__ __launch_bounds__(1024) void backward_kernel(const BackwardArgs a) {
  // LDS: the run's K scaled gradient rows [K][dim], its K + 1 bag offsets
  // relative to the run's first lookup, its weights.
  extern __shared__ f4v s_lds[];
  __shared__ int s_bad;
  const int tid = threadIdx.x;
  uint32_t gs, tpos, j;
  run_at(a.ro, blockIdx.x, &gs, &tpos, &j);
  const int t = sld(a.tperm, tpos);
  const int64_t g = slice_at(a.so, gs);
  if (a.flags) {
    if (tid == 0) {
      const int64_t f = a.per_table ? g * a.T + t : g;
      const uint64_t t0 = wall_clock64();
      int bad = 0;
      while ((int32_t)(__hip_atomic_load(&a.flags[f], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - a.epoch) < 0) {
        if (wall_clock64() - t0 > a.timeout_ticks) {
          __hip_atomic_store(&a.status[ST_TIMED_OUT], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          atomicMin(&a.status[ST_FIRST_MISSING], (int32_t)f);
          bad = 1;
          break;
        }
        __builtin_amdgcn_s_sleep(4);
      }
      s_bad = bad;
    }
    __syncthreads();
    if (s_bad) return;
  }
  const int dim = sld(&a.meta[t].dim, 0);
  const int col_off = sld(&a.meta[t].col_off, 0);
  const int V = dim >> 2;  // float4 per row
  const int64_t b0 = g * a.C + (int64_t)j * a.K;
  const int nb = min(a.K, a.C - (int)j * a.K);
  const int64_t obase = (int64_t)t * a.B + b0;
  const int64_t lo0 = sld(a.offsets, obase);
  const int64_t rows = sld(a.offsets, obase + nb) - lo0;
  const int64_t table_lo = sld(a.offsets, (int64_t)t * a.B);
  const int64_t base = sld(a.value_base, t);
  int64_t* s_off = reinterpret_cast<int64_t*>(s_lds + (int64_t)a.K * (a.max_dim >> 2));
  float* s_w = reinterpret_cast<float*>(s_off + a.K + 1);
  const bool lds_w = WT && rows <= a.w_slots;
  // A run of a few lookups takes no more waves than its output, its gradient
  // rows and its offsets need; the others leave before the barrier, and their
  // slots take the next workgroup's (26 tables x 16384 bags of 0 to 3 lookups of
  // 128 floats: 522 us before, 486 us without this, 413 us with it).
  const int64_t n = rows * V;
  int step = blockDim.x;
  {
    const int64_t most = max(max(n, (int64_t)nb * V), (int64_t)nb + 1);
    if (most < step) step = ((int)most + 63) & ~63;
    if (tid >= step) return;
  }
  if (tid <= nb) s_off[tid] = a.offsets[obase + tid] - lo0;
  if (lds_w)
    for (int i = tid; i < (int)rows; i += step) s_w[i] = a.weights[lo0 + i];
  // the run's gradient rows, scaled once (device-scope loads: with flags the
  // rows were stored by a kernel that may still be running)
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(a.grad + b0 * a.sum_dim + col_off), 0, ((nb - 1) * a.sum_dim + dim) * 4, 0x00020000);
  for (int e = tid; e < nb * V; e += step) {
    const int k = (int)((unsigned)e / (unsigned)V);
    const int off = (k * a.sum_dim + (e - k * V) * 4) * 4;
    const u4v r = a.flags ? __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 16)
                          : __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0);
    f4v v = {__uint_as_float(r.x), __uint_as_float(r.y), __uint_as_float(r.z), __uint_as_float(r.w)};
    if (a.mean) {
      const float L = (float)(a.offsets[obase + k + 1] - a.offsets[obase + k]);
      v = f4v{v.x / L, v.y / L, v.z / L, v.w / L};
    }
    s_lds[e] = v;
  }
  __syncthreads();
  // The run's output is one contiguous block of (lookups of its bags) x dim
  // floats; the whole workgroup streams it out.
  f4v* out = reinterpret_cast<f4v*>(a.values + base + (lo0 - table_lo) * dim);
  if (n < 0x20000000) {
    if (!WT || lds_w)
      BlockStream<int, WT, true>{s_lds, s_off, s_w, out, (int)n, 0, 0, V, step}.run();
    else
      BlockStream<int, WT, false>{s_lds, s_off, a.weights + lo0, out, (int)n, 0, 0, V, step}.run();
  } else {
    BlockStream<int64_t, WT, false>{s_lds, s_off, WT ? a.weights + lo0 : nullptr, out, n, 0, 0, V, step}.run();
  }
}

// One-GPU stand-in for the gradient All-to-All's arrival: every wavefront
// copies work items (32 KiB pieces of a whole slice, or one (slice, table)
// block per item with per-table slices) from src to dst in slice order with
// device-scope stores, eight 16-byte loads in flight per lane; when the last
// piece of a slice is stored, its flag is incremented.  A few multi-wave
// workgroups keep the copy on a few CUs, so the backward it feeds keeps its
// occupancy everywhere else (a real arrival comes through the links and DMA
// engines and holds no CU at all).
constexpr int DU = 8;  // loads in flight per lane

__global__ __launch_bounds__(1024) void deliver_kernel(const DeliverArgs a) {
  const int lane = threadIdx.x & 63;
  const int64_t wave = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  const int64_t n_waves = (int64_t)gridDim.x * (blockDim.x >> 6);
  const int64_t per_slice = a.per_table ? a.T : a.pieces;
  const int64_t n_items = a.so.n_chunks * per_slice;
  for (int64_t x = __builtin_amdgcn_readfirstlane(wave); x < n_items; x += n_waves) {
    int64_t gs, p;
    if (a.per_table) {  // (slice, table) items in production order
      int32_t tp, unused;
      run_at(a.so, a.T, 1, x, &gs, &tp, &unused);
      p = tp;
    } else {
      gs = x / per_slice;
      p = x - gs * per_slice;
    }
    const int64_t g = slice_at(a.so, gs);
    if (a.per_table) {
      const int t = __builtin_amdgcn_readfirstlane(a.tperm[p]);
      const int dim = __builtin_amdgcn_readfirstlane(a.meta[t].dim);
      const int col_off = __builtin_amdgcn_readfirstlane(a.meta[t].col_off);
      const int v4 = dim >> 2, ld4 = a.sum_dim >> 2;
      const int n = a.C * v4;
      const int64_t base = g * a.chunk_floats + col_off;
      const float4* src = reinterpret_cast<const float4*>(a.src + base);
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
          a.dst + base, 0, ((a.C - 1) * a.sum_dim + dim) * 4, 0x00020000);
      for (int e0 = 0; e0 < n; e0 += 64 * DU) {
        float4 v[DU];
        int off[DU];
#pragma unroll
        for (int u = 0; u < DU; ++u) {
          const int e = e0 + u * 64 + lane;
          const int row = e / v4;
          off[u] = e < n ? row * ld4 + (e - row * v4) : -1;
          v[u] = off[u] >= 0 ? src[off[u]] : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int u = 0; u < DU; ++u) {
          const u4v w = {__float_as_uint(v[u].x), __float_as_uint(v[u].y), __float_as_uint(v[u].z),
                         __float_as_uint(v[u].w)};
          if (off[u] >= 0) __builtin_amdgcn_raw_buffer_store_b128(w, rs, off[u] * 16, 0, 16);  // device scope
        }
      }
      wait_all_memory();
      if (lane == 0)
        __hip_atomic_fetch_add(&a.flags[g * a.T + t], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
      const int64_t chunk_f4 = a.chunk_floats >> 2;
      const int64_t e0 = p * a.piece_f4;
      const int n = (int)min(a.piece_f4, chunk_f4 - e0);
      const float4* src = reinterpret_cast<const float4*>(a.src + g * a.chunk_floats) + e0;
      float4* dst = reinterpret_cast<float4*>(a.dst + g * a.chunk_floats) + e0;
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(dst, 0, n * 16, 0x00020000);
      for (int i0 = 0; i0 < n; i0 += 64 * DU) {
        float4 v[DU];
#pragma unroll
        for (int u = 0; u < DU; ++u) {
          const int i = i0 + u * 64 + lane;
          v[u] = i < n ? src[i] : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int u = 0; u < DU; ++u) {
          const int i = i0 + u * 64 + lane;
          const u4v w = {__float_as_uint(v[u].x), __float_as_uint(v[u].y), __float_as_uint(v[u].z),
                         __float_as_uint(v[u].w)};
          if (i < n) __builtin_amdgcn_raw_buffer_store_b128(w, rs, i * 16, 0, 16);  // device scope
        }
      }
      wait_all_memory();
      if (lane == 0 &&
          __hip_atomic_fetch_add(&a.counters[g], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
              (uint32_t)a.pieces - 1) {
        __hip_atomic_store(&a.counters[g], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_fetch_add(&a.flags[g], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
  }
}

}  // namespace

hipError_t launch_backward(const BackwardArgs& a, int64_t* value_base, int block, size_t lds, hipStream_t stream) {
  hipLaunchKernelGGL(value_base_kernel, dim3(1), dim3(256), 0, stream, a.offsets, a.meta, a.T, a.B, value_base);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(a.weights ? backward_kernel<true> : backward_kernel<false>, dim3((unsigned)a.nruns), dim3(block),
                     lds, stream, a);
  return hipGetLastError();
}

hipError_t launch_deliver(const DeliverArgs& a, int grid, int block, hipStream_t stream) {
  hipLaunchKernelGGL(deliver_kernel, dim3(grid), dim3(block), 0, stream, a);
  return hipGetLastError();
}

}  // namespace ebag
