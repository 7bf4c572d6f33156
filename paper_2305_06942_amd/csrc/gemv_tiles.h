// Which workgroup takes which row tile of a GEMV + AllReduce, and into how many
// workgroups a tile is split.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace ebag {

constexpr int kMaxRanks = 16;

// Tiles owned by rank q: [own[q], own[q + 1]); own_mod[q] = own[q] mod P.
// Unsigned: with up to 2^31 - 1 tiles a workgroup's walk, P tiles at a time,
// ends past 2^31.
struct TileOwners {
  uint32_t own[kMaxRanks + 1];
  uint32_t own_mod[kMaxRanks];
};

inline void make_owners(int64_t n_tiles, int32_t R, int32_t P, TileOwners* o) {
  for (int q = 0; q <= R; ++q) o->own[q] = (uint32_t)((q * n_tiles + R - 1) / R);
  for (int q = 0; q < R; ++q) o->own_mod[q] = o->own[q] % (uint32_t)P;
}

// First tile of owner q's block that workgroup p < P handles.
__host__ __device__ inline uint32_t first_tile(const TileOwners& o, int q, uint32_t p, uint32_t P) {
  const uint32_t m = o.own_mod[q];
  return o.own[q] + (p < m ? p + P - m : p - m);
}

// Workgroups a tile's rows are split over: up to kTargetWaves wavefronts in all
// `wgs` workgroups of W waves, each with at least one row and 4 KiB of the matrix
// per tile.  Few waves leave small M idle: 1 x 3233 x 8096 fp32 (51 tiles) took 92
// us unsplit and takes 28 us, 1 x 16384 x 4096 fp16 (512 waves) 40.6 and 29.7.  1024
// waves of 16 KiB in flight are enough: at 2 x 16384 x 4096 fp16 split in two, each
// half staging x again, 53.4 us, whole 50.5 us.  More in all (4096, 8192) were no
// faster and at 1 x 4096 x 4096 bf16 slower (17.0 us at 2048, 23.6, 23.3).
constexpr int64_t kTargetWaves = 1536;
inline int32_t split_for(int64_t wgs, int32_t W, int32_t TM, int64_t row_bytes, int32_t* sub_rows) {
  const int64_t min_rows = row_bytes >= 4096 ? 1 : 4096 / row_bytes;
  int64_t split = kTargetWaves / (wgs * W);
  if (split > TM / (W * min_rows)) split = TM / (W * min_rows);
  if (split < 1) split = 1;
  *sub_rows = (int32_t)((TM + split - 1) / split);
  return (TM + *sub_rows - 1) / *sub_rows;
}

}  // namespace ebag
