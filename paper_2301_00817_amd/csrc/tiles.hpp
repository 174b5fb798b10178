// What the kernels that march (i, j) tiles along k share: the deal of tiles to
// XCDs, the columns a tile reads, and the moves between lanes of a tile row.
#pragma once

#include "plane_io.hpp"

namespace lesjet {

// Workgroups are dealt to the eight XCDs (each with its own L2) in turn.  The
// hardware id is remapped so that XCD x receives a contiguous run of tiles,
// i fastest, then j, then the k-chunk: tiles that share halos run at the
// same time on the same L2.
constexpr int NXCD = 8;

struct TileMap {
  int gx, gy, gz;       // tiles along i, j and k-chunks
  int per_xcd;          // ceil(gx gy gz / NXCD)
};

inline TileMap tile_map(int gx, int gy, int gz) {
  TileMap tm;
  tm.gx = gx;
  tm.gy = gy;
  tm.gz = gz;
  tm.per_xcd = (int)(((long long)gx * gy * gz + NXCD - 1) / NXCD);
  return tm;
}

// Tile of this block; false for the blocks that fill up the last XCD's share.
__device__ __forceinline__ bool tile_of_block(const TileMap& tm, int& bx, int& by, int& bz) {
  const int hw = blockIdx.x;
  const int tile = (hw % NXCD) * tm.per_xcd + hw / NXCD;
  if (tile >= tm.gx * tm.gy * tm.gz) return false;
  bx = tile % tm.gx;
  by = (tile / tm.gx) % tm.gy;
  bz = tile / (tm.gx * tm.gy);
  return true;
}

// Byte offset of a column a thread reads: outside the padded box the nearest
// point of it (finite data that no output uses; clamping instead of a
// default value spares the moves that would set the default before every
// load).
template <typename T>
__device__ __forceinline__ unsigned q_col(const Grid& g, int i, int j) {
  return col_off<T>(g, min(max(i, -NG), g.nx + NG - 1), min(max(j, -NG), g.nr + NG - 1));
}

// Value of the lane one column to the left (right) in a tile row of X threads:
// a data-parallel move within the wave (16-lane rows, or the whole wave where
// a row is 32 lanes), executed with every lane active.  The first (last) lane
// of a row gets zero or another row's value, which nothing uses.
template <int CTRL>
__device__ __forceinline__ int lane_mov(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ __forceinline__ float lane_mov(float v) {
  return __builtin_bit_cast(float, lane_mov<CTRL>(__builtin_bit_cast(int, v)));
}
template <int CTRL>
__device__ __forceinline__ double lane_mov(double v) {
  const long long b = __builtin_bit_cast(long long, v);
  const int lo = lane_mov<CTRL>((int)b), hi = lane_mov<CTRL>((int)(b >> 32));
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}
template <int X, typename T>
__device__ __forceinline__ T from_left(T v) {
  static_assert(X == 16 || X == 32, "tile rows of 16 or 32 lanes");
  return lane_mov<X == 16 ? 0x111 : 0x138>(v);      // row_shr:1, wave_shr:1
}
template <int X, typename T>
__device__ __forceinline__ T from_right(T v) {
  return lane_mov<X == 16 ? 0x101 : 0x130>(v);      // row_shl:1, wave_shl:1
}

}  // namespace lesjet
