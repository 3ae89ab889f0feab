// Scan of the cells around a target, shared by the kernels that look for its neighbours.
#pragma once

#include "common.h"

namespace mbd {

// Packed cell offsets (dx, dy, dz) of a list entry, and the shift sum_a o_a h_a they stand
// for (formed in double, then rounded, as everywhere in this file).
__device__ __forceinline__ int pack_off(int dx, int dy, int dz) {
  return ((dx + 512) << 20) | ((dy + 512) << 10) | (dz + 512);
}
template <typename R>
__device__ __forceinline__ void cell_shift(const Geometry& geo, int off, R& sx, R& sy, R& sz) {
  const int dx = (off >> 20) - 512, dy = ((off >> 10) & 1023) - 512, dz = (off & 1023) - 512;
  sx = (R)(dx * geo.hv[0][0] + dy * geo.hv[1][0] + dz * geo.hv[2][0]);
  sy = (R)(dx * geo.hv[0][1] + dy * geo.hv[1][1] + dz * geo.hv[2][1]);
  sz = (R)(dx * geo.hv[0][2] + dy * geo.hv[1][2] + dz * geo.hv[2][2]);
}

// Cell ci of the scan around (cx, cy, cz) (x fastest): its packed offset and its index.
__device__ __forceinline__ int scan_cell(const Geometry& geo, int cx, int cy, int cz, int ci,
                                         int& off) {
  const int nx = 2 * geo.nr[0] + 1, ny = 2 * geo.nr[1] + 1;
  const int dx = ci % nx - geo.nr[0], dy = (ci / nx) % ny - geo.nr[1],
            dz = ci / (nx * ny) - geo.nr[2];
  int wx = (cx + dx) % geo.nc[0]; if (wx < 0) wx += geo.nc[0];
  int wy = (cy + dy) % geo.nc[1]; if (wy < 0) wy += geo.nc[1];
  int wz = (cz + dz) % geo.nc[2]; if (wz < 0) wz += geo.nc[2];
  off = pack_off(dx, dy, dz);
  return cell_index(wx, wy, wz);
}

}  // namespace mbd
