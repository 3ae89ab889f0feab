// Scan of the cells around a target, shared by the kernels that look for its neighbours.
#pragma once

#include "common.h"

namespace mbd {

// Offset of a cell from a target's, in cells, and the shift sum_a o_a h_a it stands for
// (formed in double, then rounded, in every kernel).
struct CellOffset {
  int x, y, z;
};
template <typename R>
__device__ __forceinline__ void cell_shift(const Geometry& geo, CellOffset o, R& sx, R& sy,
                                           R& sz) {
  sx = (R)(o.x * geo.hv[0][0] + o.y * geo.hv[1][0] + o.z * geo.hv[2][0]);
  sy = (R)(o.x * geo.hv[0][1] + o.y * geo.hv[1][1] + o.z * geo.hv[2][1]);
  sz = (R)(o.x * geo.hv[0][2] + o.y * geo.hv[1][2] + o.z * geo.hv[2][2]);
}

// The offset of a list entry in one word, for scans of at most kPackedRange cells each way.
constexpr int kPackedRange = 511;
__device__ __forceinline__ int pack_off(CellOffset o) {
  return ((o.x + 512) << 20) | ((o.y + 512) << 10) | (o.z + 512);
}
__device__ __forceinline__ CellOffset unpack_off(int off) {
  return {(off >> 20) - 512, ((off >> 10) & 1023) - 512, (off & 1023) - 512};
}

// Cells of the scan around a target's, and cell ci of it around (cx, cy, cz) (x fastest): its
// offset and its index. The target's own cell is the middle one, number cells / 2.
__host__ __device__ inline int scan_cells(const Geometry& geo) {
  return (2 * geo.nr[0] + 1) * (2 * geo.nr[1] + 1) * (2 * geo.nr[2] + 1);
}
__device__ __forceinline__ int scan_cell(const Geometry& geo, int cx, int cy, int cz, int ci,
                                         CellOffset& o) {
  const int nx = 2 * geo.nr[0] + 1, ny = 2 * geo.nr[1] + 1;
  o = {ci % nx - geo.nr[0], (ci / nx) % ny - geo.nr[1], ci / (nx * ny) - geo.nr[2]};
  int wx = (cx + o.x) % geo.nc[0]; if (wx < 0) wx += geo.nc[0];
  int wy = (cy + o.y) % geo.nc[1]; if (wy < 0) wy += geo.nc[1];
  int wz = (cz + o.z) % geo.nc[2]; if (wz < 0) wz += geo.nc[2];
  return cell_index(wx, wy, wz);
}

}  // namespace mbd
