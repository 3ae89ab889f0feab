// Launch rules that are plain arithmetic, apart from the kernels so that the CPU checks can
// run them.
#pragma once

#include <algorithm>

namespace mbd {

// gridDim.x of a list-kernel launch whose groups' candidates are split over `parts`
// work-groups and whose right-hand sides over `slices`: a work-group per group (a multiple of
// 8, so that each of the 8 XCDs gets the same number), or as many as keep the launch within
// `cap` work-groups in all (0: no cap); each then walks several groups.
inline int pair_grid_x(int ngroups, int parts, int slices, int cap) {
  const int all = (ngroups + 7) / 8 * 8;
  return cap > 0 ? std::min(all, std::max(8, cap / (parts * slices) / 8 * 8)) : all;
}

}  // namespace mbd
