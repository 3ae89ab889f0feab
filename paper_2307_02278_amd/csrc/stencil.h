// Weight of one grid point for component c of a Cartesian dipole, dW/dR_c with
// W = M_p(x) M_p(y) M_p(z) in u and m_a = Mu[a][c]. The operations are spelled out, so that
// every spread kernel forms the same bits.
#pragma once

#include <hip/hip_runtime.h>

namespace mbd {

// The part of an (x, y) column: s for the value of the z spline, t for its slope.
template <typename R>
struct ColumnWeight {
  R s, t;
};
template <typename R>
__device__ __forceinline__ ColumnWeight<R> column_weight(R m0, R m1, R m2, R wx, R dwx, R wy,
                                                         R dwy) {
  ColumnWeight<R> c;
  c.s = fma(m1, wx * dwy, m0 * (dwx * wy));
  c.t = m2 * (wx * wy);
  return c;
}
template <typename R>
__device__ __forceinline__ R point_weight(const ColumnWeight<R>& c, R wz, R dwz) {
  return fma(c.s, wz, c.t * dwz);
}

}  // namespace mbd
