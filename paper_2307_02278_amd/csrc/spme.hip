// SPME spreading and gather (eqs. dipolarr and spme).
//
// Spread: D(k) = sum_j sum_a d_ja dW_j(k)/dR_a with W_j(k) = prod_a M_p(u_ja - k_a),
// stencil k_a = base_a - t_a (t_a = 0..p-1, periodic wrap). With u = Mu R (Mu = rows
// K_a a*_a, any cell), d . grad_R W = sum_b (Mu d)_b dW/du_b: the kernels transform the
// dipole (spread), the gradient (gather) and the Hessian (force gather) with Mu and
// use the derivative tables in u.
// One wavefront owns a 4x4x4 tile of grid points for one chunk of BG right-hand
// sides, accumulates in registers every atom whose stencil reaches the tile, in a
// fixed order, and writes the tile once: no atomics, no clearing pass, and a
// deterministic sum. Chunks of 16 and more multiply the atoms' weights with their dipoles
// on the matrix cores (k_spread); narrower ones share the tile's points out to the lanes of
// each right-hand side (k_spread_brick).
//
// Gather + epilogue: E_rec,i = sum_k grad_i W_i(k) phi(k) (eq. spme), then the
// generalized field E* = E_dir + E_rec + E_self and
//   l~ = Omega w + Diag(g) E*      (eq. lk3, in double precision)
// with per-block partial sums of w . l~ for a_k (eq. recurs2). The lanes of a wavefront are
// right-hand sides x sub-lanes that share an atom's stencil rows x atoms (Lanes below).
#include <algorithm>

#include "common.h"
#include "mfma.h"
#include "stencil.h"

namespace mbd {

namespace {

// Lanes of a gather wavefront: BL right-hand sides x NS sub-lanes that share one atom's
// stencil rows (the P^2 (y, z) rows of P points) x AW atoms. BL is the chunk width BG, or 16
// in small systems: a chunk is then BG / 16 slices of the launch, each wavefront's chain of
// rows is that much shorter and there are that many more wavefronts. Narrow chunks keep NS at 16 or
// less, because 36 rows over 64 sub-lanes leave 28 of them idle, and take several atoms per
// wavefront instead.
template <int BL>
struct Lanes {
  static constexpr int NS = BL >= 8 ? 64 / BL : (BL == 4 ? 8 : 16);
  static constexpr int LA = BL * NS;   // lanes per atom
  static constexpr int AW = 64 / LA;   // atoms per wavefront
};

// The tile points of a spread lane: NSUB = 64 / BG sub-lanes split the 4x4x4 points of a
// tile into NX x NY x NZ bricks, so that a lane's weights along each axis are a run of the
// staged ones.
template <int BG>
struct Brick {
  static constexpr int T = kSpreadTile;
  static constexpr int NP = T * T * T * BG / 64;  // points per lane
  static constexpr int NX = NP < T ? NP : T;
  static constexpr int NY = NP / NX < T ? NP / NX : T;
  static constexpr int NZ = NP / (NX * NY);
  static constexpr int BX = T / NX, BY = T / NY;  // bricks per tile along x and y
};

// Spread with register tiles, for fewer than 16 right-hand sides: one wavefront owns a
// 4x4x4 tile of grid points and keeps the point values of its lane's brick in registers.
// It walks the tile's atom list in a fixed order, so the result is deterministic.
// For one atom the weights along each axis of the tile are
//   w_a(q) = M_p(u_a - k_a) for the tile point k_a = tile origin + q,
// nonzero only when 0 <= t = (base_a - k_a) mod K_a < p, i.e. t = o_a - q with
// o_a = (base_a - origin_a) mod K_a; a batch of atoms at a time has them staged in LDS.
// Bound by the latency of the dipole loads, it stages them beside the weights.
template <typename R, int P, int BG>
__global__ void __launch_bounds__(256)
k_spread_brick(const Geometry geo, const int* __restrict__ tile_start,
         const int* __restrict__ tile_atoms, const int* __restrict__ base,
         const R* __restrict__ th, const R* __restrict__ dth, const R* __restrict__ dv, int B,
         R* __restrict__ grid, size_t chunk_elems, int chunk0) {
  constexpr int T = kSpreadTile;
  typedef Brick<BG> Bk;
  constexpr int NX = Bk::NX, NY = Bk::NY, NZ = Bk::NZ;
  constexpr int NWT = 6 * T;            // staged weights per atom: w, dw along x, y, z
  // atoms per batch: about 20 touch a tile at 0.1 atoms per A^3 and 1.5 points per A; the
  // stage of a work-group stays at 24 KB, so that LDS does not limit the resident waves
  constexpr int NBAT = sizeof(R) == 8 ? 16 : 32;
  constexpr int NPART = 64 / NBAT;      // staging lanes per atom
  __shared__ R wts_all[4][NBAT][NWT];
  __shared__ R dip_all[4][NBAT][3 * BG];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform
  const int lane = threadIdx.x & 63;
  R(*wts)[NWT] = wts_all[wave];
  const int ntiles = geo.tiles[0] * geo.tiles[1] * geo.tiles[2];
  // Blocks are dealt round-robin to the 8 XCDs (gridDim.x is a multiple of 8):
  // each XCD takes one contiguous range of tiles, a slab of the grid, so the
  // dipoles of the atoms it spreads stay in its L2.
  const int per = gridDim.x / 8;
  const int tile = ((blockIdx.x % 8) * per + blockIdx.x / 8) * 4 + wave;
  if (tile >= ntiles) return;
  const int chunk = blockIdx.y + chunk0;
  const int b = lane % BG;
  const int sub = lane / BG;
  // origin of the lane's brick in the tile
  const int px0 = (sub % Bk::BX) * NX, py0 = (sub / Bk::BX % Bk::BY) * NY,
            pz0 = sub / (Bk::BX * Bk::BY) * NZ;
  const int tx = tile % geo.tiles[0];
  const int ty = (tile / geo.tiles[0]) % geo.tiles[1];
  const int tz = tile / (geo.tiles[0] * geo.tiles[1]);
  const int x0 = tx * T, y0 = ty * T, z0 = tz * T;
  const int K1 = geo.K[0], K2 = geo.K[1], K3 = geo.K[2];
  R acc[NX * NY * NZ];
#pragma unroll
  for (int i = 0; i < NX * NY * NZ; ++i) acc[i] = R(0);
  const int lo = tile_start[tile], hi = tile_start[tile + 1];
  for (int a0 = lo; a0 < hi; a0 += NBAT) {
    const int na = min(NBAT, hi - a0);
    // Stage: lane i computes the tile-clipped weights of the batch's atom i % NBAT, the
    // NPART lanes of an atom every NPART-th of its six weight rows.
    {
      const int i = lane % NBAT, part = lane / NBAT;
      if (i < na) {
        const int s = tile_atoms[a0 + i];
        int o[3] = {base[3 * s] - x0, base[3 * s + 1] - y0, base[3 * s + 2] - z0};
        if (o[0] < 0) o[0] += K1;
        if (o[1] < 0) o[1] += K2;
        if (o[2] < 0) o[2] += K3;
        const R* thp = th + (size_t)s * 3 * P;
        const R* dthp = dth + (size_t)s * 3 * P;
#pragma unroll
        for (int ax = 0; ax < 3; ++ax)
#pragma unroll
          for (int d = 0; d < 2; ++d) {
            if ((2 * ax + d) % NPART != part) continue;
#pragma unroll
            for (int q = 0; q < T; ++q) {
              const int t = o[ax] - q;
              const bool v = t >= 0 && t < P;
              wts[i][(2 * ax + d) * T + q] = v ? (d ? dthp : thp)[ax * P + t] : R(0);
            }
          }
        for (int e = part; e < 3 * BG; e += NPART)
          dip_all[wave][i][e] = dv[((size_t)s * 3 + e / BG) * B + chunk * BG + e % BG];
      }
    }
    // the batch's LDS writes are visible to the whole wavefront before it reads them
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const R m00 = (R)geo.Mu[0][0], m01 = (R)geo.Mu[0][1], m02 = (R)geo.Mu[0][2];
    const R m10 = (R)geo.Mu[1][0], m11 = (R)geo.Mu[1][1], m12 = (R)geo.Mu[1][2];
    const R m20 = (R)geo.Mu[2][0], m21 = (R)geo.Mu[2][1], m22 = (R)geo.Mu[2][2];
    for (int a = 0; a < na; ++a) {
      // dipole in u: (Mu d)_b
      const R* n = &dip_all[wave][a][b];
      const R d0 = m00 * n[0] + m01 * n[BG] + m02 * n[2 * BG];
      const R d1 = m10 * n[0] + m11 * n[BG] + m12 * n[2 * BG];
      const R d2 = m20 * n[0] + m21 * n[BG] + m22 * n[2 * BG];
      const R* wa = wts[a];
      R wx[NX], dwx[NX], wy[NY], dwy[NY], wz[NZ], dwz[NZ];
#pragma unroll
      for (int q = 0; q < NX; ++q) { wx[q] = wa[px0 + q]; dwx[q] = wa[T + px0 + q]; }
#pragma unroll
      for (int q = 0; q < NY; ++q) { wy[q] = wa[2 * T + py0 + q]; dwy[q] = wa[3 * T + py0 + q]; }
#pragma unroll
      for (int q = 0; q < NZ; ++q) { wz[q] = wa[4 * T + pz0 + q]; dwz[q] = wa[5 * T + pz0 + q]; }
      // every point of the brick: the staged weights are zero outside the stencil, and
      // a branch-free loop issues fewer instructions than uniform per-point tests
#pragma unroll
      for (int pz = 0; pz < NZ; ++pz) {
#pragma unroll
        for (int py = 0; py < NY; ++py) {
          const R A = d0 * wy[py] * wz[pz];
          const R Bc = d1 * dwy[py] * wz[pz] + d2 * wy[py] * dwz[pz];
#pragma unroll
          for (int px = 0; px < NX; ++px) {
            R& q = acc[(pz * NY + py) * NX + px];
            q = fma(dwx[px], A, q);
            q = fma(wx[px], Bc, q);
          }
        }
      }
    }
    // all reads of this batch are done before the next batch overwrites the stage
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  R* g = grid + (size_t)chunk * chunk_elems;
  const int XS = K1 + 2;
#pragma unroll
  for (int i = 0; i < NX * NY * NZ; ++i) {
    const int x = x0 + px0 + i % NX, y = y0 + py0 + (i / NX) % NY, z = z0 + pz0 + i / (NX * NY);
    if (x < K1 && y < K2 && z < K3) g[(((size_t)z * K2 + y) * XS + x) * BG + b] = acc[i];
  }
}

// Spread on the matrix cores, for chunks of BG = 16 NT right-hand sides: over the atoms of
// its list a 4x4x4 tile is a dense product,
//   D[point][rhs] = sum_k W[point][k] d[k][rhs],  k = 3 atom + component,
// of four 16-point planes (rows; one z each) with NT column tiles. A wavefront owns a tile
// for a chunk and takes four atoms (12 rows of k, three instructions of four) at a time: in
// step u lane row r holds k = 4 u + r, so its atom and component are fixed, and it forms the
// weights of its (x, y) column for the four planes from the staged splines. Column col of
// tile t is right-hand side NT col + t, so dipoles and grid rows move as vectors. The sum
// runs in list order, atom by atom, component by component, whatever the split into fours
// (zero weights outside a stencil add nothing). With one lane per right-hand side, an atom is
// one serial step of 128 multiply-adds in every lane; here four are one step of 48 matrix
// instructions. Boxes of 525 to 4200 atoms, 64 right-hand sides: 26.6 us a launch before,
// 20.4 here; 651 atoms, 16: 15.8 and 12.3; 24k atoms, K = 96, 64: 112 and 105, of which the
// matrix instructions are 46, the weights and the staging about 35 and the 226 MB grid
// write, which starts when a tile is done, 38.
template <typename R, int P, int NT>
__global__ void __launch_bounds__(256)
k_spread(const Geometry geo, const int* __restrict__ tile_start,
         const int* __restrict__ tile_atoms, const int* __restrict__ base,
         const R* __restrict__ th, const R* __restrict__ dth, const R* __restrict__ dv, int B,
         R* __restrict__ grid, size_t chunk_elems, int chunk0) {
  typedef typename Mma<R>::acc Acc;
  constexpr int T = kSpreadTile;
  constexpr int BG = 16 * NT;
  constexpr int VN = NT * (int)sizeof(R) > 16 ? 16 / (int)sizeof(R) : NT;  // reals per vector
  constexpr int NWT = 6 * T;            // staged weights per atom: w, dw along x, y, z
  constexpr int NBAT = sizeof(R) == 8 ? 32 : 64;  // atoms per batch (24 KB a work-group)
  __shared__ alignas(16) R wts_all[4][NBAT][NWT];
  __shared__ int sat_all[4][NBAT];      // atom index of each staged slot
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform
  const int lane = threadIdx.x & 63;
  const int col = lane & 15, row = lane >> 4;
  R(*wts)[NWT] = wts_all[wave];
  int* sat = sat_all[wave];
  const int ntiles = geo.tiles[0] * geo.tiles[1] * geo.tiles[2];
  // each XCD takes one contiguous range of tiles (gridDim.x is a multiple of 8), a slab of
  // the grid, so the dipoles of the atoms it spreads stay in its L2
  const int per = gridDim.x / 8;
  const int tile = ((blockIdx.x % 8) * per + blockIdx.x / 8) * 4 + wave;
  if (tile >= ntiles) return;
  const int chunk = blockIdx.y + chunk0;
  const int tx = tile % geo.tiles[0];
  const int ty = (tile / geo.tiles[0]) % geo.tiles[1];
  const int tz = tile / (geo.tiles[0] * geo.tiles[1]);
  const int x0 = tx * T, y0 = ty * T, z0 = tz * T;
  const int K1 = geo.K[0], K2 = geo.K[1], K3 = geo.K[2];
  // step u of a block of four atoms: this lane's atom, component and column of Mu
  int au[3], cu[3];
  R mu[3][3];
#pragma unroll
  for (int u = 0; u < 3; ++u) {
    au[u] = (4 * u + row) / 3;
    cu[u] = (4 * u + row) % 3;
#pragma unroll
    for (int a = 0; a < 3; ++a) mu[u][a] = (R)geo.Mu[a][cu[u]];
  }
  const int px = col % T, py = col / T;  // the lane's (x, y) column as a matrix row
  const R* dcol = dv + chunk * BG + NT * col;
  Acc acc[T][NT];
#pragma unroll
  for (int z = 0; z < T; ++z)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[z][t] = Acc{R(0), R(0), R(0), R(0)};
  const int lo = tile_start[tile], hi = tile_start[tile + 1];
  for (int a0 = lo; a0 < hi; a0 += NBAT) {
    const int na = min(NBAT, hi - a0);
    const int na4 = (na + 3) & ~3;  // (zero weights on the last atom's dipoles past na)
    // Stage the tile-clipped weights, one (atom, axis, value or slope) row of four a lane
    // and pass: an atom's rows are neighbours in memory, and every lane has one
    for (int e = lane; e < 6 * na4; e += 64) {
      const int i = e / 6, ax = e % 6 % 3, d = e % 6 / 3;
      const int s = tile_atoms[a0 + min(i, na - 1)];
      int o = base[3 * s + ax] - (ax == 0 ? x0 : ax == 1 ? y0 : z0);
      if (o < 0) o += ax == 0 ? K1 : ax == 1 ? K2 : K3;
      const R* p = (d ? dth : th) + ((size_t)s * 3 + ax) * P;
#pragma unroll
      for (int q = 0; q < T; ++q) {
        const int t = o - q;
        const bool v = i < na && t >= 0 && t < P;
        wts[i][(2 * ax + d) * T + q] = v ? p[t] : R(0);
      }
      if (e % 6 == 0) sat[i] = s;
    }
    // the batch's LDS writes are visible to the whole wavefront before it reads them
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    R d[3][NT];  // dipoles of the next four atoms
    auto fetch = [&](int a) {
#pragma unroll
      for (int u = 0; u < 3; ++u) {
        const Pack<R, VN>* p = reinterpret_cast<const Pack<R, VN>*>(
            dcol + ((size_t)sat[a + au[u]] * 3 + cu[u]) * B);
#pragma unroll
        for (int q = 0; q < NT / VN; ++q) {
          const Pack<R, VN> v = p[q];
#pragma unroll
          for (int w = 0; w < VN; ++w) d[u][VN * q + w] = v.v[w];
        }
      }
    };
    fetch(0);
    for (int a = 0; a < na4; a += 4) {
      R cur[3][NT];
#pragma unroll
      for (int u = 0; u < 3; ++u)
#pragma unroll
        for (int t = 0; t < NT; ++t) cur[u][t] = d[u][t];
      if (a + 4 < na4) fetch(a + 4);
#pragma unroll
      for (int u = 0; u < 3; ++u) {
        const R* wa = wts[a + au[u]];
        const ColumnWeight<R> cw = column_weight<R>(mu[u][0], mu[u][1], mu[u][2], wa[px],
                                                    wa[T + px], wa[2 * T + py], wa[3 * T + py]);
#pragma unroll
        for (int z = 0; z < T; ++z) {
          const R w = point_weight<R>(cw, wa[4 * T + z], wa[5 * T + z]);
#pragma unroll
          for (int t = 0; t < NT; ++t) acc[z][t] = Mma<R>::fma(w, cur[u][t], acc[z][t]);
        }
      }
    }
    // all reads of this batch are done before the next batch overwrites the stage
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  R* g = grid + (size_t)chunk * chunk_elems + NT * col;
  const int XS = K1 + 2;
#pragma unroll
  for (int z = 0; z < T; ++z)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = Mma<R>::row(row, r);
      const int x = x0 + i % T, y = y0 + i / T;
      if (x >= K1 || y >= K2 || z0 + z >= K3) continue;
      Pack<R, VN>* o =
          reinterpret_cast<Pack<R, VN>*>(g + (((size_t)(z0 + z) * K2 + y) * XS + x) * BG);
#pragma unroll
      for (int q = 0; q < NT / VN; ++q) {
        Pack<R, VN> v;
#pragma unroll
        for (int w = 0; w < VN; ++w) v.v[w] = acc[z][VN * q + w][r];
        o[q] = v;
      }
    }
}

// Row r = P t3 + t2 of an atom's stencil rows: its first grid value (without the x index).
template <typename R, int P, int BG>
__device__ __forceinline__ const R* stencil_row(const R* gr, int by, int bz, int t2, int t3,
                                                int K2, int K3, int XS) {
  int k2 = by - t2, k3 = bz - t3;
  if (k2 < 0) k2 += K2;
  if (k3 < 0) k3 += K3;
  return gr + ((size_t)k3 * K2 + k2) * XS * BG;
}

// The rest of one application of C for one atom and right-hand side: from the gathered field
// of the reciprocal part (in u) to lt = g (E_rec + E_dir + E_self) + om2 w.
template <typename R>
struct Epilogue {
  const R* Ed;        // direct field, ed_parts partial sums
  int ed_parts;
  const double* w;    // the vector C is applied to
  const double* g;
  const double* om2;
  uint32_t comps;
  double self_coef;
  double* lt;
};

// One component per sub-lane where there are at least three, else all by the first. Returns
// this lane's share of w . lt.
template <typename R, int NS>
__device__ __forceinline__ double finish_field(const Epilogue<R>& ep, int n, int s, int sub,
                                               int bg, int B, R e0, R e1, R e2) {
  double dot = 0.0;
  const double gs = ep.g[s];
  const double o2 = ep.om2[s];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    if (NS >= 4 ? a != sub : sub != 0) continue;
    const size_t idx = ((size_t)s * 3 + a) * B + bg;
    const double wv = ep.w[idx];
    double E = (a == 0) ? (double)e0 : (a == 1) ? (double)e1 : (double)e2;
    if (ep.comps & MBD_C_DIR) {
      E += (double)ep.Ed[idx];
      // the parts in order, five loads in flight (past the last part: a zero)
      const size_t pstride = (size_t)3 * n * B;
      for (int q0 = 1; q0 < ep.ed_parts; q0 += 5) {
        R x[5];
#pragma unroll
        for (int i = 0; i < 5; ++i) x[i] = ep.Ed[min(q0 + i, ep.ed_parts - 1) * pstride + idx];
#pragma unroll
        for (int i = 0; i < 5; ++i) E += q0 + i < ep.ed_parts ? (double)x[i] : 0.0;
      }
    }
    if (ep.comps & MBD_C_SELF) E += ep.self_coef * gs * wv;
    double l = gs * E;
    if (ep.comps & MBD_C_DIAG) l += o2 * wv;
    ep.lt[idx] = l;
    dot += wv * l;
  }
  return dot;
}

template <typename R, int P, int BG, int BL>
__global__ void __launch_bounds__(512)
k_gather_epilogue(const Geometry geo, const int* __restrict__ base, const R* __restrict__ th,
                  const R* __restrict__ dth, const R* __restrict__ grid, size_t chunk_elems,
                  const Epilogue<R> ep, int B, double* __restrict__ part, int chunk0) {
  constexpr int NS = Lanes<BL>::NS, LA = Lanes<BL>::LA, AW = Lanes<BL>::AW;
  __shared__ double red[8 * BL];
  const int nw = blockDim.x >> 6;  // wavefronts per work-group (4 or 8)
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform
  const int lane = threadIdx.x & 63;
  const int slice = blockIdx.y % (BG / BL);  // of the chunk's right-hand sides
  const int b = slice * BL + lane % BL;
  const int sub = lane % LA / BL;
  const int chunk = blockIdx.y / (BG / BL) + chunk0;
  const int bg = chunk * BG + b;
  const R* gr = grid + (size_t)chunk * chunk_elems;
  const int K1 = geo.K[0], K2 = geo.K[1], K3 = geo.K[2];
  const int XS = K1 + 2;
  double dot = 0.0;
  // Blocks are dealt round-robin to the 8 XCDs. Each XCD takes one contiguous range
  // of sorted atoms and sweeps it with all of its wavefronts side by side (wave lw
  // takes atoms lo + AW lw, lo + AW (lw + nwx), ...), so the atoms in flight on an XCD
  // at any time are consecutive, i.e. spatially compact, and their stencils share L2.
  const int nb8 = gridDim.x / 8;
  const int xcd = blockIdx.x % 8;
  const int nwx = nb8 * nw;
  const int lw = (blockIdx.x / 8) * nw + wave;
  const int x_lo = (int)(((long)geo.n * xcd) / 8);
  const int x_hi = (int)(((long)geo.n * (xcd + 1)) / 8);
  for (int s0 = x_lo + lw * AW; s0 < x_hi; s0 += nwx * AW) {
    // (past the range: its last atom again, computed and dropped)
    const int s = AW == 1 ? s0 : min(s0 + lane / LA, x_hi - 1);
    const bool valid = AW == 1 || s0 + lane / LA < x_hi;
    R e0 = R(0), e1 = R(0), e2 = R(0);
    if (ep.comps & MBD_C_REC) {
      const R* thp = th + s * 3 * P;
      const R* dthp = dth + s * 3 * P;
      R mx[P], dmx[P];
#pragma unroll
      for (int t = 0; t < P; ++t) { mx[t] = thp[t]; dmx[t] = dthp[t]; }
      const int bx = base[3 * s], by = base[3 * s + 1], bz = base[3 * s + 2];
      int kxs[P];
#pragma unroll
      for (int t1 = 0; t1 < P; ++t1) {
        int k1 = bx - t1;
        if (k1 < 0) k1 += K1;
        kxs[t1] = k1 * BG + b;
      }
      auto row = [&](const R* line, R my, R dmy, R mz, R dmz) {
        R sx = R(0), sy = R(0);
#pragma unroll
        for (int t1 = 0; t1 < P; ++t1) {
          const R phi = line[kxs[t1]];
          sx += dmx[t1] * phi;
          sy += mx[t1] * phi;
        }
        e0 += sx * my * mz;
        e1 += sy * dmy * mz;
        e2 += sy * my * dmz;
      };
      if constexpr (NS == 1) {
        R my[P], dmy[P], mz[P], dmz[P];
#pragma unroll
        for (int t = 0; t < P; ++t) {
          my[t] = thp[P + t]; dmy[t] = dthp[P + t];
          mz[t] = thp[2 * P + t]; dmz[t] = dthp[2 * P + t];
        }
#pragma unroll
        for (int t3 = 0; t3 < P; ++t3)
#pragma unroll
          for (int t2 = 0; t2 < P; ++t2)
            row(stencil_row<R, P, BG>(gr, by, bz, t2, t3, K2, K3, XS), my[t2], dmy[t2], mz[t3],
                dmz[t3]);
      } else {
        // the rows r = sub, sub + NS, ... with the row index in a register: one pass over
        // ceil(P^2 / NS) rows for the whole wavefront (unrolled over all P^2 rows with a
        // test per row, every row is issued for the sake of the few lanes that own it)
        constexpr int NR = (P * P + NS - 1) / NS;
#pragma unroll (NR <= 5 ? NR : 3)
        for (int i = 0; i < NR; ++i) {
          const int r = min(sub + i * NS, P * P - 1);
          const bool own = sub + i * NS < P * P;
          const int t3 = r / P, t2 = r % P;
          const R mz = own ? thp[2 * P + t3] : R(0), dmz = own ? dthp[2 * P + t3] : R(0);
          row(stencil_row<R, P, BG>(gr, by, bz, t2, t3, K2, K3, XS), thp[P + t2], dthp[P + t2],
              mz, dmz);
        }
      }
      // combine the sub-lanes that split the stencil rows
#pragma unroll
      for (int off = BL; off < LA; off <<= 1) {
        e0 += __shfl_xor(e0, off);
        e1 += __shfl_xor(e1, off);
        e2 += __shfl_xor(e2, off);
      }
      // gradient in u -> gradient in R: Mu^T
      const R g0 = e0, g1 = e1, g2 = e2;
      e0 = (R)geo.Mu[0][0] * g0 + (R)geo.Mu[1][0] * g1 + (R)geo.Mu[2][0] * g2;
      e1 = (R)geo.Mu[0][1] * g0 + (R)geo.Mu[1][1] * g1 + (R)geo.Mu[2][1] * g2;
      e2 = (R)geo.Mu[0][2] * g0 + (R)geo.Mu[1][2] * g1 + (R)geo.Mu[2][2] * g2;
    }
    if (valid && sub < 3)
      dot += finish_field<R, NS>(ep, geo.n, s, sub, bg, B, e0, e1, e2);
  }
  // per-RHS sum over the lanes of a right-hand side, then the work-group's wavefronts
#pragma unroll
  for (int off = BL; off < 64; off <<= 1) dot += __shfl_xor(dot, off);
  if (lane < BL) red[wave * BL + lane] = dot;
  __syncthreads();
  if (threadIdx.x < BL) {
    double t = 0.0;
    for (int wv = 0; wv < nw; ++wv) t += red[wv * BL + threadIdx.x];
    part[((size_t)blockIdx.x * kPartSlots + 0) * B + chunk * BG + slice * BL + threadIdx.x] = t;
  }
}

// Reciprocal-space part of the bilinear force term for one reverse step: with
// S = D_p^T phi_q (D_x the spread of dipoles x, phi_x = G~ * D_x, symmetric in p, q),
//   dS/dR_a = sum_k H_a(k) (p_a phi_q(k) + q_a phi_p(k)),  H_a(k) = grad_a grad_a W_a(k),
// the Hessian of the atom's weight product (d^2/du^2 along one axis: ddth; mixed
// axes: dth dth). One call adds sum_k H_a(k) h_a phi(k) for one grid (phi) and the
// other dipole set h, summed over the chunk's right-hand sides, to fsum (wavefront
// per atom, lanes over right-hand sides and stencil rows as in the gather). With EPI the
// grid is also that of the adjoint matvec, whose gather is the same pass over the same rows
// (its two row sums are the Hessian's first two): one read of the grid instead of two. 12k
// atoms, 64 right-hand sides: gather 61 us and force 55 before, 64 us together.
template <typename R, int P, int BG, bool EPI>
__global__ void __launch_bounds__(512)
k_spme_force(const Geometry geo, const int* __restrict__ base, const R* __restrict__ th,
             const R* __restrict__ dth, const R* __restrict__ ddth, const R* __restrict__ grid,
             size_t chunk_elems, const R* __restrict__ hv, int B, int chunk0,
             double* __restrict__ fsum, const double* __restrict__ hscale,
             const Epilogue<R> ep) {
  constexpr int NS = Lanes<BG>::NS, LA = Lanes<BG>::LA, AW = Lanes<BG>::AW;
  const int nw = blockDim.x >> 6;  // wavefronts per work-group (4 or 8)
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform
  const int lane = threadIdx.x & 63;
  const int b = lane % BG;
  const int sub = lane % LA / BG;
  const int chunk = blockIdx.y + chunk0;
  const int bg = chunk * BG + b;
  const R* gr = grid + (size_t)chunk * chunk_elems;
  const int K1 = geo.K[0], K2 = geo.K[1], K3 = geo.K[2];
  const int XS = K1 + 2;
  const int nb8 = gridDim.x / 8;
  const int xcd = blockIdx.x % 8;
  const int nwx = nb8 * nw;
  const int lw = (blockIdx.x / 8) * nw + wave;
  const int x_lo = (int)(((long)geo.n * xcd) / 8);
  const int x_hi = (int)(((long)geo.n * (xcd + 1)) / 8);
  for (int s0 = x_lo + lw * AW; s0 < x_hi; s0 += nwx * AW) {
    const int s = AW == 1 ? s0 : min(s0 + lane / LA, x_hi - 1);
    const bool valid = AW == 1 || s0 + lane / LA < x_hi;
    const R* tp = th + (size_t)s * 3 * P;
    const R* dp = dth + (size_t)s * 3 * P;
    const R* ddp = ddth + (size_t)s * 3 * P;
    R mx[P], dmx[P], ddmx[P];
#pragma unroll
    for (int t = 0; t < P; ++t) {
      mx[t] = tp[t]; dmx[t] = dp[t]; ddmx[t] = ddp[t];
    }
    const int bx = base[3 * s], by = base[3 * s + 1], bz = base[3 * s + 2];
    int kxs[P];
#pragma unroll
    for (int t1 = 0; t1 < P; ++t1) {
      int k1 = bx - t1;
      if (k1 < 0) k1 += K1;
      kxs[t1] = k1 * BG + b;
    }
    R hxx = R(0), hyy = R(0), hzz = R(0), hxy = R(0), hxz = R(0), hyz = R(0);
    R e0 = R(0), e1 = R(0), e2 = R(0);
    auto row = [&](const R* line, R my, R dmy, R ddmy, R mz3, R dmz3, R ddmz3) {
      R s0 = R(0), s1 = R(0), s2 = R(0);
#pragma unroll
      for (int t1 = 0; t1 < P; ++t1) {
        const R phi = line[kxs[t1]];
        s0 += mx[t1] * phi;
        s1 += dmx[t1] * phi;
        s2 += ddmx[t1] * phi;
      }
      hxx += s2 * my * mz3;
      hyy += s0 * ddmy * mz3;
      hzz += s0 * my * ddmz3;
      hxy += s1 * dmy * mz3;
      hxz += s1 * my * dmz3;
      hyz += s0 * dmy * dmz3;
      if constexpr (EPI) {
        e0 += s1 * my * mz3;
        e1 += s0 * dmy * mz3;
        e2 += s0 * my * dmz3;
      }
    };
    if constexpr (NS == 1) {
      R my[P], dmy[P], ddmy[P];
#pragma unroll
      for (int t = 0; t < P; ++t) {
        my[t] = tp[P + t]; dmy[t] = dp[P + t]; ddmy[t] = ddp[P + t];
      }
      // one z plane of the stencil at a time (not unrolled: unrolled, the compiler keeps
      // all p^3 grid values of an atom in flight and the kernel runs at 2 waves per SIMD)
#pragma unroll 1
      for (int t3 = 0; t3 < P; ++t3) {
        const R mz3 = tp[2 * P + t3], dmz3 = dp[2 * P + t3], ddmz3 = ddp[2 * P + t3];
#pragma unroll
        for (int t2 = 0; t2 < P; ++t2)
          row(stencil_row<R, P, BG>(gr, by, bz, t2, t3, K2, K3, XS), my[t2], dmy[t2], ddmy[t2],
              mz3, dmz3, ddmz3);
      }
    } else {
      // rows by register index, as in the gather
      constexpr int NR = (P * P + NS - 1) / NS;
#pragma unroll 3
      for (int i = 0; i < NR; ++i) {
        const int r = min(sub + i * NS, P * P - 1);
        const bool own = sub + i * NS < P * P;
        const int t3 = r / P, t2 = r % P;
        row(stencil_row<R, P, BG>(gr, by, bz, t2, t3, K2, K3, XS), tp[P + t2], dp[P + t2],
            ddp[P + t2], own ? tp[2 * P + t3] : R(0), own ? dp[2 * P + t3] : R(0),
            own ? ddp[2 * P + t3] : R(0));
      }
    }
    if constexpr (EPI) {
#pragma unroll
      for (int off = BG; off < LA; off <<= 1) {
        e0 += __shfl_xor(e0, off);
        e1 += __shfl_xor(e1, off);
        e2 += __shfl_xor(e2, off);
      }
      if (valid && sub < 3)
        finish_field<R, NS>(
            ep, geo.n, s, sub, bg, B,
            (R)geo.Mu[0][0] * e0 + (R)geo.Mu[1][0] * e1 + (R)geo.Mu[2][0] * e2,
            (R)geo.Mu[0][1] * e0 + (R)geo.Mu[1][1] * e1 + (R)geo.Mu[2][1] * e2,
            (R)geo.Mu[0][2] * e0 + (R)geo.Mu[1][2] * e1 + (R)geo.Mu[2][2] * e2);
    }
    const size_t o = (size_t)s * 3 * B + bg;
    // h, times a per-right-hand-side factor when the grid belongs to a scaled dipole set
    const R hs = hscale ? (R)hscale[(size_t)bg * 16] : R(1);
    const R c0 = hs * hv[o], c1 = hs * hv[o + B], c2 = hs * hv[o + 2 * B];
    // Hessian in u: H_R = Mu^T H_u Mu, applied as Mu^T (H_u (Mu h))
    const R h0 = (R)geo.Mu[0][0] * c0 + (R)geo.Mu[0][1] * c1 + (R)geo.Mu[0][2] * c2;
    const R h1 = (R)geo.Mu[1][0] * c0 + (R)geo.Mu[1][1] * c1 + (R)geo.Mu[1][2] * c2;
    const R h2 = (R)geo.Mu[2][0] * c0 + (R)geo.Mu[2][1] * c1 + (R)geo.Mu[2][2] * c2;
    const R u0 = hxx * h0 + hxy * h1 + hxz * h2;
    const R u1 = hxy * h0 + hyy * h1 + hyz * h2;
    const R u2 = hxz * h0 + hyz * h1 + hzz * h2;
    double f0 = (double)((R)geo.Mu[0][0] * u0 + (R)geo.Mu[1][0] * u1 + (R)geo.Mu[2][0] * u2);
    double f1 = (double)((R)geo.Mu[0][1] * u0 + (R)geo.Mu[1][1] * u1 + (R)geo.Mu[2][1] * u2);
    double f2 = (double)((R)geo.Mu[0][2] * u0 + (R)geo.Mu[1][2] * u1 + (R)geo.Mu[2][2] * u2);
#pragma unroll
    for (int off = 1; off < LA; off <<= 1) {
      f0 += __shfl_xor(f0, off);
      f1 += __shfl_xor(f1, off);
      f2 += __shfl_xor(f2, off);
    }
    if (valid && lane % LA == 0) {
      fsum[3 * (size_t)s] += f0;
      fsum[3 * (size_t)s + 1] += f1;
      fsum[3 * (size_t)s + 2] += f2;
    }
  }
}

// Wavefronts per work-group of the gather-type kernels (one atom per wavefront at a time,
// more for chunks of fewer than 8 right-hand sides).
int gather_waves(const Geometry& geo) { return geo.gather_waves == 8 ? 8 : 4; }

}  // namespace

// Work-groups of a gather launch (a multiple of 8 for the XCD ranges): as many as hold every
// atom at once, up to kRedBlocks; more would only add empty partial sums for the reduction
// of a_k (96 atoms: 8 instead of 1024).
int gather_blocks(const Geometry& geo, int BG) {
  const int aw = BG >= 8 ? 1 : (BG == 1 ? 4 : 2);  // Lanes<BG>::AW
  const int per = 8 * gather_waves(geo) * aw;
  return std::min(kRedBlocks, (geo.n + per - 1) / per * 8);
}

template <typename R>
void launch_spread(const Geometry& geo, const SysBuffers& b, int B, int BG, int chunk0,
                   int nchunks, hipStream_t st) {
  const size_t chunk = (size_t)geo.K[2] * geo.K[1] * (geo.K[0] + 2) * BG;
  const int ntiles = geo.tiles[0] * geo.tiles[1] * geo.tiles[2];
  dim3 grd(((ntiles + 3) / 4 + 7) / 8 * 8, nchunks);  // a multiple of 8 (XCD remap)
#define MBD_SPREAD(KERNEL, PP, NN)                                                          \
  KERNEL<R, PP, NN><<<grd, 256, 0, st>>>(geo, b.tile_start, b.tile_atoms, b.base,          \
                                         (const R*)b.th, (const R*)b.dth, (const R*)b.dv,  \
                                         B, (R*)b.grid, chunk, chunk0)
#define MBD_SPREAD_P(KERNEL, NN)              \
  switch (geo.p) {                            \
    case 4: MBD_SPREAD(KERNEL, 4, NN); break; \
    case 6: MBD_SPREAD(KERNEL, 6, NN); break; \
    case 8: MBD_SPREAD(KERNEL, 8, NN); break; \
  }
  switch (BG) {
    case 1: MBD_SPREAD_P(k_spread_brick, 1); break;
    case 2: MBD_SPREAD_P(k_spread_brick, 2); break;
    case 4: MBD_SPREAD_P(k_spread_brick, 4); break;
    case 8: MBD_SPREAD_P(k_spread_brick, 8); break;
    case 16: MBD_SPREAD_P(k_spread, 1); break;
    case 32: MBD_SPREAD_P(k_spread, 2); break;
    case 64: MBD_SPREAD_P(k_spread, 4); break;
  }
#undef MBD_SPREAD_P
#undef MBD_SPREAD
}

template <typename R>
static Epilogue<R> epilogue_of(const Geometry& geo, const SysBuffers& b, const double* w, int B,
                               uint32_t comps) {
  return {(const R*)b.Ed, pair_parts(geo, b, B), w, b.g, b.om2, comps,
          -4.0 * geo.tau * geo.tau * geo.tau / (3.0 * sqrt(M_PI)), b.Lt};
}

template <typename R>
void launch_epilogue(const Geometry& geo, const SysBuffers& b, const double* w, int B, int BG,
                     int chunk0, int nchunks, uint32_t comps, hipStream_t st) {
  const size_t chunk = (size_t)geo.K[2] * geo.K[1] * (geo.K[0] + 2) * BG;
  // slices of 16 while whole chunks would leave about a wavefront per SIMD; then the sub-lanes
  // of a slice, which share rows unevenly, cost more. Whole and in slices, us a launch:
  // chunks of 32, 192 atoms 11.4 and 10.0, 648 11.7 and 10.6, 1029 11.6 and 11.1, 2187 15.5
  // and 16.9; chunks of 64, 192 atoms 12.3 and 10.3, 648 12.9 and 12.2, 1029 15.4 and 16.0,
  // 3000 19.9 and 27.1
  const bool sliced = geo.n < 1024;
  const dim3 grd(gather_blocks(geo, BG), nchunks * (sliced && BG > 16 ? BG / 16 : 1));
  const Epilogue<R> ep = epilogue_of<R>(geo, b, w, B, comps);
#define MBD_GATHER(PP, BB, LL)                                                              \
  k_gather_epilogue<R, PP, BB, LL><<<grd, 64 * gather_waves(geo), 0, st>>>(               \
      geo, b.base, (const R*)b.th, (const R*)b.dth, (const R*)b.grid, chunk, ep, B,        \
      b.part, chunk0)
#define MBD_GATHER_P(BB, LL)                \
  switch (geo.p) {                          \
    case 4: MBD_GATHER(4, BB, LL); break;   \
    case 6: MBD_GATHER(6, BB, LL); break;   \
    case 8: MBD_GATHER(8, BB, LL); break;   \
  }
  switch (BG) {
    case 1: MBD_GATHER_P(1, 1); break;
    case 2: MBD_GATHER_P(2, 2); break;
    case 4: MBD_GATHER_P(4, 4); break;
    case 8: MBD_GATHER_P(8, 8); break;
    case 16: MBD_GATHER_P(16, 16); break;
    case 32: if (sliced) MBD_GATHER_P(32, 16) else MBD_GATHER_P(32, 32) break;
    case 64: if (sliced) MBD_GATHER_P(64, 16) else MBD_GATHER_P(64, 64) break;
  }
#undef MBD_GATHER_P
#undef MBD_GATHER
}

// With w, also the gather of the matvec of w over the same grid (into Lt; no dot products).
template <typename R>
void launch_spme_force(const Geometry& geo, const SysBuffers& b, const void* h, int B, int BG,
                       int chunk0, hipStream_t st, const double* hscale, const double* w) {
  const size_t chunk = (size_t)geo.K[2] * geo.K[1] * (geo.K[0] + 2) * BG;
  dim3 grd(gather_blocks(geo, BG), 1);
  const Epilogue<R> ep = epilogue_of<R>(geo, b, w, B, MBD_C_ALL);
#define MBD_SF(PP, BB, EE)                                                                 \
  k_spme_force<R, PP, BB, EE><<<grd, 64 * gather_waves(geo), 0, st>>>(                     \
      geo, b.base, (const R*)b.th, (const R*)b.dth, (const R*)b.ddth, (const R*)b.grid,    \
      chunk, (const R*)h, B, chunk0, b.fsum, hscale, ep)
#define MBD_SF_E(PP, BB) if (w) MBD_SF(PP, BB, true); else MBD_SF(PP, BB, false)
#define MBD_SF_P(BB)                   \
  switch (geo.p) {                     \
    case 4: MBD_SF_E(4, BB); break;    \
    case 6: MBD_SF_E(6, BB); break;    \
    case 8: MBD_SF_E(8, BB); break;    \
  }
  switch (BG) {
    case 1: MBD_SF_P(1); break;
    case 2: MBD_SF_P(2); break;
    case 4: MBD_SF_P(4); break;
    case 8: MBD_SF_P(8); break;
    case 16: MBD_SF_P(16); break;
    case 32: MBD_SF_P(32); break;
    case 64: MBD_SF_P(64); break;
  }
#undef MBD_SF_E
#undef MBD_SF_P
#undef MBD_SF
}

template void launch_spme_force<float>(const Geometry&, const SysBuffers&, const void*, int, int,
                                       int, hipStream_t, const double*, const double*);
template void launch_spme_force<double>(const Geometry&, const SysBuffers&, const void*, int,
                                        int, int, hipStream_t, const double*, const double*);

template void launch_spread<float>(const Geometry&, const SysBuffers&, int, int, int, int,
                                   hipStream_t);
template void launch_spread<double>(const Geometry&, const SysBuffers&, int, int, int, int,
                                    hipStream_t);
template void launch_epilogue<float>(const Geometry&, const SysBuffers&, const double*, int, int,
                                     int, int, uint32_t, hipStream_t);
template void launch_epilogue<double>(const Geometry&, const SysBuffers&, const double*, int, int,
                                      int, int, uint32_t, hipStream_t);

}  // namespace mbd
