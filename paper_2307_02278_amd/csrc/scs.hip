// Range-separated self-consistent screening of the polarizabilities on the GPU.
//
// For every imaginary frequency u_q the Dyson-like screening equation (Review
// section; MBD@rsSCS) is solved matrix-free:
//   (A(iu)^-1 + T_SR(iu)) X = E,   E = three right-hand sides, E_k = unit vector k on every atom,
//   alpha_i(iu) = alpha_i / (1 + (u / omega_i)^2),
//   T_SR = (1 - f) T_GG,  T_GG = -grad grad (erf(r / sigma_ij) / r) = A I - B r r^T,
//   A = (erf z - c) / r^3,  B = (3 erf z - c (3 + 2 z^2)) / r^5,  z = r / sigma_ij,
//   c = (2 / sqrt pi) z exp(-z^2),  sigma_ij^2 = sigma_i^2 + sigma_j^2,
//   sigma_i = (sqrt(2 / pi) alpha_i(iu) / 3)^(1/3),
// with f the Fermi damping of the MBD step, summed over every periodic image within
// the plan's pair cutoff. Then alpha^SCS_i(iu) = (1/3) sum_k X_{i,k}(E_k).
//
// All right-hand sides (3 per frequency, "columns") run together through a
// Jacobi-preconditioned conjugate gradient in float64. Vectors are [n][3][ncol]
// over the plan's sorted atoms, column = 3 q + k.
#include <hip/hip_runtime.h>

#include <cmath>

#include "cells.h"
#include "common.h"
#include "mbd_math.h"

namespace mbd {
namespace {

// 1 - f = 1 / (1 + e^z) is below 1e-16 for z > 36.8: such pairs add nothing in float64
constexpr double kDampSkip = 36.8;

// CG scalar rows of ScsWork::sc ([kScsRows][ncol])
enum { kRz = 0, kPq = 1, kAlpha = 2, kBeta = 3, kRr = 4, kActive = 5, kBb = 6, kScsRows = 8 };

// Sorted cell-local positions in float64 (the same frame as the pair kernels:
// position minus the corner of its cell), the damping radius beta R_vdW, and per
// (atom, frequency) 1 / alpha(iu) and sigma(u)^2.
__global__ void k_scs_prepare(const Geometry geo, const int* __restrict__ perm,
                              const int* __restrict__ scell, const double* __restrict__ wpos,
                              const double* __restrict__ alpha, const double* __restrict__ omega,
                              const double* __restrict__ rvdw, const double* __restrict__ u,
                              int nq, double* __restrict__ locd, double* __restrict__ ainv,
                              double* __restrict__ sig2) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= geo.n) return;
  const int i = perm[s];
  int c[3];
  cell_coords(scell[s], c[0], c[1], c[2]);
  double lf[3];
  for (int a = 0; a < 3; ++a) lf[a] = wpos[3 * i + a] - (double)c[a] / geo.nc[a];
  for (int k = 0; k < 3; ++k)
    locd[4 * s + k] = lf[0] * geo.A[0][k] + lf[1] * geo.A[1][k] + lf[2] * geo.A[2][k];
  locd[4 * s + 3] = geo.beta * rvdw[i];
  const double al = alpha[i], om = omega[i];
  for (int q = 0; q < nq; ++q) {
    const double x = u[q] / om;
    const double au = al / (1.0 + x * x);
    ainv[(size_t)s * nq + q] = 1.0 / au;
    const double sg = cbrt(0.7978845608028654 * au / 3.0);  // sqrt(2 / pi) alpha / 3
    sig2[(size_t)s * nq + q] = sg * sg;
  }
}

// A pair of the screening operator, prepared once for all frequencies: r = R_j + n - R_i,
// a0 = (1 - f) / r^3, b0 = 3 (1 - f) / r^5 and r^2.
struct ScsPair {
  double rx, ry, rz, a0, b0, r2;
};
constexpr int kScsQueue = 96;  // pairs a wavefront queues; it flushes above 96 - 64

// q = A^-1 p + T_SR p. One wavefront per sorted target. The candidates of the cells around
// it are tested 64 at a time (their cells' atom counts prefix-summed), and the geometry and
// the damping of a pair in range are evaluated by its one lane, into one of two queues in
// LDS: near, where the Gaussian clouds overlap at some frequency (r < 7 sigma at u = 0, the
// widest), and far, where T_GG is the bare tensor to the last bit. The queues are flushed
// with lane = f + NQP sl: frequency f of the pairs sl, sl + SL, ... (SL = 64 / NQP lanes
// share a frequency), so every lane works, erf and exp run for near pairs only, and the SL
// partial fields are summed with cross-lane exchanges. The order is fixed by the cells.
// With every lane of a frequency walking the cells and evaluating the damping itself this
// took 315 us for 3000 atoms and 16 frequencies, 106 us here.
template <int NQP>
__global__ void __launch_bounds__(64)
k_scs_apply(const Geometry geo, const int* __restrict__ cell_start,
            const int* __restrict__ scell, const double* __restrict__ locd,
            const double* __restrict__ ainv, const double* __restrict__ sig2, int nq,
            const double* __restrict__ p, double* __restrict__ qv) {
  constexpr int SL = 64 / NQP;
  __shared__ ScsPair queue[2][kScsQueue];  // near, far
  __shared__ int qj[2][kScsQueue];
  __shared__ int pre[65], first[64];
  __shared__ double shift[3][64];
  const int s = blockIdx.x;
  const int lane = threadIdx.x;
  const int f = lane % NQP, sl = lane / NQP;
  const bool fv = f < nq;
  const int fq = fv ? f : 0;
  const int ncol = 3 * nq;
  int cx, cy, cz;
  cell_coords(scell[s], cx, cy, cz);
  const double xi = locd[4 * s], yi = locd[4 * s + 1], zi = locd[4 * s + 2];
  const double Si = locd[4 * s + 3];
  const double s2i = sig2[(size_t)s * nq + fq], s2i0 = sig2[(size_t)s * nq];
  const double rp2 = geo.r_pair * geo.r_pair;
  const double dd = geo.damp_d;
  const int ncells = scan_cells(geo);
  double acc[3][3];
#pragma unroll
  for (int a = 0; a < 3; ++a) acc[a][0] = acc[a][1] = acc[a][2] = 0.0;
  auto wave_sync = [] {  // LDS writes of other lanes are visible past this point
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  auto add = [&](const ScsPair& t, int j, double A, double Bk) {
    const double* pj = p + (size_t)j * 3 * ncol + 3 * fq;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const double x0 = pj[k], x1 = pj[ncol + k], x2 = pj[2 * ncol + k];
      const double rd = Bk * (t.rx * x0 + t.ry * x1 + t.rz * x2);
      acc[0][k] += A * x0 - t.rx * rd;
      acc[1][k] += A * x1 - t.ry * rd;
      acc[2][k] += A * x2 - t.rz * rd;
    }
  };
  int cnt[2] = {0, 0};  // queued pairs (wave-uniform)
  auto flush_near = [&] {
    for (int e = sl; e < cnt[0]; e += SL) {
      const ScsPair t = queue[0][e];
      const int j = qj[0][e];
      double A = t.a0, Bk = t.b0;
      scs_overlap(t.r2, s2i + sig2[(size_t)j * nq + fq], A, Bk);
      add(t, j, A, Bk);
    }
    cnt[0] = 0;
  };
  auto flush_far = [&] {
#pragma unroll 2
    for (int e = sl; e < cnt[1]; e += SL) {
      const ScsPair t = queue[1][e];
      add(t, qj[1][e], t.a0, t.b0);
    }
    cnt[1] = 0;
  };
  for (int cc0 = 0; cc0 < ncells; cc0 += 64) {
    int nat = 0;
    if (cc0 + lane < ncells) {
      CellOffset o;
      const int cc = scan_cell(geo, cx, cy, cz, cc0 + lane, o);
      first[lane] = cell_start[cc];
      nat = cell_start[cc + 1] - cell_start[cc];
      cell_shift<double>(geo, o, shift[0][lane], shift[1][lane], shift[2][lane]);
    }
    int v = nat;
    for (int o = 1; o < 64; o <<= 1) {
      const int u = __shfl_up(v, o);
      if (lane >= o) v += u;
    }
    pre[lane + 1] = v;
    if (lane == 0) pre[0] = 0;
    const int total = __shfl(v, 63);
    wave_sync();
    for (int r0 = 0; r0 < total; r0 += 64) {
      const int c = r0 + lane;
      bool hit = false, near = false;
      int j = 0;
      ScsPair t = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
      if (c < total) {
        int lo = 0, hi = 63;  // the cell of candidate c: largest k with pre[k] <= c
        while (lo < hi) {
          const int mid = (lo + hi + 1) >> 1;
          if (pre[mid] <= c) lo = mid; else hi = mid - 1;
        }
        j = first[lo] + (c - pre[lo]);
        t.rx = locd[4 * (size_t)j] - xi + shift[0][lo];
        t.ry = locd[4 * (size_t)j + 1] - yi + shift[1][lo];
        t.rz = locd[4 * (size_t)j + 2] - zi + shift[2][lo];
        t.r2 = t.rx * t.rx + t.ry * t.ry + t.rz * t.rz;
        if (t.r2 < rp2 && !(j == s && cc0 + lo == ncells / 2)) {
          hit = !(scs_damped(t.r2, Si + locd[4 * (size_t)j + 3], dd, t.a0, t.b0) > kDampSkip);
          near = t.r2 < 49.0 * (s2i0 + sig2[(size_t)j * nq]);
        }
      }
#pragma unroll
      for (int w = 0; w < 2; ++w) {
        const bool mine = hit && near == (w == 0);
        const unsigned long long bal = __ballot(mine);
        const int slot = cnt[w] + (int)__builtin_amdgcn_mbcnt_hi(
                                      (unsigned)(bal >> 32),
                                      __builtin_amdgcn_mbcnt_lo((unsigned)bal, 0u));
        if (mine) {
          queue[w][slot] = t;
          qj[w][slot] = j;
        }
        cnt[w] += __popcll(bal);
      }
      wave_sync();
      if (cnt[0] > kScsQueue - 64) flush_near();
      if (cnt[1] > kScsQueue - 64) flush_far();
      wave_sync();  // the queues' entries have been read
    }
    wave_sync();  // the next chunk's tables overwrite this one's
  }
  flush_near();
  flush_far();
#pragma unroll
  for (int off = NQP; off < 64; off <<= 1)
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int k = 0; k < 3; ++k) acc[a][k] += __shfl_xor(acc[a][k], off);
  if (sl == 0 && fv) {
    const double ai = ainv[(size_t)s * nq + f];
    const size_t o = (size_t)s * 3 * ncol + 3 * f;
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int k = 0; k < 3; ++k)
        qv[o + (size_t)a * ncol + k] = ai * p[o + (size_t)a * ncol + k] + acc[a][k];
  }
}

// Partial sums over blocks of rows: part[b][0][c] = sum_r X[r][c] Y[r][c] and, when X2
// is given, part[b][1][c] = sum_r X2[r][c] Y2[r][c]. Thread t takes column t % ncol and
// every (256 / ncol)-th row of the block's range; the lanes of a column are summed in
// a fixed order, so results do not depend on scheduling.
__global__ void __launch_bounds__(256)
k_col_dots(const double* __restrict__ X, const double* __restrict__ Y,
           const double* __restrict__ X2, const double* __restrict__ Y2, int rows, int ncol,
           int rows_per_block, double* __restrict__ part) {
  __shared__ double s1[256], s2[256];
  const int t = threadIdx.x;
  const int nrl = 256 / ncol;
  const int c = t % ncol, rl = t / ncol;
  const int r0 = blockIdx.x * rows_per_block;
  const int r1 = min(rows, r0 + rows_per_block);
  double a1 = 0.0, a2 = 0.0;
  if (rl < nrl) {
    for (int r = r0 + rl; r < r1; r += nrl) {
      const size_t o = (size_t)r * ncol + c;
      a1 += X[o] * Y[o];
      if (X2) a2 += X2[o] * Y2[o];
    }
  }
  s1[t] = a1;
  s2[t] = a2;
  __syncthreads();
  if (t < ncol) {
    double b1 = 0.0, b2 = 0.0;
    for (int i = 0; i < nrl; ++i) {
      b1 += s1[t + i * ncol];
      b2 += s2[t + i * ncol];
    }
    part[((size_t)blockIdx.x * 2) * ncol + t] = b1;
    part[((size_t)blockIdx.x * 2 + 1) * ncol + t] = b2;
  }
}

// x = 0, r = E, z = P r, p = z (P = diag alpha(iu), the Jacobi preconditioner).
__global__ void k_scs_init(int n, int nq, const double* __restrict__ ainv, double* __restrict__ x,
                           double* __restrict__ r, double* __restrict__ z,
                           double* __restrict__ p) {
  const int ncol = 3 * nq;
  const size_t total = (size_t)n * 3 * ncol;
  for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < total;
       e += (size_t)gridDim.x * blockDim.x) {
    const int col = (int)(e % ncol);
    const int a = (int)((e / ncol) % 3);
    const size_t s = e / (3 * (size_t)ncol);
    const int f = col / 3, k = col % 3;
    const double rv = (a == k) ? 1.0 : 0.0;
    const double zv = rv / ainv[s * nq + f];
    x[e] = 0.0;
    r[e] = rv;
    z[e] = zv;
    p[e] = zv;
  }
}

// Sums v1, v2 over the nblk row blocks of part[b][0][c] and part[b][1][c] (256 threads, one
// column): a fixed strided split and a fixed tree, so the order never changes. Thread 0
// holds the result.
__device__ __forceinline__ void col_sums(const double* __restrict__ part, int nblk, int ncol,
                                         int c, double& v1, double& v2) {
  __shared__ double r1[256], r2[256];
  const int t = threadIdx.x;
  v1 = v2 = 0.0;
  for (int b = t; b < nblk; b += 256) {
    v1 += part[((size_t)b * 2) * ncol + c];
    v2 += part[((size_t)b * 2 + 1) * ncol + c];
  }
  r1[t] = v1;
  r2[t] = v2;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (t < h) {
      r1[t] += r1[t + h];
      r2[t] += r2[t + h];
    }
    __syncthreads();
  }
  v1 = r1[0];
  v2 = r2[0];
}

// After the initial dots (r.z, r.r): rz, bb = ||E_k||^2, every column active.
__global__ void __launch_bounds__(256)
k_scs_start(const double* __restrict__ part, int nblk, int ncol, double* __restrict__ sc,
            int* __restrict__ nact) {
  const int c = blockIdx.x;
  double rz, rr;
  col_sums(part, nblk, ncol, c, rz, rr);
  if (threadIdx.x != 0) return;
  sc[kRz * ncol + c] = rz;
  sc[kRr * ncol + c] = rr;
  sc[kBb * ncol + c] = rr;
  sc[kActive * ncol + c] = 1.0;
  sc[kAlpha * ncol + c] = 0.0;
  sc[kBeta * ncol + c] = 0.0;
  if (c == 0) nact[0] = ncol;
}

// alpha_c = rz_c / (p.q)_c for active columns; p.q <= 0 (or not finite) means the
// screening matrix is not positive definite: the column stops and the status is set.
__global__ void __launch_bounds__(256)
k_scs_alpha(const double* __restrict__ part, int nblk, int ncol, double* __restrict__ sc,
            int* __restrict__ nact, uint32_t* __restrict__ status) {
  const int c = blockIdx.x;
  double pq, unused;
  col_sums(part, nblk, ncol, c, pq, unused);
  if (threadIdx.x != 0) return;
  double al = 0.0;
  if (sc[kActive * ncol + c] != 0.0) {
    if (!(pq > 0.0) || !isfinite(pq)) {
      sc[kActive * ncol + c] = 0.0;
      atomicOr(status, kErrNotPosdef);
    } else {
      al = sc[kRz * ncol + c] / pq;
    }
  }
  sc[kAlpha * ncol + c] = al;
  if (c == 0) nact[0] = 0;  // counted again by k_scs_beta
}

// x += alpha p, r -= alpha q, z = P r, and the partial sums of r.z and r.r by row blocks as
// in k_col_dots.
__global__ void __launch_bounds__(256)
k_scs_update(int nq, int rows, int rows_per_block, const double* __restrict__ ainv,
             const double* __restrict__ sc, const double* __restrict__ p,
             const double* __restrict__ qv, double* __restrict__ x, double* __restrict__ r,
             double* __restrict__ z, double* __restrict__ part) {
  __shared__ double s1[256], s2[256];
  const int ncol = 3 * nq;
  const int t = threadIdx.x;
  const int nrl = 256 / ncol;
  const int c = t % ncol, rl = t / ncol;
  const int r0 = blockIdx.x * rows_per_block;
  const int r1 = min(rows, r0 + rows_per_block);
  double a1 = 0.0, a2 = 0.0;
  if (rl < nrl) {
    const double al = sc[kAlpha * ncol + c];
    for (int i = r0 + rl; i < r1; i += nrl) {
      const size_t e = (size_t)i * ncol + c;
      x[e] += al * p[e];
      const double rv = r[e] - al * qv[e];
      r[e] = rv;
      const double zv = rv / ainv[(size_t)(i / 3) * nq + c / 3];
      z[e] = zv;
      a1 += rv * zv;
      a2 += rv * rv;
    }
  }
  s1[t] = a1;
  s2[t] = a2;
  __syncthreads();
  if (t < ncol) {
    double b1 = 0.0, b2 = 0.0;
    for (int i = 0; i < nrl; ++i) {
      b1 += s1[t + i * ncol];
      b2 += s2[t + i * ncol];
    }
    part[((size_t)blockIdx.x * 2) * ncol + t] = b1;
    part[((size_t)blockIdx.x * 2 + 1) * ncol + t] = b2;
  }
}

// beta_c = (r.z)_new / (r.z)_old; a column whose ||r|| <= tol ||E_k|| stops.
__global__ void __launch_bounds__(256)
k_scs_beta(const double* __restrict__ part, int nblk, int ncol, double tol2,
           double* __restrict__ sc, int* __restrict__ nact) {
  const int c = blockIdx.x;
  double rz, rr;
  col_sums(part, nblk, ncol, c, rz, rr);
  if (threadIdx.x != 0) return;
  double be = 0.0;
  if (sc[kActive * ncol + c] != 0.0) {
    sc[kRr * ncol + c] = rr;
    if (!isfinite(rr) || rr <= tol2 * sc[kBb * ncol + c]) {
      sc[kActive * ncol + c] = 0.0;
    } else {
      be = rz / sc[kRz * ncol + c];
      sc[kRz * ncol + c] = rz;
      atomicAdd(nact, 1);
    }
  }
  sc[kBeta * ncol + c] = be;
}

// p = z + beta p.
__global__ void k_scs_direction(size_t total, int ncol, const double* __restrict__ sc,
                                const double* __restrict__ z, double* __restrict__ p) {
  for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < total;
       e += (size_t)gridDim.x * blockDim.x)
    p[e] = z[e] + sc[kBeta * ncol + (int)(e % ncol)] * p[e];
}

// alpha^SCS_i(iu_q) = (1/3) sum_k x[i][k][3q + k]; C6 by the quadrature weights w
// (node 0 is the static point u = 0 and carries no weight); omega^SCS, R^SCS.
// Outputs in the caller's atom order.
__global__ void k_scs_output(int n, int nq, const int* __restrict__ perm,
                             const double* __restrict__ x, const double* __restrict__ w,
                             const double* __restrict__ alpha, const double* __restrict__ rvdw,
                             double* __restrict__ a_out, double* __restrict__ om_out,
                             double* __restrict__ rv_out, double* __restrict__ af_out) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n) return;
  const int i = perm[s];
  const int ncol = 3 * nq;
  const double* xs = x + (size_t)s * 3 * ncol;
  double a0 = 0.0, c6 = 0.0;
  for (int f = 0; f < nq; ++f) {
    const double af = (xs[3 * f] + xs[ncol + 3 * f + 1] + xs[2 * ncol + 3 * f + 2]) / 3.0;
    if (f == 0) a0 = af;
    else {
      c6 += w[f] * af * af;
      if (af_out) af_out[(size_t)(f - 1) * n + i] = af;
    }
  }
  c6 *= 3.0 / M_PI;
  a_out[i] = a0;
  om_out[i] = 4.0 * c6 / (3.0 * a0 * a0);
  rv_out[i] = rvdw[i] * cbrt(a0 / alpha[i]);
}

int grid_for(size_t total) {
  return (int)std::min<size_t>((total + 255) / 256, 4096);
}

}  // namespace

void launch_scs_prepare(const Geometry& g, const SysBuffers& b, const double* alpha,
                        const double* omega, const double* rvdw, const double* u,
                        const ScsWork& w, hipStream_t st) {
  k_scs_prepare<<<(g.n + 127) / 128, 128, 0, st>>>(g, b.perm, b.scell, b.wpos, alpha, omega,
                                                   rvdw, u, w.nq, w.locd, w.ainv, w.sig2);
}

void launch_scs_apply(const Geometry& g, const SysBuffers& b, const ScsWork& w, const double* p,
                      double* q, hipStream_t st) {
#define MBD_SCS(NQP)                                                                           \
  k_scs_apply<NQP><<<g.n, 64, 0, st>>>(g, b.cell_start, b.scell, w.locd, w.ainv, w.sig2, w.nq, \
                                       p, q)
  if (w.nq <= 2) MBD_SCS(2);
  else if (w.nq <= 4) MBD_SCS(4);
  else if (w.nq <= 8) MBD_SCS(8);
  else if (w.nq <= 16) MBD_SCS(16);
  else MBD_SCS(32);
#undef MBD_SCS
}

void launch_scs_dots(const ScsWork& w, const double* X, const double* Y, const double* X2,
                     const double* Y2, hipStream_t st) {
  const int rows = 3 * w.n;
  const int per = (rows + w.nblk - 1) / w.nblk;
  k_col_dots<<<w.nblk, 256, 0, st>>>(X, Y, X2, Y2, rows, w.ncol, per, w.part);
}

void launch_scs_init(const ScsWork& w, hipStream_t st) {
  const size_t total = (size_t)w.n * 3 * w.ncol;
  k_scs_init<<<grid_for(total), 256, 0, st>>>(w.n, w.nq, w.ainv, w.x, w.r, w.z, w.p);
  launch_scs_dots(w, w.r, w.z, w.r, w.r, st);
  k_scs_start<<<w.ncol, 256, 0, st>>>(w.part, w.nblk, w.ncol, w.sc, w.nact);
}

void launch_scs_iteration(const Geometry& g, const SysBuffers& b, const ScsWork& w, double tol,
                          uint32_t* status, hipStream_t st) {
  const size_t total = (size_t)w.n * 3 * w.ncol;
  const int rows = 3 * w.n;
  launch_scs_apply(g, b, w, w.p, w.q, st);
  launch_scs_dots(w, w.p, w.q, nullptr, nullptr, st);
  k_scs_alpha<<<w.ncol, 256, 0, st>>>(w.part, w.nblk, w.ncol, w.sc, w.nact, status);
  k_scs_update<<<w.nblk, 256, 0, st>>>(w.nq, rows, (rows + w.nblk - 1) / w.nblk, w.ainv, w.sc,
                                       w.p, w.q, w.x, w.r, w.z, w.part);
  k_scs_beta<<<w.ncol, 256, 0, st>>>(w.part, w.nblk, w.ncol, tol * tol, w.sc, w.nact);
  k_scs_direction<<<grid_for(total), 256, 0, st>>>(total, w.ncol, w.sc, w.z, w.p);
}

void launch_scs_output(const SysBuffers& b, const ScsWork& w, const double* wq,
                       const double* alpha, const double* rvdw, double* a_out, double* om_out,
                       double* rv_out, double* af_out, hipStream_t st) {
  k_scs_output<<<(w.n + 127) / 128, 128, 0, st>>>(w.n, w.nq, b.perm, w.x, wq, alpha, rvdw,
                                                  a_out, om_out, rv_out, af_out);
}

}  // namespace mbd
