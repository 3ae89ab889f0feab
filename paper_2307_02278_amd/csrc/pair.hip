// Direct-space Ewald field with the damping correction (eq. fld_ewald):
//   E_dir,i = sum over images n and atoms j with |R_j + n - R_i| < r_pair,
//             except (j = i, n = 0), of T_dir(R_j + n - R_i) d_j,
//   T_dir = T_erfc - (1 - f_ij) T = A(r) I - B(r) r r^T.
// Cell list: atoms sorted by cell (slices of the fractional coordinates, width
// >= r_pair / 2 perpendicular to the faces); the neighbour cells of a cell are the
// offsets o in [-nr, nr]^3, wrapped periodically, and the displacement is
// r = loc_j - loc_i + sum_a o_a h_a with cell-local Cartesian coordinates and the
// cell shift vectors h_a = a_a / nc_a, so it stays accurate in single precision,
// works for any cell shape and covers several images when r_pair exceeds half the box.
//
// Which kernel runs:
//  - B <= 8: a neighbour list. Per target the sources within r_pair with A and B of their
//    tensors (k_nbr_build, once per device setup), applied by one to four wavefronts per
//    target (k_pair_nbr), or the same sum over the cells where there is no list;
//  - B >= 16: a tensor list. The positions do not change during a Lanczos run, so the
//    tensors are evaluated once per device setup (k_pair_build) and kept in device memory,
//    grouped by 16 consecutive sorted target atoms: for every source image within r_pair of
//    at least one target of the group, a header (source index, 16-bit mask of the targets
//    within range) and the six components of T_dir for each target (zeros outside the mask).
//    float64 and float blocks of 16 and 32 multiply it on the matrix cores of their own type
//    (k_pair_mfma), float blocks of 64 and more on the bfloat16 ones in three planes
//    (k_pair_split, pair_mode 1 and 2) or with one vector lane per right-hand side
//    (k_pair_list, pair_mode 0).
#include <algorithm>

#include "cells.h"
#include "common.h"
#include "launch_rules.h"
#include "mbd_math.h"
#include "mfma.h"

namespace mbd {

namespace {

// ---------------------------------------------------------------------------
// Neighbour list of the narrow blocks (B <= 8): build (once per device setup), apply.
// ---------------------------------------------------------------------------

template <typename R>
struct alignas(2 * sizeof(R)) NbrAB {
  R A, B;
};

// One wavefront per target. The cells around it are taken 64 at a time, their atom counts
// prefix-summed, and every lane tests one candidate of a 64-candidate round; the hits are
// appended in scan order (source atom, packed cell offset), and A and B of T_dir are then
// evaluated one lane per kept pair, so no lane of the erfc and exp evaluation idles on a
// candidate out of range (about 3 of 4 are). Every pair is counted, at most cap are kept;
// with cap == 0 only the counts are produced.
template <typename R>
__global__ void __launch_bounds__(256)
k_nbr_build(const Geometry geo, const int* __restrict__ cell_start,
            const int* __restrict__ scell, const R* __restrict__ loc, int cap,
            int2* __restrict__ hdr, NbrAB<R>* __restrict__ ab, int* __restrict__ count,
            int* __restrict__ maxcount) {
  __shared__ int pre_all[4][65], first_all[4][64], off_all[4][64];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int* pre = pre_all[wave];
  int* first = first_all[wave];
  int* offs = off_all[wave];
  const int s = blockIdx.x * 4 + wave;
  if (s >= geo.n) return;  // the wavefronts are independent: no barrier below
  int cx, cy, cz;
  cell_coords(scell[s], cx, cy, cz);
  const R xi = loc[4 * (size_t)s], yi = loc[4 * (size_t)s + 1], zi = loc[4 * (size_t)s + 2],
          si = loc[4 * (size_t)s + 3];
  const R rp2 = (R)(geo.r_pair * geo.r_pair);
  const int ncells = scan_cells(geo);
  const int home = pack_off({0, 0, 0});
  int2* H = hdr + (size_t)s * cap;
  int cnt = 0;
  for (int cc0 = 0; cc0 < ncells; cc0 += 64) {
    int nat = 0;
    if (cc0 + lane < ncells) {
      CellOffset o;
      const int cc = scan_cell(geo, cx, cy, cz, cc0 + lane, o);
      first[lane] = cell_start[cc];
      nat = cell_start[cc + 1] - cell_start[cc];
      offs[lane] = pack_off(o);
    }
    int v = nat;
    for (int o = 1; o < 64; o <<= 1) {
      const int u = __shfl_up(v, o);
      if (lane >= o) v += u;
    }
    pre[lane + 1] = v;
    if (lane == 0) pre[0] = 0;
    const int total = __shfl(v, 63);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    for (int r0 = 0; r0 < total; r0 += 64) {
      const int c = r0 + lane;
      bool hit = false;
      int j = 0, off = home;
      if (c < total) {
        int lo = 0, hi = 63;  // the cell of candidate c: largest k with pre[k] <= c
        while (lo < hi) {
          const int mid = (lo + hi + 1) >> 1;
          if (pre[mid] <= c) lo = mid; else hi = mid - 1;
        }
        j = first[lo] + (c - pre[lo]);
        off = offs[lo];
        R sx, sy, sz;
        cell_shift<R>(geo, unpack_off(off), sx, sy, sz);
        const R rx = loc[4 * (size_t)j] - xi + sx;
        const R ry = loc[4 * (size_t)j + 1] - yi + sy;
        const R rz = loc[4 * (size_t)j + 2] - zi + sz;
        hit = rx * rx + ry * ry + rz * rz < rp2 && !(j == s && off == home);
      }
      const unsigned long long bal = __ballot(hit);
      const int slot = cnt + (int)__builtin_amdgcn_mbcnt_hi(
                                 (unsigned)(bal >> 32),
                                 __builtin_amdgcn_mbcnt_lo((unsigned)bal, 0u));
      if (hit && slot < cap) H[slot] = make_int2(j, off);
      cnt += __popcll(bal);
    }
    // the next chunk's tables overwrite this one's
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  // (the fence above also made the headers of other lanes visible to this one)
  const R tau = (R)geo.tau, dd = (R)geo.damp_d;
  const int kept = min(cnt, cap);
  for (int k = lane; k < kept; k += 64) {
    const int2 h = H[k];
    R sx, sy, sz;
    cell_shift<R>(geo, unpack_off(h.y), sx, sy, sz);
    const R* lj = loc + 4 * (size_t)h.x;
    const R rx = lj[0] - xi + sx, ry = lj[1] - yi + sy, rz = lj[2] - zi + sz;
    NbrAB<R> t;
    direct_kernel<R>(rx * rx + ry * ry + rz * rz, tau, R(1) / (lj[3] + si), dd, t.A, t.B);
    ab[(size_t)s * cap + k] = t;
  }
  if (lane == 0) {
    count[s] = cnt;
    if (maxcount) atomicMax(maxcount, cnt);
  }
}

// E_dir of B = NB <= 8 right-hand sides: WV wavefronts per target, lane = right-hand side
// + NB x list entry, so a wavefront takes 64 / NB neighbours at a time and the partial
// fields are added across lanes (then across the WV wavefronts, in LDS) in a fixed order.
// One thread per target instead runs one serial chain of several hundred loads per thread
// and re-evaluates erfc and exp for every candidate in every matvec.
// A target with more pairs than the list holds (positions far denser than those the plan
// was sized for, a list too large to keep, or a scan too wide for its packed offsets) is
// summed on the fly over the cells.
template <typename R, int NB, int WV>
__global__ void __launch_bounds__(256)
k_pair_nbr(const Geometry geo, const int* __restrict__ cell_start,
           const int* __restrict__ scell, const R* __restrict__ loc, int cap,
           const int* __restrict__ count, const int2* __restrict__ hdr,
           const NbrAB<R>* __restrict__ ab, const R* __restrict__ dv, R* __restrict__ Ed) {
  constexpr int TPB = 4 / WV;    // targets per work-group
  constexpr int EW = 64 / NB;    // entries per wavefront and step
  constexpr int EL = EW * WV;    // entries per target and step
  __shared__ R red[WV > 1 ? 4 * NB * 3 : 1];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int b = lane % NB, e = lane / NB + (wave % WV) * EW;
  // each XCD takes a contiguous range of sorted targets (gridDim.x is a multiple of 8):
  // their sources' positions and dipoles stay in its L2
  const int blk = (blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
  const int s = blk * TPB + wave / WV;
  if (s >= geo.n) return;  // WV > 1: uniform over the work-group
  const R xi = loc[4 * (size_t)s], yi = loc[4 * (size_t)s + 1], zi = loc[4 * (size_t)s + 2];
  R e0 = R(0), e1 = R(0), e2 = R(0);
  auto add = [&](int j, R rx, R ry, R rz, R A, R Bk) {
    const R* d = dv + (size_t)j * 3 * NB + b;
    const R d0 = d[0], d1 = d[NB], d2 = d[2 * NB];
    const R rd = Bk * (rx * d0 + ry * d1 + rz * d2);
    e0 += A * d0 - rx * rd;
    e1 += A * d1 - ry * rd;
    e2 += A * d2 - rz * rd;
  };
  const int cnt = count[s];
  if (cap > 0 && cnt <= cap) {
    const int2* H = hdr + (size_t)s * cap;
    const NbrAB<R>* T = ab + (size_t)s * cap;
#pragma unroll 2
    for (int k = e; k < cnt; k += EL) {
      const int2 h = H[k];
      const NbrAB<R> t = T[k];
      R sx, sy, sz;
      cell_shift<R>(geo, unpack_off(h.y), sx, sy, sz);
      const R* lj = loc + 4 * (size_t)h.x;
      add(h.x, lj[0] - xi + sx, lj[1] - yi + sy, lj[2] - zi + sz, t.A, t.B);
    }
  } else {
    const R si = loc[4 * (size_t)s + 3], tau = (R)geo.tau, dd = (R)geo.damp_d;
    const R rp2 = (R)(geo.r_pair * geo.r_pair);
    const int ncells = scan_cells(geo);
    int cx, cy, cz;
    cell_coords(scell[s], cx, cy, cz);
    for (int ci = 0; ci < ncells; ++ci) {
      CellOffset o;
      const int cc = scan_cell(geo, cx, cy, cz, ci, o);
      R sx, sy, sz;
      cell_shift<R>(geo, o, sx, sy, sz);
      const int j1 = cell_start[cc + 1];
      for (int j = cell_start[cc] + e; j < j1; j += EL) {
        const R* lj = loc + 4 * (size_t)j;
        const R rx = lj[0] - xi + sx, ry = lj[1] - yi + sy, rz = lj[2] - zi + sz;
        const R r2 = rx * rx + ry * ry + rz * rz;
        if (r2 >= rp2 || (j == s && ci == ncells / 2)) continue;
        R A, Bk;
        direct_kernel<R>(r2, tau, R(1) / (lj[3] + si), dd, A, Bk);
        add(j, rx, ry, rz, A, Bk);
      }
    }
  }
#pragma unroll
  for (int o = NB; o < 64; o <<= 1) {
    e0 += __shfl_xor(e0, o);
    e1 += __shfl_xor(e1, o);
    e2 += __shfl_xor(e2, o);
  }
  R* out = Ed + (size_t)s * 3 * NB;
  if constexpr (WV == 1) {
    if (lane < NB) {
      out[b] = e0;
      out[NB + b] = e1;
      out[2 * NB + b] = e2;
    }
  } else {
    if (lane < NB) {
      red[(wave * 3 + 0) * NB + b] = e0;
      red[(wave * 3 + 1) * NB + b] = e1;
      red[(wave * 3 + 2) * NB + b] = e2;
    }
    __syncthreads();
    if (threadIdx.x < 3 * NB) {
      R v = red[threadIdx.x];
#pragma unroll
      for (int w = 1; w < 4; ++w) v += red[w * 3 * NB + threadIdx.x];
      out[threadIdx.x] = v;
    }
  }
}


// ---------------------------------------------------------------------------
// Tensor list: build (once per device setup) and apply (every matvec).
// ---------------------------------------------------------------------------

// One work-group (BT threads) per group of kGroup consecutive sorted targets.
// Candidate sources are the atoms of the cells around the group whose distance to
// the group's bounding box is below r_pair; those within r_pair of at least one
// target are appended with their tensors, in the order of the cell scan (z, y, x,
// then atom index). The cells are taken in chunks: their atom counts are prefix-summed
// in LDS, every thread tests one candidate of a BT-candidate round, the hits are
// compacted in order (wavefront ballots plus a prefix over the wavefronts), and
// the tensors of a round are then written with one thread per (candidate, target)
// pair, so that consecutive threads store consecutive tensor words. With cap == 0
// only the counts are produced (plan sizing).
constexpr int kBuildCells = 256;  // cells per chunk of the scan
template <typename R, int BT>
__global__ void __launch_bounds__(BT)
k_pair_build(const Geometry geo, const int* __restrict__ cell_start,
             const int* __restrict__ scell, const R* __restrict__ loc, int cap,
             int2* __restrict__ hdr, R* __restrict__ Tg, R* __restrict__ Fg,
             int* __restrict__ gcount, int* __restrict__ maxcount) {
  __shared__ R tgt[kGroup][4];
  __shared__ int tcell[kGroup][3];
  __shared__ int red_i[6];
  __shared__ R red_r[6];
  __shared__ int c_pre[kBuildCells + 1];   // prefix of the chunk's cell atom counts
  __shared__ int c_first[kBuildCells];     // first atom of each cell
  __shared__ int c_off[kBuildCells];       // packed (dx, dy, dz) cell offsets
  __shared__ int wcnt[BT / 64];
  __shared__ R s_p[BT][4];                // compacted hits of a round: position, radius
  __shared__ int s_m[BT];                  // their target masks
  __shared__ int s_o[BT];                 // their packed cell offsets
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int group = blockIdx.x;
  const int g0 = group * kGroup;
  const int n = geo.n;
  const int nc0 = geo.nc[0], nc1 = geo.nc[1], nc2 = geo.nc[2];
  int c0x, c0y, c0z;
  cell_coords(scell[g0], c0x, c0y, c0z);
  const int ntg = min(kGroup, n - g0);
  // targets relative to the corner of the group's first cell
  if (tid < kGroup) {
    const int ti = g0 + (tid < ntg ? tid : 0);
    int tcx, tcy, tcz;
    cell_coords(scell[ti], tcx, tcy, tcz);
    const int dcx = tcx - c0x, dcy = tcy - c0y, dcz = tcz - c0z;
    const R* tl = loc + 4 * (size_t)ti;
    tgt[tid][0] = tl[0] + (R)(dcx * geo.hv[0][0] + dcy * geo.hv[1][0] + dcz * geo.hv[2][0]);
    tgt[tid][1] = tl[1] + (R)(dcx * geo.hv[0][1] + dcy * geo.hv[1][1] + dcz * geo.hv[2][1]);
    tgt[tid][2] = tl[2] + (R)(dcx * geo.hv[0][2] + dcy * geo.hv[1][2] + dcz * geo.hv[2][2]);
    tgt[tid][3] = tl[3];
    tcell[tid][0] = dcx; tcell[tid][1] = dcy; tcell[tid][2] = dcz;
  }
  __syncthreads();
  // bounding box of the targets and their cell-offset range (wavefront 0 reduces)
  if (wave == 0) {
    const int t = lane < ntg ? lane : 0;
    R b0 = tgt[t][0], b1 = tgt[t][0], b2 = tgt[t][1], b3 = tgt[t][1], b4 = tgt[t][2],
      b5 = tgt[t][2];
    int m0 = tcell[t][0], m1 = tcell[t][0], m2 = tcell[t][1], m3 = tcell[t][1],
        m4 = tcell[t][2], m5 = tcell[t][2];
    for (int off = 1; off < 16; off <<= 1) {
      b0 = min(b0, __shfl_xor(b0, off)); b1 = max(b1, __shfl_xor(b1, off));
      b2 = min(b2, __shfl_xor(b2, off)); b3 = max(b3, __shfl_xor(b3, off));
      b4 = min(b4, __shfl_xor(b4, off)); b5 = max(b5, __shfl_xor(b5, off));
      m0 = min(m0, __shfl_xor(m0, off)); m1 = max(m1, __shfl_xor(m1, off));
      m2 = min(m2, __shfl_xor(m2, off)); m3 = max(m3, __shfl_xor(m3, off));
      m4 = min(m4, __shfl_xor(m4, off)); m5 = max(m5, __shfl_xor(m5, off));
    }
    if (lane == 0) {
      red_r[0] = b0; red_r[1] = b1; red_r[2] = b2;
      red_r[3] = b3; red_r[4] = b4; red_r[5] = b5;
      red_i[0] = m0; red_i[1] = m1; red_i[2] = m2;
      red_i[3] = m3; red_i[4] = m4; red_i[5] = m5;
    }
  }
  __syncthreads();
  const R bx0 = red_r[0], bx1 = red_r[1], by0 = red_r[2], by1 = red_r[3];
  const R bz0 = red_r[4], bz1 = red_r[5];
  const int dx0 = red_i[0] - geo.nr[0], dx1 = red_i[1] + geo.nr[0];
  const int dy0 = red_i[2] - geo.nr[1], dy1 = red_i[3] + geo.nr[1];
  const int dz0 = red_i[4] - geo.nr[2], dz1 = red_i[5] + geo.nr[2];
  const int nx = dx1 - dx0 + 1, ny = dy1 - dy0 + 1, nz = dz1 - dz0 + 1;
  const int ncells = nx * ny * nz;
  const R tau = (R)geo.tau, dd = (R)geo.damp_d;
  const R rp2 = (R)(geo.r_pair * geo.r_pair);
  int count = 0;
  for (int cc0 = 0; cc0 < ncells; cc0 += kBuildCells) {
    const int ncc = min(kBuildCells, ncells - cc0);
    __syncthreads();  // the previous chunk's tables are no longer read
    int cnt_cell = 0;
    if (tid < ncc) {
      const int ci = cc0 + tid;  // scan order: z outermost, then y, then x
      const int dx = dx0 + ci % nx, dy = dy0 + (ci / nx) % ny, dz = dz0 + ci / (nx * ny);
      int wx = (c0x + dx) % nc0; if (wx < 0) wx += nc0;
      int wy = (c0y + dy) % nc1; if (wy < 0) wy += nc1;
      int wz = (c0z + dz) % nc2; if (wz < 0) wz += nc2;
      const int cc = cell_index(wx, wy, wz);
      c_first[tid] = cell_start[cc];
      cnt_cell = cell_start[cc + 1] - cell_start[cc];
      c_off[tid] = ((dx + 512) << 20) | ((dy + 512) << 10) | (dz + 512);
    }
    // prefix of the counts: scan within each wavefront, then the wavefront offsets
    int v = cnt_cell;
    for (int o = 1; o < 64; o <<= 1) {
      const int u = __shfl_up(v, o);
      if (lane >= o) v += u;
    }
    if (lane == 63) wcnt[wave] = v;
    __syncthreads();
    int woff = 0;
    for (int w = 0; w < wave; ++w) woff += wcnt[w];
    if (tid < ncc) c_pre[tid + 1] = v + woff;
    if (tid == 0) c_pre[0] = 0;
    __syncthreads();
    const int total = c_pre[ncc];
    for (int r0 = 0; r0 < total; r0 += BT) {
      const int c = r0 + tid;
      uint32_t mask = 0;
      R px = R(0), py = R(0), pz = R(0), ps = R(0);
      int off = 0, j = 0;
      if (c < total) {
        // the cell holding candidate c: largest k with c_pre[k] <= c
        int lo = 0, hi = ncc - 1;
        while (lo < hi) {
          const int mid = (lo + hi + 1) >> 1;
          if (c_pre[mid] <= c) lo = mid; else hi = mid - 1;
        }
        j = c_first[lo] + (c - c_pre[lo]);
        off = c_off[lo];
        const int dx = (off >> 20) - 512, dy = ((off >> 10) & 1023) - 512,
                  dz = (off & 1023) - 512;
        const R sx = (R)(dx * geo.hv[0][0] + dy * geo.hv[1][0] + dz * geo.hv[2][0]);
        const R sy = (R)(dx * geo.hv[0][1] + dy * geo.hv[1][1] + dz * geo.hv[2][1]);
        const R sz = (R)(dx * geo.hv[0][2] + dy * geo.hv[1][2] + dz * geo.hv[2][2]);
        px = loc[4 * (size_t)j] + sx;
        py = loc[4 * (size_t)j + 1] + sy;
        pz = loc[4 * (size_t)j + 2] + sz;
        ps = loc[4 * (size_t)j + 3];
        const R ex = max(max(bx0 - px, px - bx1), R(0));
        const R ey = max(max(by0 - py, py - by1), R(0));
        const R ez = max(max(bz0 - pz, pz - bz1), R(0));
        if (ex * ex + ey * ey + ez * ez < rp2) {
          for (int t = 0; t < ntg; ++t) {
            const R rx = px - tgt[t][0], ry = py - tgt[t][1], rz = pz - tgt[t][2];
            const bool self = (j == g0 + t) && dx == tcell[t][0] && dy == tcell[t][1] &&
                              dz == tcell[t][2];
            if (!self && rx * rx + ry * ry + rz * rz < rp2) mask |= 1u << t;
          }
        }
      }
      // in-order compaction of the hits
      const unsigned long long bal = __ballot(mask != 0u);
      const int below = (int)__builtin_amdgcn_mbcnt_hi((unsigned)(bal >> 32),
                                                        __builtin_amdgcn_mbcnt_lo((unsigned)bal, 0u));
      if (lane == 0) wcnt[wave] = __popcll(bal);
      __syncthreads();
      int wpre = 0;
      for (int w = 0; w < wave; ++w) wpre += wcnt[w];
      int nloc = 0;
#pragma unroll
      for (int w = 0; w < BT / 64; ++w) nloc += wcnt[w];
      if (mask != 0u) {
        const int li = wpre + below;
        s_p[li][0] = px; s_p[li][1] = py; s_p[li][2] = pz; s_p[li][3] = ps;
        s_m[li] = (int)mask;
        s_o[li] = off;
        const int slot = count + li;
        if (slot < cap) hdr[(size_t)group * cap + slot] = make_int2(j, (int)mask);
      }
      __syncthreads();
      if (cap > 0) {
        // tensors of the round's hits: thread <-> (hit, target)
        for (int p = tid; p < nloc * kGroup; p += BT) {
          const int li = p / kGroup, t = p % kGroup;
          const int slot = count + li;
          if (slot >= cap) continue;
          const uint32_t mk = (uint32_t)s_m[li];
          R A = R(0), Bk = R(0), rx = R(0), ry = R(0), rz = R(0);
          const R qx = s_p[li][0], qy = s_p[li][1], qz = s_p[li][2], qs = s_p[li][3];
          if ((mk >> t) & 1u) {
            rx = qx - tgt[t][0]; ry = qy - tgt[t][1]; rz = qz - tgt[t][2];
            direct_kernel<R>(rx * rx + ry * ry + rz * rz, tau, R(1) / (qs + tgt[t][3]), dd,
                             A, Bk);
          }
          const size_t e = (size_t)group * cap + slot;
          R* o = Tg + e * kCandStride + t * kTensorWords;
          o[0] = A - Bk * rx * rx;
          o[1] = A - Bk * ry * ry;
          o[2] = A - Bk * rz * rz;
          o[3] = -Bk * rx * ry;
          o[4] = -Bk * rx * rz;
          o[5] = -Bk * ry * rz;
          if (Fg) {
            // radial data for forces, evaluated in double precision
            double Ad = 0.0, Bd = 0.0, dA = 0.0, dB = 0.0;
            if ((mk >> t) & 1u) {
              const double r2 = (double)rx * rx + (double)ry * ry + (double)rz * rz;
              direct_kernel_grad(r2, geo.tau, 1.0 / ((double)qs + (double)tgt[t][3]),
                                 geo.damp_d, Ad, Bd, dA, dB);
            }
            R* f = Fg + e * kCandStride + t * kTensorWords;
            f[0] = rx; f[1] = ry; f[2] = rz;
            f[3] = (R)Bd; f[4] = (R)dA; f[5] = (R)dB;
          }
        }
      }
      count += nloc;
      __syncthreads();  // the round's staging is free again
    }
  }
  // zero tensors up to a whole block of the matrix-core kernels (cap is a multiple of it)
  if (cap > 0 && count < cap) {
    const int pad = (count + kListBlock - 1) / kListBlock * kListBlock;
    R* o = Tg + (size_t)group * cap * kCandStride;
    for (int w = count * kCandStride + tid; w < pad * kCandStride; w += BT) o[w] = R(0);
  }
  if (tid == 0) {
    gcount[group] = count;
    atomicMax(maxcount, count);
  }
}

// E_dir of one group at a time per work-group: WPB wavefronts, each with 64 / NSUB
// right-hand sides x NSUB target subsets (lane = rhs + BW * subset), so
// B = 64 WPB / NSUB. More subsets give more wavefronts per group (small systems) and
// fewer target slots per lane. Tensors of CH candidates at a time are staged in LDS;
// the wave-uniform target mask skips out-of-range (target, source) pairs.
// The launch may hold fewer work-groups than groups: each then walks its XCD's range
// of groups with a stride, which leaves compute units and LDS free for the grid
// stages running beside it on another stream.
template <typename R, int NSUB, int WPB>
__global__ void __launch_bounds__(64 * WPB)
k_pair_list(const Geometry geo, const int2* __restrict__ hdr, const R* __restrict__ Tg,
            const int* __restrict__ gcount, int cap, const R* __restrict__ dv,
            R* __restrict__ Ed, int B) {
  constexpr int NT = 64 * WPB;
  constexpr int CH = 16 * WPB < 64 ? 16 * WPB : 64;  // candidates per LDS chunk
  constexpr int KT = kGroup / NSUB;   // target slots per lane
  constexpr int BW = 64 / NSUB;       // right-hand sides per wavefront
  constexpr int W16 = (int)(kCandStride * sizeof(R) / 16);  // 16-byte words per candidate
  __shared__ uint4 Tl4[CH * W16];
  __shared__ int2 hl[CH];
  const R* Tl = reinterpret_cast<const R*>(Tl4);
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int rhs = (tid >> 6) * BW + lane % BW;
  const int sub = lane / BW;
  // XCD-aware: each XCD owns a contiguous range of groups (work-groups are dealt to
  // the 8 XCDs round-robin; gridDim.x is a multiple of 8)
  const int ngroups = (geo.n + kGroup - 1) / kGroup;
  const int per = (ngroups + 7) / 8;
  const int nbx = gridDim.x / 8;
  for (int gi = blockIdx.x / 8; gi < per; gi += nbx) {
  const int group = (blockIdx.x % 8) * per + gi;
  if (group >= ngroups) return;  // uniform over the work-group
  const int cnt = min(gcount[group], cap);
  const int2* H = hdr + (size_t)group * cap;
  const uint4* T4 = reinterpret_cast<const uint4*>(Tg + (size_t)group * cap * kCandStride);

  R acc[KT][3];
#pragma unroll
  for (int k = 0; k < KT; ++k) acc[k][0] = acc[k][1] = acc[k][2] = R(0);

  for (int c0 = 0; c0 < cnt; c0 += CH) {
    const int nc = min(CH, cnt - c0);
    __syncthreads();
    for (int w = tid; w < nc * W16; w += NT) Tl4[w] = T4[(size_t)c0 * W16 + w];
    if (tid < nc) hl[tid] = H[c0 + tid];
    __syncthreads();
    int2 h = hl[0];
    int j = __builtin_amdgcn_readfirstlane(h.x);
    const R* dj = dv + (size_t)j * 3 * B + rhs;
    R n0 = dj[0], n1 = dj[B], n2 = dj[2 * B];
    for (int c = 0; c < nc; ++c) {
      const uint32_t msk = (uint32_t)__builtin_amdgcn_readfirstlane(h.y);
      const R d0 = n0, d1 = n1, d2 = n2;
      if (c + 1 < nc) {  // next candidate's dipoles while this one is applied
        h = hl[c + 1];
        j = __builtin_amdgcn_readfirstlane(h.x);
        dj = dv + (size_t)j * 3 * B + rhs;
        n0 = dj[0]; n1 = dj[B]; n2 = dj[2 * B];
      }
      const R* Tc = Tl + c * kCandStride + sub * kTensorWords;
      // masked slots only (the kernel is close to the LDS read bandwidth); the sums
      // go into the accumulators as fused multiply-add chains
#pragma unroll
      for (int k = 0; k < KT; ++k) {
        if ((msk >> (k * NSUB)) & ((1u << NSUB) - 1u)) {
          const R* t = Tc + k * NSUB * kTensorWords;
          const R txx = t[0], tyy = t[1], tzz = t[2], txy = t[3], txz = t[4], tyz = t[5];
          R* a = acc[k];
          a[0] = fma(txx, d0, a[0]);
          a[0] = fma(txy, d1, a[0]);
          a[0] = fma(txz, d2, a[0]);
          a[1] = fma(txy, d0, a[1]);
          a[1] = fma(tyy, d1, a[1]);
          a[1] = fma(tyz, d2, a[1]);
          a[2] = fma(txz, d0, a[2]);
          a[2] = fma(tyz, d1, a[2]);
          a[2] = fma(tzz, d2, a[2]);
        }
      }
    }
  }
#pragma unroll
  for (int k = 0; k < KT; ++k) {
    const int i = group * kGroup + k * NSUB + sub;
    if (i < geo.n) {
      Ed[((size_t)i * 3 + 0) * B + rhs] = acc[k][0];
      Ed[((size_t)i * 3 + 1) * B + rhs] = acc[k][1];
      Ed[((size_t)i * 3 + 2) * B + rhs] = acc[k][2];
    }
  }
  }  // groups of this work-group
}

// The dense products below give every target of a group 0 x d of the candidates out of its
// range: not a number where d is not finite. The bfloat16 planes of k_pair_split besides turn
// floats above the largest bfloat16 into infinities, and below 2^-110 the last plane falls
// under the smallest bfloat16 (2^-133), an error of 2^-134 a dipole and so about as much in
// the field. Where an element of a column's field is not finite, or smaller than the floor
// that the caller gives, the work-group sums that column again over the pairs in range alone,
// in the list's type, as the vector kernel does. Columns of ordinary values keep their bits;
// testing them costs an LDS flag and a barrier a group.
// A matvec's floor is 2^-104, 2^24 times that error with a factor of 64 to spare. The reverse
// sweep has none: the adjoint vectors of the last steps are that small as a matter of course
// (they fall with the square of the converging Lanczos vectors' weights), and add nothing to
// forces whose other terms are 10^20 times larger; summed again, they doubled the direct
// sum's share of a reverse sweep.
template <typename R>
__device__ __forceinline__ bool out_of_bounds(R v, R floor) {
  const R a = fabs(v);
  const R huge = sizeof(R) == 4 ? (R)3.4028235e38f : (R)1.7976931348623157e308;
  return !(a <= huge) || (a < floor && a > R(0));
}

// Columns of a work-group whose field is to be summed again, marked with the number of the
// group (its turn, from 1): nothing is cleared between groups. A mark of the next group comes
// after the barriers around that group's candidates, so past every thread's reading here (a
// group without candidates has nothing to mark).
template <int W>
struct Redo {
  int turn[W];
  int any;
  __device__ __forceinline__ void clear() {
    if (threadIdx.x < W) turn[threadIdx.x] = 0;
    if (threadIdx.x == 0) any = 0;
  }
  // bit t of odd: the lane's column first + step * ST (t / ST) + t % ST
  __device__ __forceinline__ void mark(int now, unsigned odd, int first, int step, int ST) {
    any = now;
    for (; odd; odd &= odd - 1u) {
      const int t = __ffs(odd) - 1;
      turn[first + step * ST * (t / ST) + t % ST] = now;
    }
  }
};

// The marked columns (of W, at dv and Ed) of one group over its candidates [lo, hi).
template <typename R, int W>
__device__ __forceinline__ void sum_in_range(const Geometry& geo, const Redo<W>& redo, int now,
                                             int group, const int2* H, const R* T, int lo, int hi,
                                             const R* dv, R* Ed, size_t Bs) {
  // (opaque, so that nothing of this is kept in registers across the products)
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int c = tid % W;
  if (redo.turn[c] != now) return;
#pragma unroll 1
  for (int t = tid / W; t < kGroup; t += 256 / W) {
    const int i = group * kGroup + t;
    if (i >= geo.n) break;
    R e0 = R(0), e1 = R(0), e2 = R(0);
#pragma unroll 1
    for (int k = lo; k < hi; ++k) {
      const int2 h = H[k];
      if (!(((uint32_t)h.y >> t) & 1u)) continue;
      const R* q = T + ((size_t)k * kGroup + t) * kTensorWords;
      const R* d = dv + (size_t)h.x * 3 * Bs + c;
      const R d0 = d[0], d1 = d[Bs], d2 = d[2 * Bs];
      e0 = fma(q[4], d2, fma(q[3], d1, fma(q[0], d0, e0)));
      e1 = fma(q[5], d2, fma(q[1], d1, fma(q[3], d0, e1)));
      e2 = fma(q[2], d2, fma(q[5], d1, fma(q[4], d0, e2)));
    }
    R* o = Ed + (size_t)i * 3 * Bs + c;
    o[0] = e0;
    o[Bs] = e1;
    o[2 * Bs] = e2;
  }
}

// E_dir of a group on the matrix cores. For the group's 16 targets t the field is one
// dense product over k = 3 c + b (candidate c, component b):
//   E[t][a][rhs] = sum_k T_(c,t)[a][b] d_(j(c))[b][rhs],
// the list's zero tensors standing for out-of-range (target, candidate) pairs. It is
// computed as three 16-row tiles (a = x, y, z) times NT column tiles of 16 right-hand
// sides with v_mfma_f32_16x16x4_f32 or v_mfma_f64_16x16x4_f64, four rows of k per
// instruction: the instruction takes A[i][k] from lane i + 16 k and B[k][j] from lane
// j + 16 k and leaves D[i][j], in float, in register i % 4 of lane j + 16 (i / 4), and in
// double in register i / 4 of lane j + 16 (i % 4). A wavefront owns 16 NT right-hand sides
// and every NK-th block of four candidates (three steps of four k rows); the NK partial
// products of a group are added in LDS in wavefront order, so the result does not depend
// on timing. The source atoms of up to kMfmaChunk candidates at a time are staged in LDS;
// each lane then reads its tensor row and dipole component straight from global memory,
// one block of three steps ahead of the matrix instructions that use them.
// Float blocks of 64 and more run k_pair_split instead.
// Small systems: a launch of one work-group per group leaves most of the GPU idle (41 of
// 256 CUs at 648 atoms) while each wavefront walks several hundred candidates, so the
// candidates of a group are also split over gridDim.y work-groups, each writing its own
// part of the field; the gather adds the parts in order (pair_parts).
constexpr int kMfmaChunk = 1024;  // candidates per LDS chunk (a multiple of 4)

template <typename R, int NT>
struct MfmaOperands {
  R a[3];
  R b[NT];
};

template <typename R, int NK, int NT, int NN>
__global__ void __launch_bounds__(256)
k_pair_mfma(const Geometry geo, const int2* __restrict__ hdr, const R* __restrict__ Tg,
            const R* __restrict__ Tz, const int* __restrict__ gcount, int cap,
            const R* __restrict__ dv, R* __restrict__ Ed, int B) {
  typedef typename Mma<R>::acc Acc;
  constexpr int VN = NT * (int)sizeof(R) > 16 ? 16 / (int)sizeof(R) : NT;  // reals per vector
  // partial tiles of one component for the NK-way reduction: [wavefront][tile][row][lane]
  // for the work-group's NN x NK wavefronts (NN column wavefronts)
  __shared__ R red[NK > 1 ? NN * NK * NT * 256 : 1];
  __shared__ int jl[kMfmaChunk];
  __shared__ Redo<16 * NT * NN> redo;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int wk = wave % NK, wn = wave / NK;
  const int col = lane & 15, row = lane >> 4;
  // column col of column tile t is right-hand side rhs + t: a lane's NT right-hand
  // sides are contiguous, so its dipoles and results move as vectors of 16 bytes
  const int rhs = wn * 16 * NT + NT * col;
  const size_t Bs = (size_t)B;
  // this work-group's part of every candidate list, in units of four candidates
  const int part = blockIdx.y, parts = gridDim.y;
  Ed += (size_t)part * 3 * geo.n * Bs;
  // XCD-aware walk over groups, as in the vector list kernel
  const int ngroups = (geo.n + kGroup - 1) / kGroup;
  const int per = (ngroups + 7) / 8;
  const int nbx = gridDim.x / 8;
  redo.clear();
  for (int gi = blockIdx.x / 8; gi < per; gi += nbx) {
    const int group = (blockIdx.x % 8) * per + gi;
    if (group >= ngroups) return;  // uniform over the work-group
    const int full = min(gcount[group], cap);
    const int q4 = (full + 3) / 4;
    const int clo = 4 * (int)((long)q4 * part / parts);
    const int cnt = min(full, 4 * (int)((long)q4 * (part + 1) / parts));
    const int2* H = hdr + (size_t)group * cap;
    const R* T = Tg + (size_t)group * cap * kCandStride;
    Acc acc[3][NT];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[a][t] = Acc{R(0), R(0), R(0), R(0)};
    for (int c0 = clo; c0 < cnt; c0 += kMfmaChunk) {
      const int nc = min(kMfmaChunk, cnt - c0);
      __syncthreads();  // the previous chunk's source atoms have been read
      for (int c = threadIdx.x; c < nc; c += blockDim.x) jl[c] = H[c0 + c].x;
      __syncthreads();
      const R* Tc = T + (size_t)c0 * kCandStride;
      // operands of one step: row b of the symmetric tensor (xx, yy, zz, xy, xz, yz) of
      // candidate c and target col (b = 0: xx xy xz, b = 1: xy yy yz, b = 2: xz yz zz)
      // and component b of the candidate's dipoles. Every load is issued: candidates
      // past the chunk read the zero tensor Tz and the chunk's first dipoles, so no
      // branch hides a load from the compiler's count of loads in flight.
      auto load = [&](int c, int b, const int (&w)[3], MfmaOperands<R, NT>& o) {
        const bool ok = c < nc;
        const R* tt = ok ? Tc + ((size_t)c * kGroup + col) * kTensorWords : Tz;
        const Pack<R, VN>* dj = reinterpret_cast<const Pack<R, VN>*>(
            dv + ((size_t)jl[ok ? c : 0] * 3 + b) * Bs + rhs);
        o.a[0] = tt[w[0]]; o.a[1] = tt[w[1]]; o.a[2] = tt[w[2]];
#pragma unroll
        for (int q = 0; q < NT / VN; ++q) {
          const Pack<R, VN> v = dj[q];
#pragma unroll
          for (int u = 0; u < VN; ++u) o.b[VN * q + u] = v.v[u];
        }
      };
      auto apply = [&](const MfmaOperands<R, NT>& o) {
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
          for (int t = 0; t < NT; ++t) acc[a][t] = Mma<R>::fma(o.a[a], o.b[t], acc[a][t]);
      };
      // The work comes in blocks of 4 candidates = 12 rows of k = 3 steps, and the
      // wavefront takes blocks p = wk, wk + NK, ...: lane row r of step u of block p has
      // k = 12 p + 4 u + r, so its candidate 4 p + (4 u + r) / 3 and component
      // (4 u + r) % 3 are fixed per lane and step. The operands of the next block are in
      // flight while the matrix instructions of this one run.
      int cu[3], bu[3], wu[3][3];
#pragma unroll
      for (int u = 0; u < 3; ++u) {
        const int kq = 4 * u + row;
        cu[u] = kq / 3;
        bu[u] = kq % 3;
        wu[u][0] = bu[u] == 0 ? 0 : bu[u] == 1 ? 3 : 4;
        wu[u][1] = bu[u] == 0 ? 3 : bu[u] == 1 ? 1 : 5;
        wu[u][2] = bu[u] == 0 ? 4 : bu[u] == 1 ? 5 : 2;
      }
      const int nb = (nc + 3) / 4;
      const int m = wk < nb ? (nb - wk + NK - 1) / NK : 0;  // this wavefront's blocks
      MfmaOperands<R, NT> buf[3];
#pragma unroll
      for (int u = 0; u < 3; ++u) load(4 * wk + cu[u], bu[u], wu[u], buf[u]);
      for (int i = 0; i < m; ++i) {
        const int cn = 4 * (wk + NK * (i + 1));  // first candidate of the next block
#pragma unroll
        for (int u = 0; u < 3; ++u) {
          apply(buf[u]);
          load(cn + cu[u], bu[u], wu[u], buf[u]);
          // keep each step's instructions together: interleaving the accumulator chains
          // of neighbouring steps makes the register allocator double the accumulators
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    unsigned odd = 0u;  // column tiles with a value out of bounds
    // component a of the lane's NT right-hand sides for the target of register r
    auto store = [&](int a, int r, const R (&v)[NT]) {
      const int i = group * kGroup + Mma<R>::row(row, r);
      if (i >= geo.n) return;
#pragma unroll
      for (int t = 0; t < NT; ++t) odd |= (unsigned)out_of_bounds<R>(v[t], R(0)) << t;
      Pack<R, VN>* o = reinterpret_cast<Pack<R, VN>*>(Ed + ((size_t)i * 3 + a) * Bs + rhs);
#pragma unroll
      for (int q = 0; q < NT / VN; ++q) {
        Pack<R, VN> w;
#pragma unroll
        for (int u = 0; u < VN; ++u) w.v[u] = v[VN * q + u];
        o[q] = w;
      }
    };
    if constexpr (NK == 1) {
#pragma unroll
      for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          R v[NT];
#pragma unroll
          for (int t = 0; t < NT; ++t) v[t] = acc[a][t][r];
          store(a, r, v);
        }
    } else {
      // one component at a time: every wavefront leaves its partial tiles in LDS, then
      // wavefront wk adds the NK partials of the rows r = wk, wk + NK, ... in wavefront
      // order and stores them
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        __syncthreads();  // the previous round's partials have been read
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            red[(((wn * NK + wk) * NT + t) * 4 + r) * 64 + lane] = acc[a][t][r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if (r % NK != wk) continue;
          R v[NT];
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            v[t] = red[((wn * NK * NT + t) * 4 + r) * 64 + lane];
#pragma unroll
            for (int w = 1; w < NK; ++w)
              v[t] += red[(((wn * NK + w) * NT + t) * 4 + r) * 64 + lane];
          }
          store(a, r, v);
        }
      }
    }
    if (odd) redo.mark(gi + 1, odd, rhs, 1, NT);
    __syncthreads();
    if (redo.any == gi + 1)
      sum_in_range<R, 16 * NT * NN>(geo, redo, gi + 1, group, H, T, clo, cnt, dv, Ed, Bs);
  }  // groups of this work-group
}


typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// x = h + m + l in bfloat16, each the rounded remainder of the ones before: 8 bits each with
// signs, so the 24 bits of a float between 2^-110 and the largest bfloat16 (3.39e38).
struct Split8 {
  bf16x8 h, m, l;
};
__device__ __forceinline__ Split8 split8(const float (&x)[8]) {
  Split8 o;
#pragma unroll
  for (int i = 0; i < 8; i += 2) {
    const f32x2 v = {x[i], x[i + 1]};
    const bf16x2 h = __builtin_convertvector(v, bf16x2);
    const f32x2 r = v - __builtin_convertvector(h, f32x2);
    const bf16x2 m = __builtin_convertvector(r, bf16x2);
    const f32x2 q = r - __builtin_convertvector(m, f32x2);
    const bf16x2 l = __builtin_convertvector(q, bf16x2);
    o.h[i] = h[0]; o.h[i + 1] = h[1];
    o.m[i] = m[0]; o.m[i + 1] = m[1];
    o.l[i] = l[0]; o.l[i + 1] = l[1];
  }
  return o;
}

// The float direct sum for 64 right-hand sides and more, on the bfloat16 matrix cores, whose
// rate is 16 times the float ones'. Tensors and dipoles are split into three bfloat16 planes
// (h, m, l) in registers, and of the nine products of planes the six down to 2^-16 are
// summed, the dropped three (2^-24 and below) being under the rounding of a float product.
// For one component b of 32 candidates, v_mfma_f32_16x16x32_bf16 multiplies the tensor
// components (a, b) of the group's 16 targets with 16 right-hand sides: it takes
// A[i][k] from lane i + 16 (k / 8), element k % 8, B[k][j] likewise from lane
// j + 16 (k / 8), and leaves D as the float instruction of k_pair_mfma does. The products of
// a block of 32 candidates start from zero, smallest first, and are added to the running sum
// in float once, so the instruction's alignment of its addends works on a block's sum and
// not on the total: against a double sum the field's error is 1.25e-7 of its norm, 2.8e-7
// with float products (24k atoms, 724 candidates a group).
// A wavefront owns 16 NT right-hand sides and every fourth block of 32 candidates; it reads
// the block's tensors once (24 bytes a pair, the list padded with zero tensors to whole
// blocks), then the dipoles of ST column tiles at a time, one step ahead of their use. The
// four partial sums are added in LDS in wavefront order; gridDim.y parts of the candidates
// as in k_pair_mfma, gridDim.z slices of the right-hand sides. 24k atoms, B = 128: 417 us a
// launch with float products, 278 us here, 12k atoms, B = 64: 122 and 78 us. What remains
// is loads: 1.7 GB of dipoles and 0.42 GB of tensors a launch, half of it from beyond L2.
// <4, 4> takes 242 registers, <8, 2> all 256 with 27 spilled: two work-groups a CU each.
template <int NT, int ST>
__global__ void __launch_bounds__(256, 2)
k_pair_split(const Geometry geo, const int2* __restrict__ hdr, const float* __restrict__ Tg,
             const int* __restrict__ gcount, int cap, const float* __restrict__ dv,
             float* __restrict__ Ed, int B, float floor) {
  constexpr int NQ = NT / ST;  // column steps of ST tiles
  __shared__ float red[4 * NT * 256];
  __shared__ int jl[kMfmaChunk];
  __shared__ Redo<16 * NT> redo;
  const int lane = threadIdx.x & 63;
  const int wk = threadIdx.x >> 6;
  const int col = lane & 15, row = lane >> 4;
  const size_t Bs = (size_t)B;
  const int rhs0 = blockIdx.z * 16 * NT;
  const int part = blockIdx.y, parts = gridDim.y;
  Ed += (size_t)part * 3 * geo.n * Bs + rhs0;
  const int ngroups = (geo.n + kGroup - 1) / kGroup;
  const int per = (ngroups + 7) / 8;
  const int nbx = gridDim.x / 8;
  redo.clear();
  for (int gi = blockIdx.x / 8; gi < per; gi += nbx) {
    const int group = (blockIdx.x % 8) * per + gi;
    if (group >= ngroups) return;  // uniform over the work-group
    const int full = min(gcount[group], cap);
    const int q32 = (full + 31) / 32;
    const int clo = 32 * (int)((long)q32 * part / parts);
    const int cnt = min(full, 32 * (int)((long)q32 * (part + 1) / parts));
    const int2* H = hdr + (size_t)group * cap;
    const float* T = Tg + (size_t)group * cap * kCandStride;
    f32x4 acc[3][NT];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[a][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int c0 = clo; c0 < cnt; c0 += kMfmaChunk) {
      const int nc = min(kMfmaChunk, cnt - c0);
      const int nb = (nc + 31) / 32;
      __syncthreads();  // the previous chunk's source atoms have been read
      for (int c = threadIdx.x; c < 32 * nb; c += 256) jl[c] = H[c0 + (c < nc ? c : 0)].x;
      __syncthreads();
      for (int p = wk; p < nb; p += 4) {
        const int cb = 32 * p + 8 * row;  // first of this lane's 8 candidates
        const float* dp[8];
#pragma unroll
        for (int e = 0; e < 8; ++e)
          dp[e] = dv + (size_t)jl[cb + e] * 3 * Bs + rhs0 + ST * col;
        float d[2][8][ST];
        auto load = [&](int b, int q, float (&o)[8][ST]) {
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const Pack<float, ST> v =
                *reinterpret_cast<const Pack<float, ST>*>(dp[e] + b * Bs + 16 * ST * q);
#pragma unroll
            for (int u = 0; u < ST; ++u) o[e][u] = v.v[u];
          }
        };
        load(0, 0, d[0]);
        Split8 tt[6];
        {
          const float2* tp =
              reinterpret_cast<const float2*>(T + ((size_t)(c0 + cb) * kGroup + col) * kTensorWords);
          float tr[6][8];
#pragma unroll
          for (int e = 0; e < 8; ++e)
#pragma unroll
            for (int w = 0; w < 3; ++w) {
              const float2 v = tp[e * (kCandStride / 2) + w];
              tr[2 * w][e] = v.x;
              tr[2 * w + 1][e] = v.y;
            }
#pragma unroll
          for (int w = 0; w < 6; ++w) tt[w] = split8(tr[w]);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int b = 0; b < 3; ++b) {
          // stored components (a, b): xx xy xz, xy yy yz, xz yz zz
          constexpr int kRow[3][3] = {{0, 3, 4}, {3, 1, 5}, {4, 5, 2}};
#pragma unroll
          for (int q = 0; q < NQ; ++q) {
            const int st = b * NQ + q;
            if (st + 1 < 3 * NQ) load((st + 1) / NQ, (st + 1) % NQ, d[(st + 1) & 1]);
#pragma unroll
            for (int u = 0; u < ST; ++u) {
              float x[8];
#pragma unroll
              for (int e = 0; e < 8; ++e) x[e] = d[st & 1][e][u];
              const Split8 s = split8(x);
              f32x4 w[3];
#pragma unroll
              for (int a = 0; a < 3; ++a) w[a] = f32x4{0.f, 0.f, 0.f, 0.f};
#define MBD_STEP(TP, DP)                                                                  \
  _Pragma("unroll") for (int a = 0; a < 3; ++a) w[a] =                                    \
      __builtin_amdgcn_mfma_f32_16x16x32_bf16(tt[kRow[b][a]].TP, s.DP, w[a], 0, 0, 0)
              MBD_STEP(l, h);
              MBD_STEP(h, l);
              MBD_STEP(m, m);
              MBD_STEP(m, h);
              MBD_STEP(h, m);
              MBD_STEP(h, h);
#undef MBD_STEP
#pragma unroll
              for (int a = 0; a < 3; ++a) acc[a][q * ST + u] += w[a];
              // tile by tile: interleaved, the tiles' splits no longer fit the registers
              __builtin_amdgcn_sched_barrier(0);
            }
          }
        }
      }
    }
    unsigned odd = 0u;  // column tiles with a value out of bounds
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      __syncthreads();  // the previous round's partials have been read
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[((wk * NT + t) * 4 + r) * 64 + lane] = acc[a][t][r];
      __syncthreads();
      // wavefront wk: matrix row 4 row + wk of every tile
      const int i = group * kGroup + 4 * row + wk;
      if (i < geo.n) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          Pack<float, ST> w;
#pragma unroll
          for (int u = 0; u < ST; ++u) {
            const int t = q * ST + u;
            float v = red[(t * 4 + wk) * 64 + lane];
#pragma unroll
            for (int k = 1; k < 4; ++k) v += red[((k * NT + t) * 4 + wk) * 64 + lane];
            w.v[u] = v;
            odd |= (unsigned)out_of_bounds<float>(v, floor) << t;
          }
          *reinterpret_cast<Pack<float, ST>*>(Ed + ((size_t)i * 3 + a) * Bs + 16 * ST * q +
                                              ST * col) = w;
        }
      }
    }
    if (odd) redo.mark(gi + 1, odd, ST * col, 16, ST);
    __syncthreads();
    if (redo.any == gi + 1)
      sum_in_range<float, 16 * NT>(geo, redo, gi + 1, group, H, T, clo, cnt, dv + rhs0, Ed, Bs);
  }
}


// Direct-space part of the bilinear force term for one reverse step: with
// p = g * lbar_k and q = g * y_k, dS/dR_t for S = sum_(t,j,n) p_t^T T_dir(r) q_j is
//   dS/dR_t = -sum_(j,n) grad_r u,  u = p_t^T T_dir(r) q_j + q_t^T T_dir(r) p_j,
// r = R_j + n - R_t; with T_dir = A I - B r r^T, X = p_t.q_j + q_t.p_j and
// Y = (p_t.r)(q_j.r) + (q_t.r)(p_j.r):
//   grad_r u = r (A'/r X - B'/r Y) - B [p_t (q_j.r) + q_j (p_t.r) + q_t (p_j.r) + p_j (q_t.r)].
// Work-group per group: TW x RS wavefronts; wavefront (tw, rs) owns the targets
// [tw 16/TW, (tw+1) 16/TW) and the right-hand sides [rs BW, (rs+1) BW) (BW = 64/NSUB,
// NSUB > 1 only when B < 64), so the mask branch is uniform and no lane idles on an
// out-of-range pair. TP target slots per pass keep p_t and q_t in registers. The sum
// over right-hand sides is reduced per target and added to fsum (each group owns its
// targets: no atomics, fixed order).
template <typename R, int NSUB, int TW, int RS, int TP>
__global__ void __launch_bounds__(64 * TW * RS)
k_pair_force(const Geometry geo, const int2* __restrict__ hdr, const R* __restrict__ Fg,
             const int* __restrict__ gcount, int cap, const R* __restrict__ pv,
             const R* __restrict__ qv, double* __restrict__ fsum, int B) {
  constexpr int NT = 64 * TW * RS;
  constexpr int CH = 16 * TW * RS < 64 ? 16 * TW * RS : 64;
  constexpr int TPW = kGroup / TW;
  constexpr int KT = TPW / NSUB;
  constexpr int NPASS = KT / TP;
  constexpr int BW = 64 / NSUB;
  constexpr int W16 = (int)(kCandStride * sizeof(R) / 16);
  static_assert(KT >= 1 && KT * NSUB * TW == kGroup && NPASS * TP == KT, "bad split");
  __shared__ uint4 Fl4[CH * W16];
  __shared__ int2 hl[CH];
  __shared__ double red[RS][kGroup][3];
  const R* Fl = reinterpret_cast<const R*>(Fl4);
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int tw = wave % TW, rs = wave / TW;
  const int t0 = tw * TPW;
  const int rhs = rs * BW + lane % BW;
  const int sub = lane / BW;
  const int per = (gridDim.x + 7) / 8;
  const int group = (blockIdx.x % 8) * per + blockIdx.x / 8;
  const int ngroups = (geo.n + kGroup - 1) / kGroup;
  if (group >= ngroups) return;  // uniform over the work-group
  // this work-group's part of the candidates, with its own force sums
  const int full = min(gcount[group], cap);
  const int clo = (int)((long)full * blockIdx.y / gridDim.y);
  const int cnt = (int)((long)full * (blockIdx.y + 1) / gridDim.y);
  fsum += (size_t)blockIdx.y * 3 * geo.n;
  const int2* H = hdr + (size_t)group * cap;
  const uint4* F4 = reinterpret_cast<const uint4*>(Fg + (size_t)group * cap * kCandStride);
  for (int pass = 0; pass < NPASS; ++pass) {
    R pt[TP][3], qt[TP][3], G[TP][3];
#pragma unroll
    for (int k = 0; k < TP; ++k) {
      const int i = group * kGroup + t0 + (pass * TP + k) * NSUB + sub;
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        pt[k][a] = i < geo.n ? pv[((size_t)i * 3 + a) * B + rhs] : R(0);
        qt[k][a] = i < geo.n ? qv[((size_t)i * 3 + a) * B + rhs] : R(0);
        G[k][a] = R(0);
      }
    }
    for (int c0 = clo; c0 < cnt; c0 += CH) {
      const int nc = min(CH, cnt - c0);
      __syncthreads();
      for (int w = tid; w < nc * W16; w += NT) Fl4[w] = F4[(size_t)c0 * W16 + w];
      if (tid < nc) hl[tid] = H[c0 + tid];
      __syncthreads();
      for (int c = 0; c < nc; ++c) {
        const int2 h = hl[c];
        const int j = __builtin_amdgcn_readfirstlane(h.x);
        const uint32_t msk = (uint32_t)__builtin_amdgcn_readfirstlane(h.y) >> t0;
        const R* pj = pv + (size_t)j * 3 * B + rhs;
        const R* qj = qv + (size_t)j * 3 * B + rhs;
        const R p0 = pj[0], p1 = pj[B], p2 = pj[2 * B];
        const R q0 = qj[0], q1 = qj[B], q2 = qj[2 * B];
        const R* Fc = Fl + c * kCandStride + (t0 + sub) * kTensorWords;
#pragma unroll
        for (int k = 0; k < TP; ++k) {
          const int slot = pass * TP + k;
          if ((msk >> (slot * NSUB)) & ((1u << NSUB) - 1u)) {
            const R* f = Fc + slot * NSUB * kTensorWords;
            const R rx = f[0], ry = f[1], rz = f[2], Bk = f[3], c1 = f[4], c2 = f[5];
            const R prt = pt[k][0] * rx + pt[k][1] * ry + pt[k][2] * rz;
            const R qrt = qt[k][0] * rx + qt[k][1] * ry + qt[k][2] * rz;
            const R prj = p0 * rx + p1 * ry + p2 * rz;
            const R qrj = q0 * rx + q1 * ry + q2 * rz;
            const R X = pt[k][0] * q0 + pt[k][1] * q1 + pt[k][2] * q2 + qt[k][0] * p0 +
                        qt[k][1] * p1 + qt[k][2] * p2;
            const R Y = prt * qrj + qrt * prj;
            const R sc = c1 * X - c2 * Y;
            G[k][0] -= sc * rx - Bk * (pt[k][0] * qrj + q0 * prt + qt[k][0] * prj + p0 * qrt);
            G[k][1] -= sc * ry - Bk * (pt[k][1] * qrj + q1 * prt + qt[k][1] * prj + p1 * qrt);
            G[k][2] -= sc * rz - Bk * (pt[k][2] * qrj + q2 * prt + qt[k][2] * prj + p2 * qrt);
          }
        }
      }
    }
    // sum over the right-hand sides: the BW lanes of a target subset, then the slices
#pragma unroll
    for (int k = 0; k < TP; ++k) {
      double g0 = G[k][0], g1 = G[k][1], g2 = G[k][2];
      for (int off = 1; off < BW; off <<= 1) {
        g0 += __shfl_xor(g0, off);
        g1 += __shfl_xor(g1, off);
        g2 += __shfl_xor(g2, off);
      }
      const int t = t0 + (pass * TP + k) * NSUB + sub;
      if (lane % BW == 0) {
        red[rs][t][0] = g0;
        red[rs][t][1] = g1;
        red[rs][t][2] = g2;
      }
    }
    __syncthreads();
    if (tid < kGroup * 3) {
      const int t = tid / 3, a = tid % 3;
      if (((t % TPW) / NSUB) / TP == pass) {  // target t was handled in this pass
        double v = 0.0;
        for (int r = 0; r < RS; ++r) v += red[r][t][a];
        const int i = group * kGroup + t;
        if (i < geo.n) fsum[3 * (size_t)i + a] += v;
      }
    }
  }
}


// The same direct force term on the bfloat16 matrix cores (float, B a multiple of 16, at
// most 128). Summed over the right-hand sides, a pair's term needs only one 3x3 matrix,
//   M = sum_rhs p_t q_j^T + q_t p_j^T:
//   X = tr M,  (M + M^T) r = sum_rhs [p_t (q_j.r) + q_j (p_t.r) + q_t (p_j.r) + p_j (q_t.r)]
//   =: m,  Y = r.m / 2,  grad_r u = r (A'/r X - B'/r Y) - B m.
// For a group's 16 targets and a block of 16 candidates, M is 9 tiles of 16 x 16 (component
// pairs (a, b), rows = targets, columns = candidates), dense products over the 2 B values
// k = (p_t | q_t) against (q_j | p_j), 32 a step. The floats are split into three bfloat16
// planes and the six products above 2^-24 summed, as in k_pair_split: the targets' once per
// group, into LDS, the candidates' in registers, their loads one step ahead. After a block's
// last step each lane holds M of the pairs (targets 4 row .. 4 row + 3, candidate lane % 16)
// and adds their terms (in-range pairs only) to its float64 partial forces; the 16 candidate
// lanes, then the four wavefronts of the group are summed in a fixed order and the group's
// forces added to this part's fsum (each group owns its targets: no atomics). 12k atoms,
// B = 64, beside the grid stages: 447 us a launch with float products, 369 us here. At most
// 168 registers, so that three work-groups fit on a CU: 752 of them are one round on the
// GPU's 768 places, not two on 512 (alone: 255 us with two a CU, 195 with three).
constexpr int kForceChunk = 512;  // candidates per LDS chunk (a multiple of 16)
inline size_t force_lds(int B) { return (size_t)3 * 3 * kGroup * (2 * B + 8) * 2; }

__global__ void __launch_bounds__(256, 3)
k_pair_force_split(const Geometry geo, const int2* __restrict__ hdr,
                   const float* __restrict__ Fg, const int* __restrict__ gcount, int cap,
                   const float* __restrict__ pv, const float* __restrict__ qv,
                   double* __restrict__ fsum, int B) {
  // [plane][a][t][k], rows padded by 16 bytes; the start of the next group waits for it
  extern __shared__ unsigned char smem_raw[];
  __bf16* tl = reinterpret_cast<__bf16*>(smem_raw);
  __shared__ int jl[kForceChunk];
  __shared__ int ml[kForceChunk];
  __shared__ double red[4][kGroup][3];
  const int RP = 2 * B + 8;                 // padded row
  const int plane = 3 * kGroup * RP;        // elements of one plane
  const int lane = threadIdx.x & 63;
  const int wk = threadIdx.x >> 6;
  const int col = lane & 15, row = lane >> 4;
  const size_t Bs = (size_t)B;
  fsum += (size_t)blockIdx.y * 3 * geo.n;
  const int ngroups = (geo.n + kGroup - 1) / kGroup;
  const int per = (ngroups + 7) / 8;
  const int nbx = gridDim.x / 8;
  for (int gi = blockIdx.x / 8; gi < per; gi += nbx) {
    const int group = (blockIdx.x % 8) * per + gi;
    if (group >= ngroups) return;  // uniform over the work-group
    // this work-group's part of the candidates (in blocks of 16), with its own force sums
    const int full = min(gcount[group], cap);
    const int q16 = (full + 15) / 16;
    const int clo = 16 * (int)((long)q16 * blockIdx.y / gridDim.y);
    const int cnt = min(full, 16 * (int)((long)q16 * (blockIdx.y + 1) / gridDim.y));
    const int2* H = hdr + (size_t)group * cap;
    const float* F = Fg + (size_t)group * cap * kCandStride;
    __syncthreads();  // the previous group's LDS contents have been read
    // the group's (p_t | q_t) in planes, zero for targets past the end: 8 values a thread
    for (int e = threadIdx.x; e < 3 * kGroup * B / 4; e += 256) {
      const int k8 = e % (B / 4), t = e / (B / 4) % kGroup, a = e / (B / 4 * kGroup);
      const int i = group * kGroup + t;
      const bool second = 8 * k8 >= B;
      const float* src = (second ? qv : pv) + ((size_t)i * 3 + a) * Bs + (8 * k8 - (second ? B : 0));
      float x[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) x[u] = i < geo.n ? src[u] : 0.f;
      const Split8 sp = split8(x);
      __bf16* o = tl + (a * kGroup + t) * RP + 8 * k8;
      *reinterpret_cast<bf16x8*>(o) = sp.h;
      *reinterpret_cast<bf16x8*>(o + plane) = sp.m;
      *reinterpret_cast<bf16x8*>(o + 2 * plane) = sp.l;
    }
    double G[4][3];
#pragma unroll
    for (int r = 0; r < 4; ++r) G[r][0] = G[r][1] = G[r][2] = 0.0;
    for (int c0 = clo; c0 < cnt; c0 += kForceChunk) {
      const int nc = min(kForceChunk, cnt - c0);
      __syncthreads();  // the previous chunk's lists have been read
      for (int c = threadIdx.x; c < nc; c += 256) {
        const int2 h = H[c0 + c];
        jl[c] = h.x;
        ml[c] = h.y;
      }
      __syncthreads();
      const int nb = (nc + 15) / 16;  // blocks of 16 candidates
      for (int blk = wk; blk < nb; blk += 4) {
        const int c = blk * 16 + col;  // this lane's candidate column
        const bool ok = c < nc;
        const int j = jl[ok ? c : 0];
        const float* pj = pv + (size_t)j * 3 * Bs;
        const float* qj = qv + (size_t)j * 3 * Bs;
        f32x4 acc[9];
#pragma unroll
        for (int q = 0; q < 9; ++q) acc[q] = f32x4{0.f, 0.f, 0.f, 0.f};
        // candidate values of step s: components b of (q_j | p_j) at k = 32 s + 8 row .. + 7
        const int steps = B / 16;
        auto load = [&](int s, float (&o)[3][8]) {
          const int k = 32 * min(s, steps - 1) + 8 * row;
          const float* src = k < B ? qj + k : pj + (k - B);
#pragma unroll
          for (int b = 0; b < 3; ++b) {
            const float4 u = *reinterpret_cast<const float4*>(src + b * Bs);
            const float4 v = *reinterpret_cast<const float4*>(src + b * Bs + 4);
            o[b][0] = u.x; o[b][1] = u.y; o[b][2] = u.z; o[b][3] = u.w;
            o[b][4] = v.x; o[b][5] = v.y; o[b][6] = v.z; o[b][7] = v.w;
          }
        };
        float nx[3][8];
        load(0, nx);
        for (int s = 0; s < steps; ++s) {
          Split8 sb[3];
#pragma unroll
          for (int b = 0; b < 3; ++b) sb[b] = split8(nx[b]);
          load(s + 1, nx);
          const __bf16* ta = tl + col * RP + 32 * s + 8 * row;
#pragma unroll
          for (int a = 0; a < 3; ++a) {
            const bf16x8 th = *reinterpret_cast<const bf16x8*>(ta + a * kGroup * RP);
            const bf16x8 tm = *reinterpret_cast<const bf16x8*>(ta + a * kGroup * RP + plane);
            const bf16x8 tw = *reinterpret_cast<const bf16x8*>(ta + a * kGroup * RP + 2 * plane);
            f32x4 w[3];
#pragma unroll
            for (int b = 0; b < 3; ++b) w[b] = f32x4{0.f, 0.f, 0.f, 0.f};
#define MBD_STEP(TP, DP)                                                             \
  _Pragma("unroll") for (int b = 0; b < 3; ++b) w[b] =                               \
      __builtin_amdgcn_mfma_f32_16x16x32_bf16(TP, sb[b].DP, w[b], 0, 0, 0)
            MBD_STEP(tw, h);
            MBD_STEP(th, l);
            MBD_STEP(tm, m);
            MBD_STEP(tm, h);
            MBD_STEP(th, m);
            MBD_STEP(th, h);
#undef MBD_STEP
#pragma unroll
            for (int b = 0; b < 3; ++b) acc[3 * a + b] += w[b];
          }
        }
        // the block's pairs (target 4 row + r, candidate c): D[i][j] sits in register
        // i % 4 of lane j + 16 (i / 4)
        const uint32_t msk = ok ? (uint32_t)ml[c] : 0u;
        const float* f = F + ((size_t)(c0 + (ok ? c : 0)) * kGroup + 4 * row) * kTensorWords;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if (!((msk >> (4 * row + r)) & 1u)) continue;
          const float rx = f[6 * r], ry = f[6 * r + 1], rz = f[6 * r + 2];
          const float Bk = f[6 * r + 3], c1 = f[6 * r + 4], c2 = f[6 * r + 5];
          const float m00 = acc[0][r], m11 = acc[4][r], m22 = acc[8][r];
          const float sxy = acc[1][r] + acc[3][r], sxz = acc[2][r] + acc[6][r],
                      syz = acc[5][r] + acc[7][r];
          const float X = m00 + m11 + m22;
          const float mx = (m00 + m00) * rx + sxy * ry + sxz * rz;
          const float my = sxy * rx + (m11 + m11) * ry + syz * rz;
          const float mz = sxz * rx + syz * ry + (m22 + m22) * rz;
          const float Y = 0.5f * (rx * mx + ry * my + rz * mz);
          const float sc = c1 * X - c2 * Y;
          G[r][0] -= (double)(sc * rx - Bk * mx);
          G[r][1] -= (double)(sc * ry - Bk * my);
          G[r][2] -= (double)(sc * rz - Bk * mz);
        }
      }
    }
    // sum over the 16 candidate lanes of each row, then over the wavefronts in order
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        double v = G[r][a];
        for (int off = 1; off < 16; off <<= 1) v += __shfl_xor(v, off);
        G[r][a] = v;
      }
    if (col == 0) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int a = 0; a < 3; ++a) red[wk][4 * row + r][a] = G[r][a];
    }
    __syncthreads();
    if (threadIdx.x < kGroup * 3) {
      const int t = threadIdx.x / 3, a = threadIdx.x % 3;
      double v = 0.0;
#pragma unroll
      for (int w = 0; w < 4; ++w) v += red[w][t][a];
      const int i = group * kGroup + t;
      if (i < geo.n) fsum[3 * (size_t)i + a] += v;
    }
  }  // groups of this work-group
}


// Replica method (eq. replica): E_i = sum over images n and atoms j with
// |R_j + n - R_i| < R_cut, except (j = i, n = 0), of f T(r) d_j, the damped bare tensor
// (A = f / r^3, B = 3 f / r^5). Float64, any B <= 8 right-hand sides. One work-group
// per target; its threads stride over the (image, source) pairs, and the partial
// fields are reduced in LDS. Displacements are formed from fractional coordinates.
template <int NB>
__global__ void __launch_bounds__(256)
k_replica(const Geometry geo, const int* __restrict__ perm, const double* __restrict__ frac,
          const int* __restrict__ images, const double* __restrict__ loc,
          const double* __restrict__ dv, double* __restrict__ Ed, int B) {
  __shared__ double red[256];
  const int s = blockIdx.x;
  const int n = geo.n;
  const int is = perm[s];
  const double fi0 = frac[3 * is], fi1 = frac[3 * is + 1], fi2 = frac[3 * is + 2];
  const double Si = loc[4 * s + 3];
  const double rc2 = geo.replica_cut * geo.replica_cut;
  double acc[NB][3];
#pragma unroll
  for (int b = 0; b < NB; ++b) acc[b][0] = acc[b][1] = acc[b][2] = 0.0;
  const long total = (long)geo.n_images * n;
  for (long q = threadIdx.x; q < total; q += 256) {
    const int im = (int)(q / n), j = (int)(q % n);
    const int jo = perm[j];
    const double u0 = frac[3 * jo] - fi0 + images[3 * im];
    const double u1 = frac[3 * jo + 1] - fi1 + images[3 * im + 1];
    const double u2 = frac[3 * jo + 2] - fi2 + images[3 * im + 2];
    const double rx = u0 * geo.A[0][0] + u1 * geo.A[1][0] + u2 * geo.A[2][0];
    const double ry = u0 * geo.A[0][1] + u1 * geo.A[1][1] + u2 * geo.A[2][1];
    const double rz = u0 * geo.A[0][2] + u1 * geo.A[1][2] + u2 * geo.A[2][2];
    const double r2 = rx * rx + ry * ry + rz * rz;
    if (r2 >= rc2 || (j == s && r2 < 1e-12)) continue;
    const double r = sqrt(r2);
    const double ir2 = 1.0 / r2, ir3 = ir2 / r;
    const double z = geo.damp_d * (r / (Si + loc[4 * j + 3]) - 1.0);
    const double f = 1.0 / (1.0 + exp(-z));
    const double A = f * ir3, Bk = 3.0 * f * ir3 * ir2;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      if (b >= B) break;
      const double d0 = dv[(j * 3 + 0) * B + b];
      const double d1 = dv[(j * 3 + 1) * B + b];
      const double d2 = dv[(j * 3 + 2) * B + b];
      const double rd = Bk * (rx * d0 + ry * d1 + rz * d2);
      acc[b][0] += A * d0 - rx * rd;
      acc[b][1] += A * d1 - ry * rd;
      acc[b][2] += A * d2 - rz * rd;
    }
  }
  for (int b = 0; b < NB && b < B; ++b)
    for (int a = 0; a < 3; ++a) {
      red[threadIdx.x] = acc[b][a];
      __syncthreads();
      for (int h = 128; h > 0; h >>= 1) {
        if (threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
        __syncthreads();
      }
      if (threadIdx.x == 0) Ed[((size_t)s * 3 + a) * B + b] = red[0];
      __syncthreads();
    }
}

template <typename R>
__global__ void k_count_pairs(const Geometry geo, const int* __restrict__ cell_start,
                              const int* __restrict__ scell, const R* __restrict__ loc,
                              unsigned long long* __restrict__ count) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= geo.n) return;
  const int c = scell[s];
  int cx, cy, cz;
  cell_coords(c, cx, cy, cz);
  const R xi = loc[4 * s], yi = loc[4 * s + 1], zi = loc[4 * s + 2];
  const R rp2 = (R)(geo.r_pair * geo.r_pair);
  unsigned long long cnt = 0;
  for (int oz = -geo.nr[2]; oz <= geo.nr[2]; ++oz) {
    int wz = ((cz + oz) % geo.nc[2] + geo.nc[2]) % geo.nc[2];
    for (int oy = -geo.nr[1]; oy <= geo.nr[1]; ++oy) {
      int wy = ((cy + oy) % geo.nc[1] + geo.nc[1]) % geo.nc[1];
      for (int ox = -geo.nr[0]; ox <= geo.nr[0]; ++ox) {
        int wx = ((cx + ox) % geo.nc[0] + geo.nc[0]) % geo.nc[0];
        const bool zero = (ox == 0 && oy == 0 && oz == 0);
        const int cc = cell_index(wx, wy, wz);
        for (int j = cell_start[cc]; j < cell_start[cc + 1]; ++j) {
          if (zero && j == s) continue;
          const R rx = loc[4 * j] - xi +
                       (R)(ox * geo.hv[0][0] + oy * geo.hv[1][0] + oz * geo.hv[2][0]);
          const R ry = loc[4 * j + 1] - yi +
                       (R)(ox * geo.hv[0][1] + oy * geo.hv[1][1] + oz * geo.hv[2][1]);
          const R rz = loc[4 * j + 2] - zi +
                       (R)(ox * geo.hv[0][2] + oy * geo.hv[1][2] + oz * geo.hv[2][2]);
          cnt += (rx * rx + ry * ry + rz * rz < rp2) ? 1 : 0;
        }
      }
    }
  }
  atomicAdd(count, cnt);
}

}  // namespace

template <typename R>
long long count_pairs(const Geometry& g, const SysBuffers& b, hipStream_t st) {
  unsigned long long* d = nullptr;
  unsigned long long h = 0;
  if (hipMalloc(&d, sizeof(h)) != hipSuccess) return -1;
  hipMemsetAsync(d, 0, sizeof(h), st);
  k_count_pairs<R><<<(g.n + 127) / 128, 128, 0, st>>>(g, b.cell_start, b.scell, (const R*)b.loc, d);
  hipMemcpyAsync(&h, d, sizeof(h), hipMemcpyDeviceToHost, st);
  hipStreamSynchronize(st);
  hipFree(d);
  return (long long)h;
}

template long long count_pairs<float>(const Geometry&, const SysBuffers&, hipStream_t);
template long long count_pairs<double>(const Geometry&, const SysBuffers&, hipStream_t);

// Parts the field of a list launch comes in (partial sums over disjoint candidate ranges,
// added by the gather): 1 for the vector list kernel and the neighbour list, otherwise
// what the plan sized the buffer for.
int pair_parts(const Geometry& g, const SysBuffers& b, int B) {
  if (B <= 8 || g.replica_cut > 0.0) return 1;
  const bool vec = b.pg_real == 4 && B >= 64 && g.pair_mode == 0;
  return vec ? 1 : b.ed_parts;
}

// Target subsets per wavefront of the vector list kernel (64 right-hand sides and more):
// g.pair_ns when set (1, 2 or 4); otherwise doubled (up to 4) while the launch would have
// fewer than 4096 wavefronts (4 per SIMD), so that small systems still fill the GPU.
int pair_subsets(const Geometry& g, int ngroups, int B) {
  if (g.pair_ns > 0) return std::min(4, g.pair_ns);
  int ns = 1;
  while (ns < 4 && (long)ngroups * B * ns / 64 < 4096) ns *= 2;
  return ns;
}

template <typename R>
void launch_pair(const Geometry& g, const SysBuffers& b, int B, hipStream_t st, bool reverse) {
  const R* loc = (const R*)b.loc;
  const R* dv = (const R*)b.dv;
  R* Ed = (R*)b.Ed;
  if (B <= 8) {
    // four wavefronts per target while that shortens the chain of a target's entries: with
    // one right-hand side a wavefront takes 64 entries a step, so a target (about 300) is
    // done in five and the exchange between wavefronts costs more than it saves. One and
    // four, us, float64: B = 1, 648 atoms 6.9 and 7.0, 1029 7.5 and 8.4, 3000 9.2 and 12.7;
    // B = 8, 648 atoms 16.2 and 12.3, 5184 56 and 51, 12288 108 and 109; float, B = 8, 8232
    // atoms 48 and 46
    const bool wide = g.n < (B == 1 ? 1024 : 8192);
    const int blocks = ((wide ? g.n : (g.n + 3) / 4) + 7) / 8 * 8;
#define MBD_NB(NBV)                                                                        \
    if (wide)                                                                              \
      k_pair_nbr<R, NBV, 4><<<blocks, 256, 0, st>>>(g, b.cell_start, b.scell, loc, b.nb_cap, \
          b.nb_count, b.nb_hdr, (const NbrAB<R>*)b.nb_ab, dv, Ed);                         \
    else                                                                                   \
      k_pair_nbr<R, NBV, 1><<<blocks, 256, 0, st>>>(g, b.cell_start, b.scell, loc, b.nb_cap, \
          b.nb_count, b.nb_hdr, (const NbrAB<R>*)b.nb_ab, dv, Ed)
    switch (B) {
      case 1: MBD_NB(1); break;
      case 2: MBD_NB(2); break;
      case 4: MBD_NB(4); break;
      default: MBD_NB(8); break;
    }
#undef MBD_NB
    return;
  }
  const int ngroups = (g.n + kGroup - 1) / kGroup;
  const int2* H = b.pg_hdr;
  const R* T = (const R*)b.pg_T;
  const int nparts = pair_parts(g, b, B);
  const dim3 grd(pair_grid_x(ngroups, nparts, 1, g.pair_blocks), nparts);
#define MBD_PM(NK, NT, NN)                                                                   \
  k_pair_mfma<R, NK, NT, NN><<<grd, 64 * nn * nk, 0, st>>>(g, H, T, (const R*)b.pg_zero,    \
                                                          b.pg_count, b.pg_cap, dv, Ed, B)
  if constexpr (sizeof(R) == 8) {
    // float64: always the matrix cores, up to 64 right-hand sides per wavefront, four
    // wavefronts per group (3000 atoms, B = 16, r_c = 7 A: 424 us a launch with one vector
    // lane per right-hand side and one work-group per group, 24 us here in 5 parts)
    const int nn = B <= 64 ? 1 : B / 64, nk = 4 / nn;
    switch (B) {
      case 16: MBD_PM(4, 1, 1); break;
      case 32: MBD_PM(4, 2, 1); break;
      case 64: MBD_PM(4, 4, 1); break;
      case 128: MBD_PM(2, 4, 2); break;
      default: MBD_PM(1, 4, 4); break;
    }
    return;
  } else {
    // one wavefront holds the whole block, four share a group's candidates (648 atoms,
    // B = 32: 298 us a launch of the vector kernel, 11 us here in 16 parts)
    if (B < 64) {
      const int nn = 1, nk = 4;
      if (B == 16) MBD_PM(4, 1, 1); else MBD_PM(4, 2, 1);
      return;
    }
    // 128 right-hand sides per wavefront, 64 when B = 64 or with pair_mode 2
    if (g.pair_mode == 1 || g.pair_mode == 2) {
      const bool wide = g.pair_mode == 1 && B % 128 == 0;
      const int slices = B / (wide ? 128 : 64);
      const float floor = reverse ? 0.f : 0x1p-104f;
      const dim3 sliced(pair_grid_x(ngroups, nparts, slices, g.pair_blocks), nparts, slices);
      if (wide)
        k_pair_split<8, 2><<<sliced, 256, 0, st>>>(g, H, (const float*)T, b.pg_count, b.pg_cap,
                                                   (const float*)dv, (float*)Ed, B, floor);
      else
        k_pair_split<4, 4><<<sliced, 256, 0, st>>>(g, H, (const float*)T, b.pg_count, b.pg_cap,
                                                   (const float*)dv, (float*)Ed, B, floor);
      return;
    }
#undef MBD_PM
    const int ns = pair_subsets(g, ngroups, B);
#define MBD_PL(NS, WP) \
  k_pair_list<R, NS, WP><<<grd.x, 64 * WP, 0, st>>>(g, H, T, b.pg_count, b.pg_cap, dv, Ed, B)
    switch (B * 16 + ns) {
      case 64 * 16 + 1: MBD_PL(1, 1); break;
      case 64 * 16 + 2: MBD_PL(2, 2); break;
      case 64 * 16 + 4: MBD_PL(4, 4); break;
      case 128 * 16 + 1: MBD_PL(1, 2); break;
      case 128 * 16 + 2: MBD_PL(2, 4); break;
      case 128 * 16 + 4: MBD_PL(4, 8); break;
      case 256 * 16 + 1: MBD_PL(1, 4); break;
      case 256 * 16 + 2: MBD_PL(2, 8); break;
      default: MBD_PL(4, 16); break;
    }
#undef MBD_PL
  }
}

template <typename R>
void launch_pair_build(const Geometry& g, const SysBuffers& b, bool count_only, hipStream_t st) {
  const int ngroups = (g.n + kGroup - 1) / kGroup;
  fill_int(b.pg_max, 0, 1, st);
#define MBD_PB(BT)                                                                        \
  k_pair_build<R, BT><<<ngroups, BT, 0, st>>>(                                            \
      g, b.cell_start, b.scell, (const R*)b.loc, count_only ? 0 : b.pg_cap, b.pg_hdr,     \
      (R*)b.pg_T, count_only ? nullptr : (R*)b.pg_F, b.pg_count, b.pg_max)
  // below four work-groups per CU a group's scan is a latency chain: four times the threads.
  // set_positions with 256 and 1024, us: 648 atoms, float, 134 and 98; 8232 atoms 247 and
  // 218; 15,798 atoms (988 groups) 367 and 324, in float64 417 and 400. 1024 threads leave 128
  // registers each, of which the tensors spill 36 to 39: with the force tensors as well,
  // float64, 3000 atoms, 275 and 219, 14,739 atoms 571 and 568, 15,798 atoms 563 and 615
  if (ngroups < 1024) MBD_PB(1024); else MBD_PB(256);
#undef MBD_PB
}

template <typename R>
void launch_nbr_build(const Geometry& g, const SysBuffers& b, int* maxcount, hipStream_t st) {
  k_nbr_build<R><<<(g.n + 3) / 4, 256, 0, st>>>(g, b.cell_start, b.scell, (const R*)b.loc,
                                               b.nb_cap, b.nb_hdr, (NbrAB<R>*)b.nb_ab,
                                               b.nb_count, maxcount);
}

template void launch_nbr_build<float>(const Geometry&, const SysBuffers&, int*, hipStream_t);
template void launch_nbr_build<double>(const Geometry&, const SysBuffers&, int*, hipStream_t);

template <typename R>
void launch_pair_force(const Geometry& g, const SysBuffers& b, int B, hipStream_t st) {
  const int ngroups = (g.n + kGroup - 1) / kGroup;
  const int nblk = (ngroups + 7) / 8 * 8;
  const int2* H = b.pg_hdr;
  const R* F = (const R*)b.pg_F;
  const R* p = (const R*)b.dv;
  const R* q = (const R*)b.dq;
  if constexpr (sizeof(R) == 4) {
    // matrix cores, with the matrix-core direct sum: four wavefronts per group and part
    if ((g.pair_mode == 1 || g.pair_mode == 2 || B < 64) && B % 16 == 0 && B <= 128) {
      // every group resident, whatever residency cap the direct sum runs with
      const size_t lds = force_lds(B);
      if (lds > 65536)  // B = 128: 76 KB, two work-groups a CU
        hipFuncSetAttribute(reinterpret_cast<const void*>(&k_pair_force_split),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      k_pair_force_split<<<dim3(nblk, b.fs_parts), 256, lds, st>>>(
          g, H, (const float*)F, b.pg_count, b.pg_cap, (const float*)p, (const float*)q,
          b.fsum + 3 * (size_t)g.n, B);
      return;
    }
  }
  // right-hand-side slices of 64 (or target subsets when B < 64), then target splits
  // over 1-4 wavefronts until the launch has 4096 wavefronts
  const int rs = B >= 64 ? B / 64 : 1;
  const int nsub = B >= 64 ? 1 : 64 / B;  // lane subsets: at most 16 / nsub wavefronts
  int tw = 1;
  while (tw < 4 && tw * nsub < 16 && tw * rs < 16 && (long)ngroups * tw * rs < 4096) tw *= 2;
#define MBD_PF(NS, TWV, RSV, TPV)                                                        \
  k_pair_force<R, NS, TWV, RSV, TPV><<<dim3(nblk, b.fs_parts), 64 * TWV * RSV, 0, st>>>( \
      g, H, F, b.pg_count, b.pg_cap, p, q, b.fsum + 3 * (size_t)g.n, B)
  // (float blocks of 16 and 32 never come here)
#define MBD_PF64(...) if constexpr (sizeof(R) == 8) MBD_PF(__VA_ARGS__)
  switch (B * 16 + tw) {
    case 4 * 16 + 1: MBD_PF(16, 1, 1, 1); break;
    case 8 * 16 + 1: MBD_PF(8, 1, 1, 2); break;
    case 8 * 16 + 2: MBD_PF(8, 2, 1, 1); break;
    case 16 * 16 + 1: MBD_PF64(4, 1, 1, 4); break;
    case 16 * 16 + 2: MBD_PF64(4, 2, 1, 2); break;
    case 16 * 16 + 4: MBD_PF64(4, 4, 1, 1); break;
    case 32 * 16 + 1: MBD_PF64(2, 1, 1, 8); break;
    case 32 * 16 + 2: MBD_PF64(2, 2, 1, 4); break;
    case 32 * 16 + 4: MBD_PF64(2, 4, 1, 2); break;
    case 64 * 16 + 1: MBD_PF(1, 1, 1, 8); break;
    case 64 * 16 + 2: MBD_PF(1, 2, 1, 8); break;
    case 64 * 16 + 4: MBD_PF(1, 4, 1, 4); break;
    case 128 * 16 + 1: MBD_PF(1, 1, 2, 8); break;
    case 128 * 16 + 2: MBD_PF(1, 2, 2, 8); break;
    case 128 * 16 + 4: MBD_PF(1, 4, 2, 4); break;
    case 256 * 16 + 1: MBD_PF(1, 1, 4, 8); break;
    case 256 * 16 + 2: MBD_PF(1, 2, 4, 8); break;
    default: MBD_PF(1, 4, 4, 4); break;
  }
#undef MBD_PF64
#undef MBD_PF
}

template void launch_pair_force<float>(const Geometry&, const SysBuffers&, int, hipStream_t);
template void launch_pair_force<double>(const Geometry&, const SysBuffers&, int, hipStream_t);


void launch_replica(const Geometry& g, const SysBuffers& b, int B, hipStream_t st) {
  const double* loc = (const double*)b.loc;
  const double* dv = (const double*)b.dv;
  double* Ed = (double*)b.Ed;
  switch (B) {
    case 1: k_replica<1><<<g.n, 256, 0, st>>>(g, b.perm, b.wpos, b.images, loc, dv, Ed, B); break;
    case 2: k_replica<2><<<g.n, 256, 0, st>>>(g, b.perm, b.wpos, b.images, loc, dv, Ed, B); break;
    case 4: k_replica<4><<<g.n, 256, 0, st>>>(g, b.perm, b.wpos, b.images, loc, dv, Ed, B); break;
    default: k_replica<8><<<g.n, 256, 0, st>>>(g, b.perm, b.wpos, b.images, loc, dv, Ed, B); break;
  }
}

template void launch_pair<float>(const Geometry&, const SysBuffers&, int, hipStream_t, bool);
template void launch_pair<double>(const Geometry&, const SysBuffers&, int, hipStream_t, bool);
template void launch_pair_build<float>(const Geometry&, const SysBuffers&, bool, hipStream_t);
template void launch_pair_build<double>(const Geometry&, const SysBuffers&, bool, hipStream_t);

}  // namespace mbd
