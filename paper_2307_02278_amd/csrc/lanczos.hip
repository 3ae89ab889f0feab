// Lanczos recurrence, Gauss quadrature and energy in double precision
// (eqs. hutch, dds, recurs2, sl3, sl4, plasmonic2; Algorithms 1 and 2).
//
// The Krylov vectors are kept unnormalized: w_0 = v (||v|| = 1), and with
// nrm_k = ||w_k||, y_k = w_k / nrm_k, l~_k = C w_k,
//   a_k     = (w_k . l~_k) / nrm_k^2
//   w_{k+1} = l~_k / nrm_k - a_k w_k / nrm_k - nrm_k w_{k-1} / nrm_{k-1}
// which is the three-term recurrence b_{k+1} y_{k+1} = l_k - a_k y_k - b_k y_{k-1}
// with b_{k+1} = nrm_{k+1}; the generalized dipoles of the next step are
// d = g * w_{k+1} (stored in the SPME precision). Every reduction over atoms is
// done in a fixed order (per-block partial sums, then one block per RHS).
#include <algorithm>

#include "common.h"
#include "mbd_math.h"

namespace mbd {

namespace {

// Block layout for [n][3][B] element-wise kernels: RB lanes over right-hand
// sides, 256 / RB rows over (atom, component); blockIdx.y selects the RHS group.
template <int RB>
struct RowLayout {
  static constexpr int ROWS = 256 / RB;
};

__device__ __forceinline__ void block_reduce_rows(double* red, int rb_lanes, int rows) {
  const int lane = threadIdx.x % rb_lanes;
  const int row = threadIdx.x / rb_lanes;
  for (int h = rows / 2; h > 0; h >>= 1) {
    if (row < h) red[threadIdx.x] += red[threadIdx.x + h * rb_lanes];
    __syncthreads();
  }
  (void)lane;
}

template <int RB>
__global__ void __launch_bounds__(256)
k_probes(int n, int B, int nb, int probe0, uint64_t zs, const int* __restrict__ perm,
         const double* __restrict__ g, double* __restrict__ w0, double* __restrict__ dtmp,
         float* __restrict__ df, int use_float) {
  constexpr int ROWS = 256 / RB;
  const int b = blockIdx.y * RB + threadIdx.x % RB;
  const int row0 = blockIdx.x * ROWS + threadIdx.x / RB;
  if (b >= B) return;
  const uint64_t D = 3ull * (uint64_t)n;
  const double inv = 1.0 / sqrt((double)D);
  for (int row = row0; row < 3 * n; row += gridDim.x * ROWS) {
    const int s = row / 3, a = row % 3;
    double v = 0.0;
    if (b < nb) {
      const uint64_t l = (uint64_t)(probe0 + b);
      const uint64_t idx = l * D + 3ull * (uint64_t)perm[s] + (uint64_t)a;
      const uint64_t h = splitmix_at(zs, idx);
      v = (h >> 63) ? -inv : inv;
    }
    const size_t o = (size_t)row * B + b;
    w0[o] = v;
    const double d = g[s] * v;
    if (use_float) df[o] = (float)d; else dtmp[o] = d;
  }
}

// Partial-sum slot of ||w_k||^2: two alternate, so that an update can still read the sums
// of w_k while other work-groups write those of w_{k+1}.
__host__ __device__ inline int norm_slot(int k) { return 1 + (k & 1); }

// Scalars of step k of probe l from the sums dot = w_k . l~_k and sq = ||w_k||^2. A probe
// ends when ||w_k|| <= 1e-12 of the scale of the step before: meff, the steps done, becomes
// k. (Another work-group of the same launch may already have stored that; a probe that
// ended in an earlier step has meff < k.)
struct StepScalars {
  double nk, ak;
  bool was, live;  // alive before the norm of this step was looked at, and after
};
__device__ __forceinline__ StepScalars step_scalars(int l, int k, int m, double dot, double sq,
                                                    const double* nrm, const double* a, int me) {
  StepScalars t;
  t.was = me >= k && (k > 0 || me > 0);
  t.nk = k > 0 ? sqrt(sq) : nrm[l * m];
  t.live = t.was;
  if (k > 0) {
    const double scale = fmax(fabs(a[l * m + k - 1]), nrm[l * m + k - 1]);
    if (!(t.nk > 1e-12 * scale)) t.live = false;
  }
  t.ak = dot / (t.nk * t.nk);
  return t;
}
__device__ __forceinline__ void store_scalars(const StepScalars& t, int l, int k, int m,
                                              double* nrm, double* a, int* meff,
                                              uint32_t* status) {
  if (!t.was) return;
  if (k > 0) nrm[l * m + k] = t.nk;
  if (!isfinite(t.nk) || (t.live && !isfinite(t.ak))) atomicOr(status, kErrNonfinite);
  if (t.live) a[l * m + k] = t.ak;
  else meff[l] = k;
}

// w_{k+1} from l~_k, w_k, w_{k-1}. With ng > 0 the scalars of step k are formed here, by
// every work-group alike from the ng + nu partial sums (work-group 0 stores them): for
// small systems that costs less than the separate launch it saves. With ng = 0 they were
// stored before.
template <int RB>
__global__ void __launch_bounds__(256)
k_update(int n, int B, int nb, int k, int m, int probe0, const double* __restrict__ lt,
         const double* __restrict__ wk, const double* __restrict__ wkm1, double* a, double* nrm,
         int* meff, const double* __restrict__ g, double* __restrict__ wn,
         double* __restrict__ dtmp, float* __restrict__ df, int use_float, int write_d,
         double* part, int ng, int nu, uint32_t* __restrict__ status) {
  constexpr int ROWS = 256 / RB;
  __shared__ double red[256], red2[256];
  const int lane = threadIdx.x % RB;
  const int b = blockIdx.y * RB + lane;
  const int row0 = blockIdx.x * ROWS + threadIdx.x / RB;
  double dot = 0.0, sq = 0.0;
  if (ng > 0) {
    if (b < B) {
#pragma unroll 8
      for (int i = threadIdx.x / RB; i < ng; i += ROWS) dot += part[(size_t)i * kPartSlots * B + b];
      if (k > 0)
#pragma unroll 8
        for (int i = threadIdx.x / RB; i < nu; i += ROWS)
          sq += part[((size_t)i * kPartSlots + norm_slot(k)) * B + b];
    }
    red[threadIdx.x] = dot;
    red2[threadIdx.x] = sq;
    __syncthreads();
    for (int h = ROWS / 2; h > 0; h >>= 1) {
      if (threadIdx.x / RB < h) {
        red[threadIdx.x] += red[threadIdx.x + h * RB];
        red2[threadIdx.x] += red2[threadIdx.x + h * RB];
      }
      __syncthreads();
    }
    dot = red[lane];
    sq = red2[lane];
    __syncthreads();
  }
  double ss = 0.0;
  if (b < B) {
    bool live = false;
    double c_l = 0.0, c_k = 0.0, c_km1 = 0.0;
    if (b < nb) {
      const int l = probe0 + b;
      double nk, ak;
      if (ng > 0) {
        const StepScalars t = step_scalars(l, k, m, dot, sq, nrm, a, meff[l]);
        nk = t.nk;
        ak = t.ak;
        live = t.live;
        if (blockIdx.x == 0 && threadIdx.x < RB) store_scalars(t, l, k, m, nrm, a, meff, status);
      } else {
        nk = nrm[l * m + k];
        ak = a[l * m + k];
        live = meff[l] > k;  // w_{k+1} is needed only while the probe has not broken down
      }
      c_l = 1.0 / nk;
      c_k = ak / nk;
      c_km1 = (k > 0) ? nk / nrm[l * m + k - 1] : 0.0;
    }
    for (int row = row0; row < 3 * n; row += gridDim.x * ROWS) {
      const size_t o = (size_t)row * B + b;
      double v = 0.0;
      if (live) {
        v = c_l * lt[o] - c_k * wk[o];
        if (k > 0) v -= c_km1 * wkm1[o];
      }
      wn[o] = v;
      ss += v * v;
      if (write_d) {
        const double d = g[row / 3] * v;
        if (use_float) df[o] = (float)d; else dtmp[o] = d;
      }
    }
  }
  red[threadIdx.x] = ss;
  __syncthreads();
  block_reduce_rows(red, RB, ROWS);
  if (threadIdx.x < RB && b < B)
    part[((size_t)blockIdx.x * kPartSlots + norm_slot(k + 1)) * B + b] = red[threadIdx.x];
}

// Dot products of w with earlier Krylov vectors for re-orthogonalization:
// coef[b][j] partials of (w . w_j) for j in [j0, j1), written to part slot 2.. via a
// separate pass per j (the count is small: 2 for LOCAL).
template <int RB>
__global__ void __launch_bounds__(256)
k_dot(int n, int B, const double* __restrict__ x, const double* __restrict__ y,
      double* __restrict__ part, int slot) {
  constexpr int ROWS = 256 / RB;
  __shared__ double red[256];
  const int lane = threadIdx.x % RB;
  const int b = blockIdx.y * RB + lane;
  const int row0 = blockIdx.x * ROWS + threadIdx.x / RB;
  double ss = 0.0;
  if (b < B)
    for (int row = row0; row < 3 * n; row += gridDim.x * ROWS) {
      const size_t o = (size_t)row * B + b;
      ss += x[o] * y[o];
    }
  red[threadIdx.x] = ss;
  __syncthreads();
  block_reduce_rows(red, RB, ROWS);
  if (threadIdx.x < RB && b < B) part[((size_t)blockIdx.x * kPartSlots + slot) * B + b] = red[threadIdx.x];
}

// Sum the nblk per-block partials of one slot for each RHS, in a fixed order.
__global__ void __launch_bounds__(256)
k_sum_slot(int B, int slot, int nblk, const double* __restrict__ part,
           double* __restrict__ out) {
  __shared__ double red[256];
  const int b = blockIdx.x;
  double s = 0.0;
  for (int k = threadIdx.x; k < nblk; k += 256) s += part[((size_t)k * kPartSlots + slot) * B + b];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[b] = red[0];
}

// w <- w - sum_j c_j w_j with c_j = (w . w_j) / nrm_j^2 for the listed j; then the
// norm partials and (optionally) the dipoles.
template <int RB>
__global__ void __launch_bounds__(256)
k_orth_apply(int n, int B, int nb, int m, int probe0, const double* __restrict__ W,
             size_t vstride, int j0, int j1, const double* __restrict__ dots,
             const double* __restrict__ nrm, const int* __restrict__ meff, int k,
             const double* __restrict__ g, double* __restrict__ w, double* __restrict__ dtmp,
             float* __restrict__ df, int use_float, double* __restrict__ part, int slot) {
  constexpr int ROWS = 256 / RB;
  __shared__ double red[256];
  const int lane = threadIdx.x % RB;
  const int b = blockIdx.y * RB + lane;
  const int row0 = blockIdx.x * ROWS + threadIdx.x / RB;
  double ss = 0.0;
  if (b < B) {
    double c[kMaxSteps < 64 ? kMaxSteps : 64];
    const int nj = j1 - j0;
    bool live = false;
    if (b < nb) {
      const int l = probe0 + b;
      live = meff[l] > k;
      for (int j = 0; j < nj; ++j) {
        const double nj2 = nrm[l * m + j0 + j];
        c[j] = dots[(size_t)j * B + b] / (nj2 * nj2);
      }
    }
    for (int row = row0; row < 3 * n; row += gridDim.x * ROWS) {
      const size_t o = (size_t)row * B + b;
      double v = w[o];
      if (live)
        for (int j = 0; j < nj; ++j) v -= c[j] * W[(size_t)(j0 + j) * vstride + o];
      else
        v = 0.0;
      w[o] = v;
      ss += v * v;
      const double d = g[row / 3] * v;
      if (use_float) df[o] = (float)d; else dtmp[o] = d;
    }
  }
  red[threadIdx.x] = ss;
  __syncthreads();
  block_reduce_rows(red, RB, ROWS);
  if (threadIdx.x < RB && b < B)
    part[((size_t)blockIdx.x * kPartSlots + slot) * B + b] = red[threadIdx.x];
}

// Scalars of step k, one work-group per right-hand side: the sums over the ng partials of
// a_k and the nu partials of ||w_k||^2 in a fixed order, then step_scalars.
__global__ void __launch_bounds__(256)
k_finish_step(int B, int nb, int k, int m, int probe0, int ng, int nu,
              const double* __restrict__ part, double* __restrict__ nrm,
              double* __restrict__ a, int* __restrict__ meff, uint32_t* __restrict__ status) {
  __shared__ double red[256], red2[256];
  const int b = blockIdx.x;
  double s = 0.0, s2 = 0.0;
  for (int i = threadIdx.x; i < ng; i += 256) s += part[(size_t)i * kPartSlots * B + b];
  if (k > 0)
    for (int i = threadIdx.x; i < nu; i += 256)
      s2 += part[((size_t)i * kPartSlots + norm_slot(k)) * B + b];
  red[threadIdx.x] = s;
  red2[threadIdx.x] = s2;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (threadIdx.x < h) {
      red[threadIdx.x] += red[threadIdx.x + h];
      red2[threadIdx.x] += red2[threadIdx.x + h];
    }
    __syncthreads();
  }
  if (threadIdx.x != 0 || b >= nb) return;
  const int l = probe0 + b;
  store_scalars(step_scalars(l, k, m, red[0], red2[0], nrm, a, meff[l]), l, k, m, nrm, a, meff,
                status);
}

__global__ void k_init_probe_scalars(int nb, int m, int probe0, double* __restrict__ nrm,
                                     double* __restrict__ a, int* __restrict__ meff) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= nb) return;
  const int l = probe0 + b;
  for (int k = 0; k < m; ++k) {
    nrm[l * m + k] = 0.0;
    a[l * m + k] = 0.0;
  }
  nrm[l * m] = 1.0;
  meff[l] = m;
}

// Deflation step of the implicit QR iteration, by a whole wavefront: drops converged
// trailing entries and finds the unreduced block lo..hi (hi = 0: done). e[k] counts as zero
// when |e[k]| <= eps (|d[k]| + |d[k+1]|); 64 planes are tested at a time, so the scan is no
// serial chain of LDS reads. Every lane returns the same lo and hi.
__device__ __forceinline__ void tridiag_block(const double* d, double* e, int& lo, int& hi) {
  const int lane = threadIdx.x & 63;
  const double eps = 2.220446049250313e-16;
  lo = 0;
  for (int base = (hi - 1) & ~63; hi > 0 && base >= 0;) {
    const int k = base + lane;
    const bool small = k < hi && fabs(e[k]) <= eps * (fabs(d[k]) + fabs(d[k + 1]));
    const unsigned long long m = __ballot(small);
    if (m == 0ull) {
      base -= 64;
      continue;
    }
    const int top = base + 63 - __clzll((long long)m);  // largest zero plane below hi
    if (top == hi - 1) {
      if (lane == 0) e[hi - 1] = 0.0;
      --hi;
      if (hi == base) base -= 64;
    } else {
      lo = top + 1;
      return;
    }
  }
}

// Gauss quadrature per probe from its tridiagonal (implicit QR, first-row tracking): one
// wavefront per probe, its working arrays in LDS. The rotations of a sweep are one serial
// chain, which every lane runs alike on the same values (its LDS writes coincide); the
// lanes share the scaling, the deflation tests and the final sum. For m = 50: 1222 us with
// hypot, two divisions and a serial deflation scan, 598 us here.
__global__ void __launch_bounds__(64)
k_tridiag(int m, int probe0, const double* __restrict__ a, const double* __restrict__ nrm,
          const int* __restrict__ meff, double* __restrict__ q, uint32_t* __restrict__ status) {
  __shared__ double d[kMaxSteps], e[kMaxSteps], z[kMaxSteps];
  const int l = probe0 + blockIdx.x;
  const int lane = threadIdx.x;
  const int n = meff[l];
  double big = 0.0;
  for (int k = lane; k < n; k += 64) {
    d[k] = a[l * m + k];
    e[k] = (k + 1 < n) ? nrm[l * m + k + 1] : 0.0;
    z[k] = (k == 0) ? 1.0 : 0.0;
    big = fmax(big, fmax(fabs(d[k]), fabs(e[k])));
  }
  for (int o = 1; o < 64; o <<= 1) big = fmax(big, __shfl_xor(big, o));
  const double sc = tridiag_scale(big);
  for (int k = lane; k < n; k += 64) {
    d[k] *= sc;
    e[k] *= sc;
  }
  __syncthreads();
  int hi = n - 1, iter = 0, ok = 1;
  while (true) {
    int lo;
    tridiag_block(d, e, lo, hi);
    __syncthreads();
    if (hi <= 0) break;
    if (++iter > 60 * n) {
      ok = 0;
      break;
    }
    double zk = z[lo];
    tridiag_sweep(d, e, lo, hi, [&](int k, double c, double s) {
      const double zn = z[k + 1];
      z[k] = c * zk - s * zn;
      zk = s * zk + c * zn;
    });
    z[hi] = zk;
    __syncthreads();
  }
  double v = 0.0;
  bool bad = false;  // a Ritz value <= 0
  for (int k = lane; k < n; k += 64) {
    const double th = d[k] / sc;
    bad |= k == 0 ? !(th > 0.0) : th <= 0.0;
    v += z[k] * z[k] * sqrt(th > 0.0 ? th : 0.0);
  }
  for (int o = 1; o < 64; o <<= 1) v += __shfl_xor(v, o);
  const bool neg = __any(bad);
  if (lane != 0) return;
  q[l] = v;
  if (!ok) atomicOr(status, kErrNoConverge);
  if (neg) atomicOr(status, kErrNotPosdef);
  if (!isfinite(v)) atomicOr(status, kErrNonfinite);
}

// E = 1/2 (3N / R) sum_l Q_l - 3/2 sum_i omega_i, summed in probe order.
__global__ void k_energy(int n, int R, const double* __restrict__ q,
                         const double* __restrict__ g, const double* __restrict__ om2,
                         double* __restrict__ out, double* __restrict__ sd_out,
                         uint32_t* __restrict__ status) {
  __shared__ double red[256];
  double so = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) so += sqrt(om2[i]);
  red[threadIdx.x] = so;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    double sq = 0.0;
    for (int l = 0; l < R; ++l) sq += q[l];
    const double E = 0.5 * (3.0 * n / R) * sq - 1.5 * red[0];
    out[0] = E;
    if (!isfinite(E)) atomicOr(status, kErrNonfinite);
    if (sd_out) {
      // spread of the R samples of the trace estimator (two passes, fixed order)
      const double mean = sq / R;
      double ss = 0.0;
      for (int l = 0; l < R; ++l) ss += (q[l] - mean) * (q[l] - mean);
      sd_out[0] = R > 1 ? 0.5 * (3.0 * n) * sqrt(ss / (R - 1)) / sqrt((double)R)
                        : __builtin_nan("");
    }
  }
  (void)g;
}

// Caller layout [nrhs][N][3] (caller atom order) <-> internal [n][3][B] (sorted), through
// LDS in tiles of kPackAtoms atoms x 32 right-hand sides: on the caller's side consecutive
// threads take an atom's consecutive components, on the internal side consecutive right-hand
// sides. Read or written straight from the internal order, every caller value is its own
// cache line (24k atoms x 128: 94 and 92 us a launch, 55 and 47 us here).
constexpr int kPackAtoms = 16;
constexpr int kPackRows = 3 * kPackAtoms;
__global__ void __launch_bounds__(256)
k_pack(int n, int nrhs, int B, const int* __restrict__ perm, const double* __restrict__ v,
       const double* __restrict__ g, double* __restrict__ w, double* __restrict__ dtmp,
       float* __restrict__ df, int use_float) {
  __shared__ double tile[32][kPackRows + 1];
  const int s0 = blockIdx.x * kPackAtoms, b0 = blockIdx.y * 32;
  const int rows = min(kPackRows, 3 * (n - s0)), nb = min(32, B - b0);
  for (int t = threadIdx.x; t < nb * kPackRows; t += 256) {
    const int r = t % kPackRows, b = t / kPackRows;
    if (r < rows)
      tile[b][r] = b0 + b < nrhs
                       ? v[((size_t)(b0 + b) * n + perm[s0 + r / 3]) * 3 + r % 3] : 0.0;
  }
  __syncthreads();
  for (int t = threadIdx.x; t < rows * nb; t += 256) {
    const int b = t % nb, r = t / nb;
    const double x = tile[b][r];
    const size_t o = ((size_t)3 * s0 + r) * B + b0 + b;
    w[o] = x;
    const double d = g[s0 + r / 3] * x;
    if (use_float) df[o] = (float)d; else dtmp[o] = d;
  }
}

__global__ void __launch_bounds__(256)
k_unpack(int n, int nrhs, int B, const int* __restrict__ perm, const double* __restrict__ lt,
         double* __restrict__ out) {
  __shared__ double tile[32][kPackRows + 1];
  const int s0 = blockIdx.x * kPackAtoms, b0 = blockIdx.y * 32;
  const int rows = min(kPackRows, 3 * (n - s0)), nb = min(32, nrhs - b0);
  for (int t = threadIdx.x; t < rows * nb; t += 256) {
    const int b = t % nb, r = t / nb;
    tile[b][r] = lt[((size_t)3 * s0 + r) * B + b0 + b];
  }
  __syncthreads();
  for (int t = threadIdx.x; t < nb * kPackRows; t += 256) {
    const int r = t % kPackRows, b = t / kPackRows;
    if (r < rows) out[((size_t)(b0 + b) * n + perm[s0 + r / 3]) * 3 + r % 3] = tile[b][r];
  }
}


// ---------------------------------------------------------------------------
// Forces: reverse sweep through the recurrence (derivative of the fixed-probe
// estimator). In terms of y_k = w_k / nrm_k, l_k = C y_k, b_k = nrm_k:
//   w_{k+1} = l_k - a_k y_k - b_k y_{k-1},  y_{k+1} = w_{k+1} / b_{k+1},  a_k = y_k . l_k.
// Going back from k = m-1 with the adjoints abar_k = dQ/da_k, bbar_k = dQ/db_k of the
// quadrature and ybar (adjoint of y):
//   wbar  = (ybar_{k+1} - (ybar_{k+1} . y_{k+1}) y_{k+1}) / b_{k+1} + bbar_{k+1} y_{k+1}
//   abar_k -= wbar . y_k,  bbar_k -= wbar . y_{k-1}
//   lbar_k = wbar + abar_k y_k
//   ybar_k += -a_k wbar + abar_k l_k + C lbar_k,  ybar_{k-1} += -b_k wbar
// and dQ/dR = sum_k lbar_k^T (dC/dR) y_k. l_k is rebuilt from the recurrence
// (l_k = w_{k+1} + a_k y_k + b_k y_{k-1}); the last one is the stored C w_{m-1}.
// Re-orthogonalization corrections are not differentiated.
// ---------------------------------------------------------------------------

// Per probe (one wavefront each): eigenvectors of its tridiagonal by the implicit
// symmetric QR iteration with Wilkinson shift, then the quadrature adjoint
// dQ/dT = U (F o c c^T) U^T, c = U^T e1, F_ij = 1 / (sqrt(theta_i) + sqrt(theta_j)).
// Every lane runs the rotation chain of a sweep alike (as in k_tridiag) and leaves the
// rotations in LDS; then each lane applies them to its own rows of U, one register carried
// from plane to plane. U is stored by columns, u[k ld + i] = U_ik, so the lanes' accesses
// are consecutive; up to kEigLds steps it stays in LDS (LDSU), else in tz. In the adjoint's
// O(m^3) sums the weights F_ij c_i c_j of one i are formed once, one j per lane.
constexpr int kEigLds = 64;
template <bool LDSU>
__global__ void __launch_bounds__(64)
k_tridiag_adjoint(int m, int probe0, const double* __restrict__ a,
                  const double* __restrict__ nrm, const int* __restrict__ meff,
                  double* __restrict__ tz, double* __restrict__ abar, double* __restrict__ bbar,
                  uint32_t* __restrict__ status) {
  __shared__ double d[kMaxSteps], e[kMaxSteps], cs[kMaxSteps], sn[kMaxSteps];
  __shared__ double ul[LDSU ? kEigLds * kEigLds : 1];
  const int b = blockIdx.x;
  const int lane = threadIdx.x;
  const int l = probe0 + b;
  const int n = meff[l];
  const int ld = LDSU ? kEigLds : m;
  double* u = LDSU ? ul : tz + (size_t)b * m * m;
  double* ab = abar + (size_t)b * m;
  double* bb = bbar + (size_t)b * m;
  double big = 0.0;
  for (int k = lane; k < m; k += 64) {
    ab[k] = 0.0;
    bb[k] = 0.0;
    if (k < n) {
      d[k] = a[l * m + k];
      e[k] = (k + 1 < n) ? nrm[l * m + k + 1] : 0.0;
      big = fmax(big, fmax(fabs(d[k]), fabs(e[k])));
    }
  }
  for (int o = 1; o < 64; o <<= 1) big = fmax(big, __shfl_xor(big, o));
  const double sc = tridiag_scale(big);
  for (int k = lane; k < n; k += 64) {
    d[k] *= sc;
    e[k] *= sc;
  }
  for (int i = lane; i < n; i += 64)
    for (int k = 0; k < n; ++k) u[(size_t)k * ld + i] = (i == k) ? 1.0 : 0.0;
  __syncthreads();
  int hi = n - 1, iter = 0;
  bool ok = true;
  while (true) {
    int lo;
    tridiag_block(d, e, lo, hi);
    __syncthreads();
    if (hi <= 0) break;
    if (++iter > 60 * n) {
      ok = false;
      break;
    }
    tridiag_sweep(d, e, lo, hi, [&](int k, double c, double s) {
      cs[k] = c;
      sn[k] = s;
    });
    __syncthreads();
    for (int i = lane; i < n; i += 64) {
      double uk = u[(size_t)lo * ld + i];
      for (int k = lo; k < hi; ++k) {
        const double un = u[(size_t)(k + 1) * ld + i], c = cs[k], s = sn[k];
        u[(size_t)k * ld + i] = c * uk - s * un;
        uk = s * uk + c * un;
      }
      u[(size_t)hi * ld + i] = uk;
    }
    __syncthreads();
  }
  if (!ok) {
    if (lane == 0) atomicOr(status, kErrNoConverge);
    return;
  }
  // eigenvalues d, eigenvectors in the columns of u; sqrt(theta) into cs, the weights of
  // one i into sn
  for (int k = lane; k < n; k += 64) {
    const double th = d[k] / sc;
    if (!(th > 0.0)) atomicOr(status, kErrNotPosdef);
    cs[k] = sqrt(th > 0.0 ? th : 0.0);
  }
  for (int k0 = 0; k0 < n; k0 += 64) {
    const int k = k0 + lane;
    const bool own = k < n;
    const int kr = own ? k : 0, km = kr > 0 ? kr - 1 : 0;
    double mkk = 0.0, mkm = 0.0;
    for (int i = 0; i < n; ++i) {
      __syncthreads();  // the previous weights have been read
      for (int j = lane; j < n; j += 64) {
        const double den = cs[i] + cs[j];
        sn[j] = (den > 0.0 ? 1.0 / den : 0.0) * u[(size_t)j * ld];  // c_j = U_0j
      }
      __syncthreads();
      double acc = 0.0;
      for (int j = 0; j < n; ++j) acc += sn[j] * u[(size_t)j * ld + kr];
      const double v = acc * u[(size_t)i * ld];
      mkk += u[(size_t)i * ld + kr] * v;
      mkm += u[(size_t)i * ld + km] * v;
    }
    if (own) {
      ab[k] = mkk;
      bb[k] = k > 0 ? 2.0 * mkm : 0.0;
    }
  }
}

// The reverse sweep keeps ybar_{k+1} as two addends, yn and the previous step's adjoint
// matvec lt = C lbar_{k+1}; both readers below add them up, so no pass writes the sum.
// Five dot products per right-hand side into partial slots 0..4:
//   ybar_{k+1}.w_{k+1}, ybar_{k+1}.w_k, ybar_{k+1}.w_{k-1}, w_{k+1}.w_k, w_{k+1}.w_{k-1}.
template <int RB>
__global__ void __launch_bounds__(256)
k_adj_dots(int n, int B, const double* __restrict__ yn, const double* __restrict__ lt,
           const double* __restrict__ wn, const double* __restrict__ wk, const double* __restrict__ wkm1, int has_km1,
           double* __restrict__ part) {
  constexpr int ROWS = 256 / RB;
  __shared__ double red[256];
  const int lane = threadIdx.x % RB;
  const int b = blockIdx.y * RB + lane;
  const int row0 = blockIdx.x * ROWS + threadIdx.x / RB;
  double s[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  if (b < B)
    for (int row = row0; row < 3 * n; row += gridDim.x * ROWS) {
      const size_t o = (size_t)row * B + b;
      const double y = yn[o] + lt[o], w1 = wn[o], w0 = wk[o];
      const double wm = has_km1 ? wkm1[o] : 0.0;
      s[0] += y * w1;
      s[1] += y * w0;
      s[2] += y * wm;
      s[3] += w1 * w0;
      s[4] += w1 * wm;
    }
  for (int q = 0; q < 5; ++q) {
    red[threadIdx.x] = s[q];
    __syncthreads();
    block_reduce_rows(red, RB, ROWS);
    if (threadIdx.x < RB && b < B)
      part[((size_t)blockIdx.x * kPartSlots + q) * B + b] = red[threadIdx.x];
    __syncthreads();
  }
}

// Per-probe scalars of step k, one work-group per right-hand side: the five dot sums over the
// nblk work-groups of k_adj_dots (none at k = m - 1: zeros), in a fixed order, then abar_k and
// bbar_k in place and the coefficients of the element-wise update:
//   c[0] ybar_{k+1} + c[1] w_{k+1} = wbar;  lbar = wbar + c[2] w_k;
//   l_k = w_{k+1} + c[3] w_k + c[4] w_{k-1} (k < m-1) or c[5] Lt (k = m-1);
//   ybar_k += c[6] wbar + c[7] l_k;  ybar_{k-1} = c[8] wbar;  q = g c[9] w_k.
__global__ void __launch_bounds__(256)
k_adj_scalars(int B, int nb, int k, int m, int probe0, int nblk,
              const double* __restrict__ part, const double* __restrict__ a,
              const double* __restrict__ nrm, const int* __restrict__ meff,
              double* __restrict__ abar, double* __restrict__ bbar, double* __restrict__ coef) {
  __shared__ double red[5][256];
  const int b = blockIdx.x;
  double s[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  for (int i = threadIdx.x; i < nblk; i += 256)
#pragma unroll
    for (int q = 0; q < 5; ++q) s[q] += part[((size_t)i * kPartSlots + q) * B + b];
#pragma unroll
  for (int q = 0; q < 5; ++q) red[q][threadIdx.x] = s[q];
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (threadIdx.x < h)
#pragma unroll
      for (int q = 0; q < 5; ++q) red[q][threadIdx.x] += red[q][threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x != 0) return;
  const double sums[5] = {red[0][0], red[1][0], red[2][0], red[3][0], red[4][0]};
  double* c = coef + (size_t)b * 16;
  for (int q = 0; q < 16; ++q) c[q] = 0.0;
  if (b >= nb) return;
  const int l = probe0 + b;
  const int me = meff[l];
  if (k >= me) return;
  const double nk = nrm[l * m + k];
  const double nkm1 = k > 0 ? nrm[l * m + k - 1] : 1.0;
  double c0 = 0.0, c1 = 0.0, wy_k = 0.0, wy_km1 = 0.0;
  if (k + 1 < me) {
    const double beta = nrm[l * m + k + 1];
    const double sa = sums[0] / beta;
    const double sb = sums[1] / nk;
    const double sc = k > 0 ? sums[2] / nkm1 : 0.0;
    const double sd = sums[3] / (beta * nk);
    const double se = k > 0 ? sums[4] / (beta * nkm1) : 0.0;
    const double al1 = 1.0 / beta;
    const double al2 = bbar[(size_t)b * m + k + 1] - sa / beta;
    c0 = al1;
    c1 = al2 / beta;
    wy_k = al1 * sb + al2 * sd;
    wy_km1 = al1 * sc + al2 * se;
  }
  const double ab = abar[(size_t)b * m + k] - wy_k;
  abar[(size_t)b * m + k] = ab;
  if (k > 0) bbar[(size_t)b * m + k] -= wy_km1;
  const double ak = a[l * m + k];
  c[0] = c0;
  c[1] = c1;
  c[2] = ab / nk;
  c[3] = ak / nk;
  c[4] = k > 0 ? nk / nkm1 : 0.0;
  c[5] = 1.0 / nk;
  c[6] = -ak;
  c[7] = ab;
  c[8] = -nk;
  c[9] = 1.0 / nk;
}

template <int RB>
__global__ void __launch_bounds__(256)
k_adj_update(int n, int B, int k, int m, const double* __restrict__ coef,
             const double* __restrict__ wn, const double* __restrict__ wk,
             const double* __restrict__ wkm1, const double* __restrict__ lt,
             const double* __restrict__ g, const double* __restrict__ yn, double* __restrict__ yc,
             double* __restrict__ yp, double* __restrict__ lbar, double* __restrict__ pd,
             float* __restrict__ pf, double* __restrict__ qd, float* __restrict__ qf,
             int use_float) {
  constexpr int ROWS = 256 / RB;
  const int lane = threadIdx.x % RB;
  const int b = blockIdx.y * RB + lane;
  const int row0 = blockIdx.x * ROWS + threadIdx.x / RB;
  if (b >= B) return;
  const double* c = coef + (size_t)b * 16;
  const double c0 = c[0], c1 = c[1], c2 = c[2], c3 = c[3], c4 = c[4], c5 = c[5], c6 = c[6],
               c7 = c[7], c8 = c[8], c9 = c[9];
  const bool last = (k + 1 == m);
  for (int row = row0; row < 3 * n; row += gridDim.x * ROWS) {
    const size_t o = (size_t)row * B + b;
    const double w0 = wk[o];
    double wbar = 0.0, lk;
    double y0 = 0.0;
    if (!last) {
      const double w1 = wn[o];
      wbar = c0 * (yn[o] + lt[o]) + c1 * w1;
      lk = w1 + c3 * w0 + (k > 0 ? c4 * wkm1[o] : 0.0);
      y0 = yc[o];
    } else {
      lk = c5 * lt[o];
    }
    const double lb = wbar + c2 * w0;
    yc[o] = y0 + (c6 * wbar + c7 * lk);
    if (k > 0) yp[o] = c8 * wbar;
    lbar[o] = lb;
    const double gs = g[row / 3];
    if (use_float) {
      pf[o] = (float)(gs * lb);
      qf[o] = (float)(gs * c9 * w0);
    } else {
      pd[o] = gs * lb;
      qd[o] = gs * c9 * w0;
    }
  }
}

__global__ void k_fill_double(double* __restrict__ p, double v, size_t count) {
  const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < count) p[t] = v;
}

// F = -dE/dR = -1/2 (3N / R) dsum/dR, back to caller order; dsum/dR is the sum of
// the reciprocal part and the direct (pair) parts of fsum.
__global__ void k_forces_finish(int n, int R, int parts, const int* __restrict__ perm,
                                const double* __restrict__ fsum, double* __restrict__ out) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n) return;
  const double sc = -0.5 * (3.0 * n / R);
  const int i = perm[s];
  for (int a = 0; a < 3; ++a) {
    double v = fsum[3 * (size_t)s + a];
    for (int q = 1; q <= parts; ++q) v += fsum[3 * ((size_t)q * n + s) + a];
    out[3 * i + a] = sc * v;
  }
}

inline int rb_for(int B) { return B >= 64 ? 64 : B; }

// Work-groups (and partial sums) of the row kernels along the rows: four rows per thread,
// up to kRedBlocks (96 atoms, B = 1: one instead of 1024).
inline int row_blocks(int n, int B) {
  const int rows = 4 * (256 / rb_for(B));
  return std::max(1, std::min(kRedBlocks, (3 * n + rows - 1) / rows));
}

}  // namespace

// ---------------------------------------------------------------------------
// Launch wrappers
// ---------------------------------------------------------------------------
#define MBD_RB_SWITCH(RBV, CALL)         \
  switch (RBV) {                         \
    case 1: { constexpr int RB = 1; CALL; } break;   \
    case 2: { constexpr int RB = 2; CALL; } break;   \
    case 4: { constexpr int RB = 4; CALL; } break;   \
    case 8: { constexpr int RB = 8; CALL; } break;   \
    case 16: { constexpr int RB = 16; CALL; } break; \
    case 32: { constexpr int RB = 32; CALL; } break; \
    default: { constexpr int RB = 64; CALL; } break; \
  }

void launch_probes(const Geometry& geo, const SysBuffers& b, int B, int nb, int probe0,
                   uint64_t seed, int system, bool use_float, hipStream_t st) {
  const uint64_t zs = splitmix_at(seed, (uint64_t)system);
  const int rb = rb_for(B);
  dim3 grd(row_blocks(geo.n, B), (B + rb - 1) / rb);
  MBD_RB_SWITCH(rb, (k_probes<RB><<<grd, 256, 0, st>>>(geo.n, B, nb, probe0, zs, b.perm, b.g,
                                                       b.W, (double*)b.dv, (float*)b.dv,
                                                       use_float ? 1 : 0)));
}

void launch_init_scalars(const SysBuffers& b, int nb, int m, int probe0, hipStream_t st) {
  k_init_probe_scalars<<<(nb + 63) / 64, 64, 0, st>>>(nb, m, probe0, b.b, b.a, b.meff);
}

void launch_update(const Geometry& geo, const SysBuffers& b, int B, int nb, int k, int m,
                   int probe0, bool use_float, bool write_d, int ng, uint32_t* status,
                   hipStream_t st) {
  const size_t vs = (size_t)geo.n * 3 * B;
  const int rb = rb_for(B);
  dim3 grd(row_blocks(geo.n, B), (B + rb - 1) / rb);
  const double* wk = b.W + (size_t)k * vs;
  const double* wkm1 = k > 0 ? b.W + (size_t)(k - 1) * vs : b.W;
  double* wn = b.W + (size_t)(k + 1) * vs;
  MBD_RB_SWITCH(rb, (k_update<RB><<<grd, 256, 0, st>>>(
                         geo.n, B, nb, k, m, probe0, b.Lt, wk, wkm1, b.a, b.b, b.meff, b.g, wn,
                         (double*)b.dv, (float*)b.dv, use_float ? 1 : 0, write_d ? 1 : 0,
                         b.part, ng, (int)grd.x, status)));
}

// Every work-group of k_update then reads the ng + nu partials of its right-hand sides. Up to
// 8 MB of L2 reads over the launch that takes no longer than the launch it saves. Energy of 30
// steps with the separate launch and without, us: 648 atoms, float, B = 32 (3.6 MB) 2342 and
// 2364; 1536 atoms, B = 16 (4.2 MB) 2385 and 2331; 3000 atoms, B = 16 (16 MB) 2751 and 2760,
// B = 32 (75 MB) 3381 and 3487; 3000 atoms, float64, B = 1 (14 KB) 2402 and 2333.
bool update_finishes(const Geometry& geo, int B, int ng) {
  const size_t nu = (size_t)row_blocks(geo.n, B);
  return (ng + nu) * sizeof(double) * B * nu <= ((size_t)8 << 20);
}

// Re-orthogonalize w_{k+1} against w_j for j in [j0, k] (classical Gram-Schmidt,
// in chunks of at most 64 earlier vectors).
void launch_reorth(const Geometry& geo, const SysBuffers& b, int B, int nb, int k, int m,
                   int probe0, int j0, bool use_float, hipStream_t st) {
  const size_t vs = (size_t)geo.n * 3 * B;
  const int rb = rb_for(B);
  dim3 grd(row_blocks(geo.n, B), (B + rb - 1) / rb);
  double* w = b.W + (size_t)(k + 1) * vs;
  for (int c0 = j0; c0 <= k; c0 += 64) {
    const int c1 = (k + 1 < c0 + 64) ? k + 1 : c0 + 64;
    for (int j = c0; j < c1; ++j) {
      MBD_RB_SWITCH(rb, (k_dot<RB><<<grd, 256, 0, st>>>(geo.n, B, w, b.W + (size_t)j * vs,
                                                        b.part, 3)));
      k_sum_slot<<<B, 256, 0, st>>>(B, 3, (int)grd.x, b.part, b.coef + (size_t)(j - c0) * B);
    }
    MBD_RB_SWITCH(rb, (k_orth_apply<RB><<<grd, 256, 0, st>>>(
                           geo.n, B, nb, m, probe0, b.W, vs, c0, c1, b.coef, b.b, b.meff, k,
                           b.g, w, (double*)b.dv, (float*)b.dv, use_float ? 1 : 0, b.part,
                           norm_slot(k + 1))));
  }
}

void launch_finish_step(const Geometry& geo, const SysBuffers& b, int B, int nb, int k, int m,
                        int probe0, int ng, uint32_t* status, hipStream_t st) {
  k_finish_step<<<nb, 256, 0, st>>>(B, nb, k, m, probe0, ng, row_blocks(geo.n, B), b.part, b.b,
                                    b.a, b.meff, status);
}

void launch_tridiag(const SysBuffers& b, int nb, int m, int probe0, uint32_t* status,
                    hipStream_t st) {
  k_tridiag<<<nb, 64, 0, st>>>(m, probe0, b.a, b.b, b.meff, b.q, status);
}

void launch_energy(const Geometry& geo, const SysBuffers& b, int R, double* energy_out,
                   double* sd_out, uint32_t* status, hipStream_t st) {
  k_energy<<<1, 256, 0, st>>>(geo.n, R, b.q, b.g, b.om2, energy_out, sd_out, status);
}


void fill_double(double* p, double v, size_t n, hipStream_t st) {
  if (n == 0) return;
  k_fill_double<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(p, v, n);
}

void launch_tridiag_adjoint(const SysBuffers& b, int nb, int m, int probe0, uint32_t* status,
                            hipStream_t st) {
  if (m <= kEigLds)
    k_tridiag_adjoint<true><<<nb, 64, 0, st>>>(m, probe0, b.a, b.b, b.meff, b.tz, b.abar,
                                               b.bbar, status);
  else
    k_tridiag_adjoint<false><<<nb, 64, 0, st>>>(m, probe0, b.a, b.b, b.meff, b.tz, b.abar,
                                                b.bbar, status);
}

// One reverse step k: dots, scalars and the element-wise update, which leaves lbar_k in
// b.lbar, g * lbar_k in b.dv and g * y_k in b.dq for the adjoint matvec and force terms.
// Three launches; with separate sums, fills and the matvec's accumulation it was eleven (651
// atoms, 16 right-hand sides: 37 us a step, 16 us now). b.Lt holds the forward sweep's last
// matvec at k = m - 1, and C lbar_{k+1} after that. No buffer has to start from zero: each
// one of the three ybar is written before its first read.
void launch_adjoint_step(const Geometry& geo, const SysBuffers& b, int B, int nb, int k, int m,
                         int probe0, bool use_float, hipStream_t st) {
  const size_t vs = (size_t)geo.n * 3 * B;
  const int rb = rb_for(B);
  dim3 grd(row_blocks(geo.n, B), (B + rb - 1) / rb);
  double* Y0 = b.ybar;
  double* yn = Y0 + (size_t)((k + 1) % 3) * vs;
  double* yc = Y0 + (size_t)(k % 3) * vs;
  double* yp = Y0 + (size_t)((k + 2) % 3) * vs;
  const double* wk = b.W + (size_t)k * vs;
  const double* wn = (k + 1 < m) ? b.W + (size_t)(k + 1) * vs : wk;
  const double* wkm1 = k > 0 ? b.W + (size_t)(k - 1) * vs : wk;
  if (k + 1 < m) {
    MBD_RB_SWITCH(rb, (k_adj_dots<RB><<<grd, 256, 0, st>>>(geo.n, B, yn, b.Lt, wn, wk, wkm1,
                                                           k > 0 ? 1 : 0, b.part)));
  }
  k_adj_scalars<<<B, 256, 0, st>>>(B, nb, k, m, probe0, k + 1 < m ? (int)grd.x : 0, b.part, b.a,
                                   b.b, b.meff, b.abar, b.bbar, b.adj);
  MBD_RB_SWITCH(rb, (k_adj_update<RB><<<grd, 256, 0, st>>>(
                         geo.n, B, k, m, b.adj, wn, wk, wkm1, b.Lt, b.g, yn, yc, yp, b.lbar,
                         (double*)b.dv, (float*)b.dv, (double*)b.dq, (float*)b.dq,
                         use_float ? 1 : 0)));
}

void launch_forces_finish(const Geometry& geo, const SysBuffers& b, int R, double* forces,
                          hipStream_t st) {
  k_forces_finish<<<(geo.n + 255) / 256, 256, 0, st>>>(geo.n, R, b.fs_parts, b.perm, b.fsum,
                                                           forces);
}

void launch_pack(const Geometry& geo, const SysBuffers& b, const double* v, int nrhs, int B,
                 bool use_float, hipStream_t st) {
  const dim3 grd((geo.n + kPackAtoms - 1) / kPackAtoms, (B + 31) / 32);
  k_pack<<<grd, 256, 0, st>>>(geo.n, nrhs, B, b.perm, v, b.g, b.W, (double*)b.dv, (float*)b.dv,
                              use_float ? 1 : 0);
}

void launch_unpack(const Geometry& geo, const SysBuffers& b, double* out, int nrhs, int B,
                   hipStream_t st) {
  const dim3 grd((geo.n + kPackAtoms - 1) / kPackAtoms, (nrhs + 31) / 32);
  k_unpack<<<grd, 256, 0, st>>>(geo.n, nrhs, B, b.perm, b.Lt, out);
}

}  // namespace mbd
