// Exact spectra of small S^z sectors (Sec. II: a sector of small dimension is
// diagonalised completely instead of being estimated stochastically).
//
// The dense float64 matrix of H on each sector basis (rank order) is built in
// the workspace and reduced to a symmetric tridiagonal matrix by Householder
// reflections applied from both sides, one column per step for all sectors at
// once (two launches per step, the trailing block split over row tiles so
// that large sectors spread over the chip); the eigenvalues of the
// tridiagonal matrix then come from bisection on Sturm counts, one
// workgroup per sector and one eigenvalue per thread.
#include <hip/hip_runtime.h>

#include <cmath>

#include "kpm_device.h"
#include "kpm_internal.h"

namespace kpm {

namespace {

// Sum over the workgroup, returned to every thread (fixed order).
__device__ __forceinline__ double ed_sum(double v, double* sh) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) sh[w] = v;
  __syncthreads();
  const double r = ((sh[0] + sh[1]) + sh[2]) + sh[3];
  __syncthreads();
  return r;
}

// Rows of H on a spin-s sector (digits d_i = s + m_i with sum n_up): diagonal
// sum_b J_b m_i m_j, S^+_i S^-_j and S^-_i S^+_j with amplitude
// J_b/2 sqrt(s(s+1) - m(m+1)) sqrt(s(s+1) - m'(m'-1)).  One row per thread.
__device__ void spin_rows(const EigProb& P, const EigArgs& a, const uint32_t* s_sites, const double* s_J,
                          double* A) {
  const int N = P.n_sites, two_s = P.two_s, B = two_s + 1, R1 = two_s * N + 1, D = P.dim;
  const double sv = 0.5 * two_s;
  const uint32_t* tab = a.tables + P.tab_off;
  for (int r = threadIdx.x; r < D; r += kThreads) {
    uint64_t dg = 0;
    uint32_t rem = (uint32_t)r;
    int left = P.n_up;
    for (int i = N - 1; i >= 0; --i) {
      int d = min(two_s, left);
      while (d > 0 && tab[(i * R1 + left) * B + d] > rem) --d;
      rem -= tab[(i * R1 + left) * B + d];
      dg |= (uint64_t)d << (4 * i);
      left -= d;
    }
    double diag = 0.0;
    for (int q = 0; q < P.n_bonds; ++q) {
      const int i = (int)(s_sites[q] & 0xFFu), j = (int)(s_sites[q] >> 8);
      const int di = (int)((dg >> (4 * i)) & 15u), dj = (int)((dg >> (4 * j)) & 15u);
      diag += s_J[q] * (di - sv) * (dj - sv);
      for (int w = 0; w < 2; ++w) {
        const int a1 = w == 0 ? i : j, a2 = w == 0 ? j : i;
        const int d1 = w == 0 ? di : dj, d2 = w == 0 ? dj : di;
        if (d1 >= two_s || d2 <= 0) continue;
        const double m1 = d1 - sv, m2 = d2 - sv;
        const double amp = 0.5 * s_J[q] * sqrt(sv * (sv + 1.0) - m1 * (m1 + 1.0)) *
                           sqrt(sv * (sv + 1.0) - m2 * (m2 - 1.0));
        const uint32_t c =
            spin_rank(dg + ((uint64_t)1 << (4 * a1)) - ((uint64_t)1 << (4 * a2)), N, P.n_up, R1, B, tab);
        if (c < (uint32_t)D) A[(int64_t)r * D + c] += amp;
        else if (a.err) atomicOr(a.err, 2);
      }
    }
    A[(int64_t)r * D + r] += diag;
  }
}

}  // namespace

// Dense H of every sector (one workgroup per sector, one row per thread).
__global__ __launch_bounds__(kThreads) void ed_build_kernel(const EigArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x;
  const EigProb P = a.probs[blockIdx.x];
  const int D = P.dim;
  uint32_t* sb = reinterpret_cast<uint32_t*>(smem);                       // [33 * 33]
  uint32_t* s_mask = sb + kBinomN * kBinomN;                               // [lds_bonds]
  double* s_J = reinterpret_cast<double*>(smem + a.o_bonds);              // [lds_bonds]
  for (int i = tid; i < kBinomN * kBinomN; i += kThreads) sb[i] = a.binom[i];
  for (int q = tid; q < P.n_bonds; q += kThreads) {
    s_mask[q] = a.bmask[P.bond_off + q];
    s_J[q] = a.J[P.bond_off + q];
  }
  double* A = a.mat + P.mat_off;
  for (int64_t i = tid; i < (int64_t)D * D; i += kThreads) A[i] = 0.0;
  __syncthreads();
  if (P.two_s > 1) {
    spin_rows(P, a, s_mask, s_J, A);
    return;
  }
  // s_i s_j = 1/4 for equal spins, -1/4 otherwise; unequal spins are
  // exchanged with amplitude J/2.
  for (int r = tid; r < D; r += kThreads) {
    const uint32_t s = unrank((uint32_t)r, P.n_sites, P.n_up, sb);
    double diag = 0.0;
    for (int q = 0; q < P.n_bonds; ++q) {
      const uint32_t m = s_mask[q];
      const uint32_t x = s & m;
      if (x == 0u || x == m) {
        diag += 0.25 * s_J[q];
      } else {
        diag -= 0.25 * s_J[q];
        const uint32_t c = word_rank(s ^ m, sb);
        if (c < (uint32_t)D) A[(int64_t)r * D + c] += 0.5 * s_J[q];
        else if (a.err) atomicOr(a.err, 2);
      }
    }
    A[(int64_t)r * D + r] += diag;
  }
}

// Householder step k, part 1 (one workgroup per active sector): the part of
// row k right of the diagonal, x, becomes alpha e_1 under I - 2 v v^T with
// v = (x - alpha e_1) / |x - alpha e_1|, alpha = -sign(x_0) |x|; d[k], e[k]
// are recorded.  A row that is already zero there keeps v = 0.  Step k - 1's
// update A' -= v w^T + w v^T (w = p - K v, K = v.p) has not reached the matrix
// yet: it is applied to row k here, and to the other rows in part 2, which
// reads the trailing block once a step for both.  v of step k lies in slot
// k & 1.
__global__ __launch_bounds__(kThreads) void ed_hh_vec_kernel(const EigArgs a, int k) {
  __shared__ double sh[4];
  __shared__ double x[kEdMaxDim];
  const EigProb P = a.probs[blockIdx.x];
  const int D = P.dim, n2 = D - k - 1;
  if (k + 2 >= D) return;
  const double* row = a.mat + P.mat_off + (int64_t)k * D + k;   // from the diagonal on
  double* v = a.hv + (k & 1) * a.vec_len + P.vec_off;
  double part = 0.0, diag = 0.0;
  if (k == 0) {
    if (threadIdx.x == 0) diag = row[0];
    for (int i = threadIdx.x; i < n2; i += kThreads) {
      x[i] = row[i + 1];
      part = fma(x[i], x[i], part);
    }
  } else {
    const double* u = a.hv + ((k - 1) & 1) * a.vec_len + P.vec_off;
    const double* pv = a.hp + P.vec_off;
    double* w = a.hw + P.vec_off;
    double kk = 0.0;
    for (int i = threadIdx.x; i <= n2; i += kThreads) kk = fma(u[i], pv[i], kk);
    const double K = ed_sum(kk, sh);
    const double u0 = u[0], w0 = fma(-K, u0, pv[0]);
    for (int i = threadIdx.x; i <= n2; i += kThreads) {
      const double wi = fma(-K, u[i], pv[i]);
      w[i] = wi;
      const double r = fma(-u0, wi, fma(-w0, u[i], row[i]));
      if (i == 0) {
        diag = r;
      } else {
        x[i - 1] = r;
        part = fma(r, r, part);
      }
    }
  }
  const double sigma = ed_sum(part, sh);   // x is whole behind its barriers
  const double x0 = x[0];
  const double tail = sigma - x0 * x0;
  if (threadIdx.x == 0) a.hd[P.vec_off + k] = diag;
  if (!(tail > 1e-300)) {
    if (threadIdx.x == 0) a.he[P.vec_off + k] = x0;
    for (int i = threadIdx.x; i < n2; i += kThreads) v[i] = 0.0;
    return;
  }
  const double alpha = -copysign(sqrt(sigma), x0);
  if (threadIdx.x == 0) a.he[P.vec_off + k] = alpha;
  const double v0 = x0 - alpha;
  const double inv = 1.0 / sqrt(tail + v0 * v0);
  for (int i = threadIdx.x; i < n2; i += kThreads) v[i] = (i == 0 ? v0 : x[i]) * inv;
}

// Part 2 (grid: active sectors x tiles of kEdRows rows): step k - 1's update of
// the trailing block A' (rows and columns k+1..D-1), then p = 2 A' v; each wave
// takes rows of the tile, its lanes stride over the row.  Bound by the block's
// read and write, and by the launches.  72 sectors of up to 1001 states:
// with the update in a launch of its own (a second read, and every
// workgroup's own sum of K) a step took 24.0 us, 18.1 now
// (18.8 with one row a wave and its own reads of the three vectors; four rows a
// wave are faster in the first steps, 50 us against 55, and slower in the
// last, 2.9 against 2.3).
__global__ __launch_bounds__(kThreads) void ed_hh_rows_kernel(const EigArgs a, int k) {
  const EigProb P = a.probs[blockIdx.x];
  const int D = P.dim, n2 = D - k - 1;
  if (k + 2 >= D) return;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const double* v = a.hv + (k & 1) * a.vec_len + P.vec_off;
  const double* u = a.hv + ((k + 1) & 1) * a.vec_len + P.vec_off + 1;   // of step k - 1, whose block had one row more
  const double* w = a.hw + P.vec_off + 1;
  double* pv = a.hp + P.vec_off;
  // a wave's rows together: the three vectors are read once for all of them
  constexpr int kWaves = kThreads / 64, kOwn = kEdRows / kWaves;
  const int i0 = blockIdx.y * kEdRows + wv;
  if (i0 >= n2) return;   // the same across the wave
  double* row[kOwn];
  double ui[kOwn], wi[kOwn], acc[kOwn];
#pragma unroll
  for (int q = 0; q < kOwn; ++q) {
    const int i = min(i0 + q * kWaves, n2 - 1);   // past the last row: not stored
    row[q] = a.mat + P.mat_off + (int64_t)(k + 1 + i) * D + (k + 1);
    ui[q] = k > 0 ? u[i] : 0.0;
    wi[q] = k > 0 ? w[i] : 0.0;
    acc[q] = 0.0;
  }
  for (int j = lane; j < n2; j += 64) {
    const double vj = v[j], uj = k > 0 ? u[j] : 0.0, wj = k > 0 ? w[j] : 0.0;
    double r[kOwn];
#pragma unroll
    for (int q = 0; q < kOwn; ++q)
      if (q == 0 || i0 + q * kWaves < n2) r[q] = row[q][j];
#pragma unroll
    for (int q = 0; q < kOwn; ++q) {
      if (q > 0 && i0 + q * kWaves >= n2) continue;
      if (k > 0) {
        r[q] = fma(-ui[q], wj, fma(-wi[q], uj, r[q]));
        row[q][j] = r[q];
      }
      acc[q] = fma(r[q], vj, acc[q]);
    }
  }
#pragma unroll
  for (int q = 0; q < kOwn; ++q) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc[q] += __shfl_down(acc[q], off, 64);
    if (lane == 0 && i0 + q * kWaves < n2) pv[i0 + q * kWaves] = 2.0 * acc[q];
  }
}

// Number of eigenvalues below x of the symmetric tridiagonal matrix (d, e):
// the negative pivots of the LDL^T factorisation of T - x (Sturm sequence),
// a pivot of magnitude below pivmin taken as -pivmin.
// 1/q from the hardware estimate and two Newton steps, r <- r (2 - q r)
// (each squares the relative error; |q| >= pivmin keeps q normal): the
// quotient below then differs from a correctly rounded division by a few ulps,
// which moves no pivot's sign except at the rounding level that bounds the
// bisection anyway, at a fraction of the divide sequence's latency on this
// serial chain.
__device__ __forceinline__ double sturm_recip(double q) {
  double r = __builtin_amdgcn_rcp(q);
  r = fma(r, fma(-q, r, 1.0), r);
  return fma(r, fma(-q, r, 1.0), r);
}

__device__ __forceinline__ int sturm_count(const double* d, const double* e2, int n, double x, double pivmin) {
  int cnt = 0;
  double q = d[0] - x;
  if (fabs(q) < pivmin) q = -pivmin;
  cnt += q < 0.0;
  for (int i = 1; i < n; ++i) {
    q = (d[i] - x) - e2[i - 1] * sturm_recip(q);
    if (fabs(q) < pivmin) q = -pivmin;
    cnt += q < 0.0;
  }
  return cnt;
}

// Last part, 1 (one workgroup per sector): the final 2 x 2 block, the
// squared off-diagonal, the Gershgorin interval and the pivot floor.
__global__ __launch_bounds__(kThreads) void ed_tri_kernel(const EigArgs a) {
  __shared__ double sh_lo[kThreads], sh_hi[kThreads], sh_e2[kThreads];
  const int tid = threadIdx.x;
  const EigProb P = a.probs[blockIdx.x];
  const int D = P.dim;
  double* d = a.hd + P.vec_off;
  double* e = a.he + P.vec_off;
  double* e2 = a.hp + P.vec_off;
  const double* A = a.mat + P.mat_off;
  if (tid == 0) {
    if (D >= 2) {
      double u0 = 0.0, u1 = 0.0, w0 = 0.0, w1 = 0.0;   // the last step's update
      if (D >= 3) {
        const double* u = a.hv + ((D - 3) & 1) * a.vec_len + P.vec_off;
        const double p0 = a.hp[P.vec_off], p1 = a.hp[P.vec_off + 1];
        u0 = u[0];
        u1 = u[1];
        const double K = fma(u1, p1, u0 * p0);
        w0 = fma(-K, u0, p0);
        w1 = fma(-K, u1, p1);
      }
      d[D - 2] = fma(-u0, w0, fma(-w0, u0, A[(int64_t)(D - 2) * D + (D - 2)]));
      d[D - 1] = fma(-u1, w1, fma(-w1, u1, A[(int64_t)(D - 1) * D + (D - 1)]));
      e[D - 2] = fma(-u1, w0, fma(-w1, u0, A[(int64_t)(D - 1) * D + (D - 2)]));
    } else {
      d[0] = A[0];
    }
    e[D - 1] = 0.0;
  }
  __syncthreads();
  double lo = INFINITY, hi = -INFINITY, m2 = 0.0;
  for (int i = tid; i < D; i += kThreads) {
    const double r = fabs(e[i]) + (i > 0 ? fabs(e[i - 1]) : 0.0);
    lo = fmin(lo, d[i] - r);
    hi = fmax(hi, d[i] + r);
    e2[i] = e[i] * e[i];
    m2 = fmax(m2, e2[i]);
  }
  sh_lo[tid] = lo;
  sh_hi[tid] = hi;
  sh_e2[tid] = m2;
  __syncthreads();
  for (int st = kThreads / 2; st > 0; st >>= 1) {
    if (tid < st) {
      sh_lo[tid] = fmin(sh_lo[tid], sh_lo[tid + st]);
      sh_hi[tid] = fmax(sh_hi[tid], sh_hi[tid + st]);
      sh_e2[tid] = fmax(sh_e2[tid], sh_e2[tid + st]);
    }
    __syncthreads();
  }
  if (tid == 0) {
    const double span = fmax(fabs(sh_lo[0]), fabs(sh_hi[0]));
    double* g = a.hv + P.vec_off;   // the Householder vectors are no longer needed
    g[0] = sh_lo[0] - 1e-14 * span - 1e-300;
    g[1] = sh_hi[0] + 1e-14 * span + 1e-300;
    g[2] = 1e-290 * fmax(1.0, sh_e2[0]);
    g[3] = span;
  }
}

// Last part, 2 (grid: sectors x tiles of 64 eigenvalue indices, one per
// thread): eigenvalue idx by bisection on the Sturm count from the Gershgorin
// interval, down to adjacent floating-point numbers or 1e-16 of the spectral
// radius; written in ascending order.
__global__ __launch_bounds__(64) void ed_bisect_kernel(const EigArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  const EigProb P = a.probs[blockIdx.x];
  const int D = P.dim;
  if ((int)blockIdx.y * 64 >= D) return;
  double* d = reinterpret_cast<double*>(smem);
  double* e2 = d + a.max_dim;
  for (int i = threadIdx.x; i < D; i += 64) {
    d[i] = a.hd[P.vec_off + i];
    e2[i] = a.hp[P.vec_off + i];
  }
  const double* g = a.hv + P.vec_off;
  const double g_lo = g[0], g_hi = g[1], pivmin = g[2], span = g[3];
  __syncthreads();
  const int idx = blockIdx.y * 64 + threadIdx.x;
  if (idx >= D) return;
  double x0 = g_lo, x1 = g_hi;
  for (int it = 0; it < 256; ++it) {
    const double mid = 0.5 * (x0 + x1);
    // adjacent numbers, or a width at the rounding level of the matrix
    if (!(mid > x0 && mid < x1) || x1 - x0 <= 1e-16 * span) break;
    if (sturm_count(d, e2, D, mid, pivmin) > idx) x1 = mid;
    else x0 = mid;
  }
  a.evals[(int64_t)P.out_row * a.ld + idx] = 0.5 * (x0 + x1);
}

// The sectors are sorted by descending dimension, so the sectors still active
// at step k (D > k + 2) are a prefix.
hipError_t launch_sector_eig(const EigArgs& a, const int* dims, int n_sectors, size_t lds_build,
                             size_t lds_finish, hipStream_t st) {
  if (n_sectors == 0) return hipSuccess;
  hipLaunchKernelGGL(ed_build_kernel, dim3(n_sectors), dim3(kThreads), lds_build, st, a);
  int active = n_sectors;
  for (int k = 0; k + 2 < dims[0]; ++k) {
    while (active > 0 && dims[active - 1] <= k + 2) --active;
    const int n2 = dims[0] - k - 1;
    const dim3 grid(active, (n2 + kEdRows - 1) / kEdRows);
    hipLaunchKernelGGL(ed_hh_vec_kernel, dim3(active), dim3(kThreads), 0, st, a, k);
    hipLaunchKernelGGL(ed_hh_rows_kernel, grid, dim3(kThreads), 0, st, a, k);
  }
  hipLaunchKernelGGL(ed_tri_kernel, dim3(n_sectors), dim3(kThreads), 0, st, a);
  hipLaunchKernelGGL(ed_bisect_kernel, dim3(n_sectors, (dims[0] + 63) / 64), dim3(64), lds_finish, st, a);
  return hipGetLastError();
}

}  // namespace kpm
