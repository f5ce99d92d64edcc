// Kernel damping, density-of-states weights and thermodynamics on the GPU
// (float64 throughout).
//
//  g_n      Jackson kernel, the paper's Eq. (8) with N_deg = M (the trailing
//           factor printed in Eq. (8) is a typesetting residue: with it the
//           coefficients would grow instead of damping).
//  gamma_k  weights of the Gauss-Chebyshev rule at x_k = cos(pi (k - 1/2)/Nt):
//           gamma_k = g_0 mu_0 + 2 sum_n g_n mu_n cos(n pi (k - 1/2)/Nt)
//           (Sec. II); the cosine argument is reduced exactly in integers,
//           n (2k - 1) mod 4 Nt, before scaling by pi / (2 Nt).
//  sums     per cluster and temperature, over its S^z sectors (weight 2 for
//           S^z > 0: the mirror sector, Sec. II) and the nodes, with Boltzmann
//           factors exp(-(E_k - E_ref)/T), E_k = a x_k + b, E_ref = the lowest
//           energy of the cluster at the point (no overflow; C, E, chi are
//           shift invariant, ln Z = ln(sum/Nt) - E_ref/T).  C is beta^2 times
//           the weighted variance of E taken about the mean (Eq. (2b)); chi is
//           beta times the variance of S_z (Eq. (3); <S_z> vanishes without a
//           field by the mirror sectors).
// Two kernels form the sums: the nodes of one sector at one temperature
// (sector_sums_kernel), then the sectors of a cluster at one point
// (points_kernel).  A field h only shifts a sector as a whole, by h S^z, so
// the points of a (T, h) grid share the sums over nodes of their temperature.
// Each reduction has a fixed order: results are reproducible.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "kpm_internal.h"

namespace kpm {

namespace {

// Lane sums and minima over aligned groups of kWidth lanes, the same in each.
template <int kWidth>
__device__ __forceinline__ double lanes_sum(double v) {
#pragma unroll
  for (int off = kWidth / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kWidth);
  return v;
}
template <int kWidth>
__device__ __forceinline__ double lanes_min(double v) {
#pragma unroll
  for (int off = kWidth / 2; off > 0; off >>= 1) v = fmin(v, __shfl_xor(v, off, kWidth));
  return v;
}

// cos(m pi / (2 Nt)) for the reduced argument m = n (2k - 1) mod 4 Nt.
__device__ __forceinline__ double reduced_cos(int64_t m, int64_t Nt) {
  return cos(M_PI * (double)m / (double)(2 * Nt));
}

// x_k for 1-based k.
__device__ __forceinline__ double node_x(int64_t k, int64_t Nt) {
  return cos(M_PI * ((double)k - 0.5) / (double)Nt);
}

// Problems that share the cosines of one wave of gamma_kernel, lambda_kernel:
// a cosine costs several times what one problem's term does, and four
// problems' sums still fit the registers of a fully occupied compute unit.
constexpr int kCosShare = 4;
constexpr int kOnePassSectors = 256;   // their sums in LDS, 10 kB


// Up to here each wave takes one problem: three workgroups a compute unit are in
// flight anyway, and the shared cosine would cost a chain of four problems' sums.
// T-only calls, four problems a wave against one: 75 us to 70 at 315 workgroups
// (5 problems, 500 moments), 69 to 68 at 572, 93 to 92 at 750; 85 to 87 at 800,
// 115 to 125 at 1250 and 128 to 179 at 3250.
constexpr int kGammaGroups = 768;

}  // namespace

__global__ __launch_bounds__(kThreads) void kernel_coef_kernel(int M, int kernel, double* g) {
  const int n = blockIdx.x * kThreads + threadIdx.x;
  if (n >= M) return;
  if (kernel == 0) {
    g[n] = 1.0;
    return;
  }
  const double q = M_PI / (double)(M + 1);
  g[n] = ((double)(M - n + 1) * cos(q * n) + sin(q * n) / tan(q)) / (double)(M + 1);
}

hipError_t launch_kernel_coef(int M, int kernel, double* g, hipStream_t st) {
  hipLaunchKernelGGL(kernel_coef_kernel, dim3((M + kThreads - 1) / kThreads), dim3(kThreads), 0, st,
                     M, kernel, g);
  return hipGetLastError();
}

// gamma[p][k-1] and E[p][k-1], one wave per pair of nodes k, Nt + 1 - k and
// kShare problems: cos(n theta) at the second node is (-1)^n that at the
// first, and n has the parity of its lane, so the second node costs a sign in
// the last sum.  k runs over the lower half of the spectrum, whose small
// weights keep the cosines of their own arguments.  Bound by float64 arithmetic,
// most of it the cosines': 13 sectors with 2000 moments took 200 us with a wave
// per node and problem.  Without damping the weights of the lowest nodes are
// small differences of large terms, so the sum is compensated
// (the Dot2 scheme of Ogita, Rump and Oishi, "Accurate sum and dot product",
// SIAM J. Sci. Comput. 26 (2005)): each product's rounding error from an fma,
// each addition's from TwoSum, carried in a second sum; lane l takes the terms
// n = l, l + 64, ... in order, then the lanes' (sum, error) pairs combine in a
// fixed butterfly (lane 0's order).  The reduced cosine argument
// m = n (2k - 1) mod 4 Nt advances by the reduced stride each term, exactly as
// the direct reduction gives it.
__device__ __forceinline__ void two_sum(double a, double b, double& s, double& e) {
#pragma clang fp contract(off)
  s = a + b;
  const double bb = s - a;
  e = (a - (s - bb)) + (b - bb);
}

template <int kShare>
__global__ __launch_bounds__(kThreads) void gamma_kernel(int n_probs, int M, int Nt,
                                                         const double* g, const double* mu,
                                                         const double* ab, double* gamma,
                                                         double* enode) {
#pragma clang fp contract(off)
  const int p0 = blockIdx.y * kShare;
  const int lane = threadIdx.x & 63;
  const int k = Nt - (blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6));
  if (2 * k < Nt + 1) return;   // k is the same across the wave
  const int np = min(kShare, n_probs - p0);
  const double* mp = mu + (int64_t)p0 * M;
  const int64_t period = 4 * (int64_t)Nt;
  const int64_t stride = (64 * (2 * (int64_t)k - 1)) % period;
  int64_t m = ((int64_t)lane * (2 * (int64_t)k - 1)) % period;
  double sum[kShare] = {}, err[kShare] = {};
  for (int n = lane; n < M; n += 64) {
    const double gn = g[n];
    const double cv = reduced_cos(m, Nt);
#pragma unroll
    for (int j = 0; j < kShare; ++j) {
      if (j >= np) break;
      const double cn = gn * mp[(int64_t)j * M + n] * (n == 0 ? 1.0 : 2.0);
      const double x = cn * cv;
      const double ex = fma(cn, cv, -x);
      double e;
      two_sum(sum[j], x, sum[j], e);
      err[j] += e + ex;
    }
    m += stride;
    if (m >= period) m -= period;
  }
#pragma unroll
  for (int j = 0; j < kShare; ++j) {
    if (j >= np) break;
    double v = sum[j], r = err[j];
    double vo = lane & 1 ? -v : v, ro = lane & 1 ? -r : r;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      const double v2 = __shfl_xor(v, off, 64), r2 = __shfl_xor(r, off, 64);
      const double vo2 = __shfl_xor(vo, off, 64), ro2 = __shfl_xor(ro, off, 64);
      double e;
      two_sum(v, v2, v, e);
      r += r2 + e;
      two_sum(vo, vo2, vo, e);
      ro += ro2 + e;
    }
    const int p = p0 + j;
    const double A = ab[2 * p], B = ab[2 * p + 1];
    if (lane == 0) {
      gamma[(int64_t)p * Nt + (k - 1)] = v + r;
      enode[(int64_t)p * Nt + (k - 1)] = fma(A, node_x(k, Nt), B);
    }
    const int ko = Nt + 1 - k;
    if (lane == 1 && ko != k) {
      gamma[(int64_t)p * Nt + (ko - 1)] = vo + ro;
      enode[(int64_t)p * Nt + (ko - 1)] = fma(A, node_x(ko, Nt), B);
    }
  }
}

hipError_t launch_gamma(int n_probs, int M, int n_nodes, const double* g, const double* mu,
                        const double* ab, double* gamma, double* enode, hipStream_t st) {
  constexpr int kPairsPerGroup = kThreads / 64;
  const unsigned groups = ((n_nodes + 1) / 2 + kPairsPerGroup - 1) / kPairsPerGroup;
  if ((int64_t)groups * n_probs <= kGammaGroups)
    hipLaunchKernelGGL(gamma_kernel<1>, dim3(groups, n_probs), dim3(kThreads), 0, st, n_probs, M,
                       n_nodes, g, mu, ab, gamma, enode);
  else
    hipLaunchKernelGGL(gamma_kernel<kCosShare>, dim3(groups, (n_probs + kCosShare - 1) / kCosShare),
                       dim3(kThreads), 0, st, n_probs, M, n_nodes, g, mu, ab, gamma, enode);
  return hipGetLastError();
}

// same[t] = the first point of t0 .. t with the bits of T[t]: one wave a point.
__global__ __launch_bounds__(kThreads) void same_T_kernel(const ThermoArgs a) {
  const int lane = threadIdx.x & 63;
  const int t = a.t0 + blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
  if (t >= a.t1) return;   // t is the same across the wave
  const int64_t* T = reinterpret_cast<const int64_t*>(a.T);
  const int64_t own = T[t];
  int first = t;
  for (int i0 = a.t0; i0 < t; i0 += 64) {
    const int i = i0 + lane;
    const unsigned long long hit = __ballot(i < t && T[i] == own);
    if (hit) {
      first = i0 + __ffsll(hit) - 1;
      break;
    }
  }
  if (lane == 0) a.same[t - a.t0] = first;
}

// Sums over the nodes (or exact levels) of sector p at point t's temperature, in
// a wave.  One exponential a node and pass; every shift of the whole sector (its
// lowest energy against the cluster's, the field's h S^z and its mirror) is one
// factor in point_sums.  The second pass takes the energies about the sector's
// mean, as the variance needs them.
__device__ __forceinline__ SectorSums sector_sums(const ThermoArgs& a, int p, int t, int lane) {
  const int ned = a.ed_count ? a.ed_count[p] : 0;
  const int items = ned > 0 ? ned : a.n_nodes;
  const double* en = ned > 0 ? a.evals + (int64_t)p * a.evals_ld : a.enode + (int64_t)p * a.n_nodes;
  const double* gam = ned > 0 ? nullptr : a.gamma + (int64_t)p * a.n_nodes;
  const double level = (double)a.n_nodes;   // an exact level weighs Nt nodes
  const double beta = 1.0 / a.T[t];

  double lo = INFINITY, hi = -INFINITY;
  for (int i = lane; i < items; i += 64) {
    const double E = en[i];
    lo = fmin(lo, E);
    hi = fmax(hi, E);
  }
  lo = lanes_min<64>(lo);
  hi = -lanes_min<64>(-hi);
  double s0 = 0.0, s1 = 0.0;
  for (int i = lane; i < items; i += 64) {
    const double d = en[i] - lo;
    const double w = (gam ? gam[i] : level) * exp(-beta * d);
    s0 += w;
    s1 = fma(w, d, s1);
  }
  s0 = lanes_sum<64>(s0);
  s1 = lanes_sum<64>(s1);
  // any centre gives the same variance; an improper density's mean may lie outside
  double c = lo + s1 / s0;
  if (!(c >= lo)) c = lo;
  if (c > hi) c = hi;
  double r1 = 0.0, v = 0.0;
  for (int i = lane; i < items; i += 64) {
    const double E = en[i];
    const double w = (gam ? gam[i] : level) * exp(-beta * (E - lo));
    const double d = E - c;
    r1 = fma(w, d, r1);
    v = fma(w, d * d, v);
  }
  r1 = lanes_sum<64>(r1);
  v = lanes_sum<64>(v);
  return SectorSums{lo, s0, c, r1, v};
}

// One point (T, h) of a cluster in 16 lanes, its sectors over the lanes, their
// sums from of(list position, sector).  The sector S^z = m keeps its zero-field
// DOS and every energy moves by h m (h = g mu_B B); a sector with S^z > 0 stands
// for m = +S^z and its mirror m = -S^z.  With d = E - c and D = c + h m - <E> the
// centred sum of squares is sum w (d + D)^2 = v + D (2 s1 + D s0) in each sector,
// with no cancellation.
template <typename F>
__device__ __forceinline__ void point_sums(const ThermoArgs& a, int t, int cl, int sub, F&& of) {
  const int q0 = a.cl_start[cl], q1 = a.cl_start[cl + 1];
  const double beta = 1.0 / a.T[t];
  const double hf = a.h ? a.h[t] : 0.0;

  double emin = INFINITY;
  for (int q = q0 + sub; q < q1; q += 16) {
    const int p = a.cl_list[q];
    const ThermoProb P = a.tp[p];
    const double lo = of(q, p).lo;
    emin = fmin(emin, fma(hf, P.sz, lo));
    if (P.weight > 1.0) emin = fmin(emin, fma(-hf, P.sz, lo));
  }
  const double eref = lanes_min<16>(emin);

  double S0 = 0.0, S1 = 0.0, S2 = 0.0;
  for (int q = q0 + sub; q < q1; q += 16) {
    const int p = a.cl_list[q];
    const ThermoProb P = a.tp[p];
    const SectorSums s = of(q, p);
    const double hm = hf * P.sz;
    const double fu = exp(-beta * ((s.lo + hm) - eref));
    const double fd = P.weight > 1.0 ? exp(-beta * ((s.lo - hm) - eref)) : 0.0;
    S0 += fu * s.s0 + fd * s.s0;
    S1 += fu * fma(s.s0, s.c + hm, s.s1);
    if (P.weight > 1.0) S1 += fd * fma(s.s0, s.c - hm, s.s1);
    S2 += (fu * s.s0 - fd * s.s0) * P.sz;
  }
  S0 = lanes_sum<16>(S0);
  const double Ebar = lanes_sum<16>(S1) / S0;
  const double Mbar = lanes_sum<16>(S2) / S0;

  double ve = 0.0, vm = 0.0;
  for (int q = q0 + sub; q < q1; q += 16) {
    const int p = a.cl_list[q];
    const ThermoProb P = a.tp[p];
    const SectorSums s = of(q, p);
    const int nm = P.weight > 1.0 ? 2 : 1;
    for (int j = 0; j < nm; ++j) {
      const double m = j == 0 ? P.sz : -P.sz;
      const double hm = hf * m;
      const double f = exp(-beta * ((s.lo + hm) - eref));
      const double D = (s.c + hm) - Ebar, dm = m - Mbar;
      ve = fma(f, fma(D, fma(D, s.s0, 2.0 * s.s1), s.v), ve);
      vm = fma(f * s.s0, dm * dm, vm);
    }
  }
  const double VarE = lanes_sum<16>(ve) / S0;
  const double VarM = lanes_sum<16>(vm) / S0;

  if (sub == 0) {
    const int64_t o = (int64_t)cl * a.n_T + t;
    a.lnZ[o] = (S0 > 0.0 ? log(S0 / (double)a.n_nodes) : NAN) - beta * eref;
    a.E[o] = Ebar;
    a.C[o] = beta * beta * VarE;
    a.chi[o] = beta * VarM;
    if (a.mag) a.mag[o] = Mbar;
    if (a.znonpos) a.znonpos[o] = S0 > 0.0 ? 0 : 1;
    if (a.stats) {
      double* st = a.stats + o * 6;
      st[0] = S0;
      st[1] = Ebar;
      st[2] = VarE;
      st[3] = VarM;
      st[4] = eref;
      st[5] = beta;
    }
  }
}

// Sector by temperature, in a wave: four temperatures of a sector share the
// cached node energies and weights.  200 temperatures of 13 sectors with 2000
// nodes, each at 40 fields: the sums of all 8000 points took 3.35 ms with the
// nodes' cosine and four exponentials in each point.
__global__ __launch_bounds__(kThreads) void sector_sums_kernel(const ThermoArgs a) {
  const int lane = threadIdx.x & 63;
  const int t = a.t0 + blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
  const int p = blockIdx.y;
  if (t >= a.t1 || (a.h && a.same[t - a.t0] != t)) return;   // the same across the wave
  const SectorSums s = sector_sums(a, p, t, lane);
  if (lane == 0) a.sums[(int64_t)p * (a.t1 - a.t0) + (t - a.t0)] = s;
}

__global__ __launch_bounds__(kThreads) void points_kernel(const ThermoArgs a) {
  const int t = a.t0 + blockIdx.x * (kThreads / 16) + (threadIdx.x >> 4);
  if (t >= a.t1) return;   // the same across the 16 lanes
  const SectorSums* sums = a.sums + ((a.h ? a.same[t - a.t0] : t) - a.t0);
  const int64_t ld = a.t1 - a.t0;
  point_sums(a, t, blockIdx.y, threadIdx.x & 15, [&](int, int p) { return sums[p * ld]; });
}

// A point of a cluster per workgroup, its sectors' sums over the waves and then
// in LDS: the same sums in the same order, in one launch and without the look for
// equal temperatures.  Small calls are bound by launches: 16 temperatures by 8
// fields of 8 sites with 64 nodes 72 us, with the three kernels 100.
__global__ __launch_bounds__(1024) void one_pass_kernel(const ThermoArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  SectorSums* sums = reinterpret_cast<SectorSums*>(smem);
  const int t = blockIdx.x, cl = blockIdx.y, lane = threadIdx.x & 63;
  const int q0 = a.cl_start[cl], q1 = a.cl_start[cl + 1];
  for (int q = q0 + (threadIdx.x >> 6); q < q1; q += blockDim.x >> 6) {
    const SectorSums s = sector_sums(a, a.cl_list[q], t, lane);
    if (lane == 0) sums[q - q0] = s;
  }
  __syncthreads();
  if (threadIdx.x < 16) point_sums(a, t, cl, threadIdx.x, [&](int q, int) { return sums[q - q0]; });
}

// Points per chunk: the sums of a chunk stay under 64 MB wherever 64 points do
// (a point's temperature is looked for within its chunk only).  0: the one-pass
// kernel, which evaluates the nodes at every point.  With fields, up to 2e6 of
// them: 0.7e6 91 us to 85, 1.2e6 118 to 100, 2.0e6 152 to 128 and 94 to 93; above,
// 89 to 96 at 2.1e6 and 92 to 123 at 2.6e6, where temperatures repeat 8 and 40
// times.  Without, where it saves one launch of 2 us and nothing repeats, up to
// 250,000: 62 to 59 at 6e4 and 1e5, 71 to 68 at 2.3e5; 126 to 132 at 4.2e5.
int thermo_chunk(int n_probs, int n_T, int n_nodes, int max_sectors, bool field) {
  const double nodes = (double)n_probs * n_T * n_nodes;
  if (max_sectors <= kOnePassSectors && nodes <= (field ? 2000000 : 250000)) return 0;
  const int64_t fit = (int64_t)(64 << 20) / ((int64_t)n_probs * sizeof(SectorSums));
  return (int)std::min<int64_t>(n_T, std::min<int64_t>(std::max<int64_t>(fit, 64), 16384));
}

hipError_t launch_thermo(ThermoArgs a, hipStream_t st) {
  if (a.chunk == 0) {
    const int waves = std::max(1, std::min(a.max_sectors, 16));
    hipLaunchKernelGGL(one_pass_kernel, dim3(a.n_T, a.n_clusters), dim3(64 * waves),
                       a.max_sectors * sizeof(SectorSums), st, a);
    return hipGetLastError();
  }
  for (a.t0 = 0; a.t0 < a.n_T; a.t0 = a.t1) {
    a.t1 = a.t0 + std::min(a.chunk, a.n_T - a.t0);
    const int n = a.t1 - a.t0, waves = kThreads / 64, points = kThreads / 16;
    const dim3 gw((n + waves - 1) / waves), gs(gw.x, a.n_probs), gp((n + points - 1) / points, a.n_clusters);
    if (a.h) {
      hipLaunchKernelGGL(same_T_kernel, gw, dim3(kThreads), 0, st, a);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(sector_sums_kernel, gs, dim3(kThreads), 0, st, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(points_kernel, gp, dim3(kThreads), 0, st, a);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// dL/dgamma at every node: for L = sum wC C + wchi chi,
//   dC/dgamma_k  = beta^2 W e_k ((E_k - Ebar)^2 - Var) / S0,
//   dchi/dgamma_k = beta W e_k (m^2 - <m^2>) / S0,   e_k = exp(-beta (E_k - E_ref)).
__global__ __launch_bounds__(kThreads) void node_adj_kernel(const ThermoVjpArgs a) {
  const int p = blockIdx.y;
  const int k = blockIdx.x * kThreads + threadIdx.x + 1;
  if (k > a.n_nodes) return;
  const ThermoProb P = a.tp[p];
  const double E = a.enode[(int64_t)p * a.n_nodes + (k - 1)];
  const double m2 = P.sz * P.sz;
  double acc = 0.0;
  for (int t = 0; t < a.n_T; ++t) {
    const int64_t o = (int64_t)P.cluster * a.n_T + t;
    const double* st = a.stats + o * 6;
    const double S0 = st[0], Ebar = st[1], Var = st[2], m2bar = st[3], eref = st[4], beta = st[5];
    const double e = P.weight * exp(-beta * (E - eref)) / S0;
    const double d = E - Ebar;
    acc += a.wC[o] * beta * beta * e * (d * d - Var) + a.wchi[o] * beta * e * (m2 - m2bar);
  }
  a.node_adj[(int64_t)p * a.n_nodes + (k - 1)] = acc;
}

// lambda_n = g_n (2 - delta_n0) sum_k node_adj_k cos(n pi (k - 1/2)/Nt): one
// wave per n and kCosShare problems, the nodes over the lanes, the reduced
// cosine argument advanced as in gamma_kernel.  7 sectors with 80 moments took
// 59 us with a thread per n that reduced every argument by a 64-bit division.
__global__ __launch_bounds__(kThreads) void lambda_kernel(const ThermoVjpArgs a) {
  const int p0 = blockIdx.y * kCosShare;
  const int lane = threadIdx.x & 63;
  const int n = blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
  if (n >= a.M) return;   // n is the same across the wave
  const int np = min(kCosShare, a.n_probs - p0);
  const int Nt = a.n_nodes;
  const double* adj = a.node_adj + (int64_t)p0 * Nt;
  const int64_t period = 4 * (int64_t)Nt;
  const int64_t stride = (128 * (int64_t)n) % period;
  int64_t m = ((2 * (int64_t)lane + 1) * n) % period;
  double acc[kCosShare] = {};
  for (int k = lane; k < Nt; k += 64) {
    const double cv = reduced_cos(m, Nt);
#pragma unroll
    for (int j = 0; j < kCosShare; ++j)
      if (j < np) acc[j] = fma(adj[(int64_t)j * Nt + k], cv, acc[j]);
    m += stride;
    if (m >= period) m -= period;
  }
#pragma unroll
  for (int j = 0; j < kCosShare; ++j) {
    if (j >= np) break;
    const double v = lanes_sum<64>(acc[j]);
    if (lane == 0) a.lambda[(int64_t)(p0 + j) * a.M + n] = a.g[n] * (n == 0 ? 1.0 : 2.0) * v;
  }
}

hipError_t launch_thermo_vjp(const ThermoVjpArgs& a, hipStream_t st) {
  dim3 g1((a.n_nodes + kThreads - 1) / kThreads, a.n_probs);
  hipLaunchKernelGGL(node_adj_kernel, g1, dim3(kThreads), 0, st, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  constexpr int kPerGroup = kThreads / 64;
  dim3 g2((a.M + kPerGroup - 1) / kPerGroup, (a.n_probs + kCosShare - 1) / kCosShare);
  hipLaunchKernelGGL(lambda_kernel, g2, dim3(kThreads), 0, st, a);
  return hipGetLastError();
}

}  // namespace kpm
