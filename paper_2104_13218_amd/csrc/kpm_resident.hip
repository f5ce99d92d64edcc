// Resident recursions: float64 sectors small enough for one compute unit.
//
// One workgroup owns one real column of one sector and runs every step of its
// recursion (the moments of Eqs. (6)-(7), or the Lanczos steps behind the
// bounds of Eqs. (4)-(5)) in a single launch: v_n lives in LDS (160 KB hold
// 19456 states and the bookkeeping), v_{n-1} in registers of the thread that
// owns the row, the dots are reduced inside the workgroup.  Nothing but the
// neighbour indices is read from memory per step, and those only where they
// do not fit registers.
//
// A row of H v is its diagonal (a table, +-J_b / 4 summed once) times v[r] plus
// sum_b (J_b / 2) v[P_b r] over the bonds that act, P_b the exchange of the
// bond's two sites: one index per bond, that of an element held at zero where the
// bond does not act.  (H = sum_b J_b (P_b / 2 - 1/4) over all bonds needs no
// table, but adds the bonds that do not act at full weight and takes them off
// again.  Error against 80-bit sums, as a multiple of the step kernels': 126 sets
// of 64 to 1000 moments 2.06, sawtooth chains up to 7, and 0.88 with the table; 60
// gradients 2.09 and 0.74, differences P_b v - v instead 2.08.  The table costs 2
// to 7 % of a step of the moments.)
//
// What bounds it: the LDS gathers.  A row needs one 8-byte LDS read per bond,
// 64 lanes to scattered addresses; with one row per thread the two barriers
// per step and the dot reduction cost as much again.
//
// Why: these sectors took one launch per step, 17-30 us each however few
// states they had (a chain of dependent loads through L2, then the next
// launch), and five launches per Lanczos step.  Measured: the 12-site ring
// (7 sectors, 20 columns, 128 steps) 30 -> 1.0 us per step, a whole call with
// bounds and thermodynamics 5.87 -> 0.47 ms; the 16-site ladder (9 sectors up
// to 12870 states, 200 columns, 50 steps) 111 -> 45 us per step and 117 ->
// 14 us per Lanczos step, the call 13.0 -> 3.0 ms.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kpm_device.h"
#include "kpm_internal.h"
#include "kpm_vec.h"

namespace kpm {

// ------------------------------------------------------------------ tables

// Per row: the rank of the state each bond's exchange maps it to (16 bits; the
// number of rows, where a zero is kept, if the two sites agree), eight bonds per
// 16-byte entry, entries of one chunk consecutive in the row; its diagonal, and
// a bit per bond that does not act.
__global__ __launch_bounds__(kThreads) void res_tables_kernel(const ResArgs a) {
  __shared__ uint32_t bn[kBinomN * kBinomN];
  for (int e = threadIdx.x; e < kBinomN * kBinomN; e += kThreads) bn[e] = a.binom[e];
  __syncthreads();
  const ProbDev P = a.probs[blockIdx.y];
  const ResInfo I = a.info[blockIdx.y];
  const uint32_t dim = (uint32_t)P.dim;
  const uint32_t r = blockIdx.x * kThreads + threadIdx.x;
  if (r >= dim) return;
  const uint32_t s = unrank(r, P.n_sites, P.n_up, bn);
  const uint32_t* mask = a.mask + I.coef_off;
  const double* cf = a.coef + I.coef_off;
  uint4* out = a.idx + I.idx_off;
  double dg = 0.0;
  uint32_t off = 0u;
  for (int ch = 0; ch < I.nch; ++ch) {
    uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const uint32_t m = mask[ch * 8 + t];    // 0 past the last bond
      const uint32_t v = s & m;
      const bool act = v != 0u && v != m;
      dg = fma(act ? -0.5 : 0.5, cf[ch * 8 + t], dg);   // coefficient 0 past the last bond
      uint32_t n = dim;
      if (!act) {
        off |= 1u << (ch * 8 + t);
      } else {
        n = word_rank(s ^ m, bn);
        if (n >= dim) {
          atomicOr(a.flag, 2);
          n = dim;
        }
      }
      w[t >> 1] |= n << ((t & 1) * 16);
    }
    out[(size_t)ch * dim + r] = make_uint4(w[0], w[1], w[2], w[3]);
  }
  a.diag[I.row_off + r] = dg;
  a.off[I.row_off + r] = off;
}

// ------------------------------------------------------------------ helpers

// Two sums over the wave, the first in the even lanes, the second in the odd.
__device__ __forceinline__ double wave_sum2(double p, double q, int lane) {
  const bool up = (lane & 1) != 0;
  double v = (up ? q : p) + lane_xor<1>(up ? p : q);
  v += lane_xor<2>(v);
  v += lane_xor<4>(v);
  v += lane_xor<8>(v);
  v += lane_xor<16>(v);
  v += lane_xor<32>(v);
  return v;
}

// Sum over the workgroup, known to every thread (one barrier; `slot` is 16
// doubles of LDS, not written again before the next barrier of the caller).
__device__ __forceinline__ double group_sum(double v, double* slot, int lane, int wid, int nw) {
  v += lane_xor<1>(v);
  v += lane_xor<2>(v);
  v += lane_xor<4>(v);
  v += lane_xor<8>(v);
  v += lane_xor<16>(v);
  v += lane_xor<32>(v);
  if (lane == 0) slot[wid] = v;
  __syncthreads();
  const int l = lane & 15;
  double t = l < nw ? slot[l] : 0.0;
  t += lane_xor<1>(t);
  t += lane_xor<2>(t);
  t += lane_xor<4>(t);
  t += lane_xor<8>(t);
  return t;
}

// Threads of the workgroup: a constant where a thread has more than one row
// (the launch then uses the most), so that row offsets are too.
template <int RPT>
__device__ __forceinline__ int group_threads(int most) {
  return RPT > 1 ? most : (int)blockDim.x;
}

// Element r of a row of doubles: 32-bit offset from a scalar base.
__device__ __forceinline__ double& at(double* base, uint32_t r) {
  return *reinterpret_cast<double*>(reinterpret_cast<unsigned char*>(base) + r * 8u);
}
__device__ __forceinline__ double at(const double* base, uint32_t r) {
  return *reinterpret_cast<const double*>(reinterpret_cast<const unsigned char*>(base) + r * 8u);
}

// sum_b (J_b / 2) x[exchanged row] of one row from its NCH index entries
template <int NCH>
__device__ __forceinline__ double gather_row(const uint4 (&q)[NCH], cptr<double> cf, const double* x) {
  double acc = 0.0;
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch) {
    const uint32_t w[4] = {q[ch].x, q[ch].y, q[ch].z, q[ch].w};
    double v[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) v[t] = x[(w[t >> 1] >> ((t & 1) * 16)) & 0xFFFFu];
#pragma unroll
    for (int t = 0; t < 8; ++t) acc = fma(cf[ch * 8 + t], v[t], acc);
  }
  return acc;
}

// The index entries and diagonals of a workgroup's rows: kept in registers for the whole
// recursion where they fit (at most 8 entries per thread), else read from
// L2 each step, the next row's while the current one is summed.  NCH is the
// number of entries per row (rows with fewer read repeats with coefficient 0).
template <int RPT, int NCH>
struct Rows {
  static constexpr bool kKeep = RPT * NCH <= 8;
  uint4 q[kKeep ? RPT : 1][NCH];
  double d[kKeep ? RPT : 1];
  const uint4* src;
  const double* dsrc;
  const uint32_t* osrc;
  uint32_t dim;
  int nch;
  __device__ __forceinline__ void load(int k, uint32_t r, uint4 (&o)[NCH]) const {
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch)     // 32-bit offsets from a scalar base
      o[ch] = *reinterpret_cast<const uint4*>(reinterpret_cast<const unsigned char*>(src) +
                                              (uint32_t)(((uint32_t)(ch < nch ? ch : 0) * dim + r) * 16u));
  }
};

// One product: h = sum_b (J_b/2) x[nb] and the diagonal d of each of the
// thread's rows, passed to use(k, row, on, h, d).
template <int RPT, int NCH, typename F>
__device__ __forceinline__ void product(const Rows<RPT, NCH>& R, cptr<double> cf, const double* x, int tid, int T,
                                        F&& use) {
  using RowsT = Rows<RPT, NCH>;
  if constexpr (RowsT::kKeep) {
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      const uint32_t r0 = (uint32_t)(k * T);
      if (r0 < R.dim) {
        const uint32_t r = r0 + (uint32_t)tid;
        uint4 q[NCH];
#pragma unroll
        for (int ch = 0; ch < NCH; ++ch)
          q[ch] = make_uint4(fresh(R.q[k][ch].x), fresh(R.q[k][ch].y), fresh(R.q[k][ch].z), fresh(R.q[k][ch].w));
        use(k, min(r, R.dim - 1u), r < R.dim, gather_row<NCH>(q, cf, x), R.d[k]);
      }
    }
  } else {
    uint4 cur[NCH], nxt[NCH];
    tid = (int)fresh((uint32_t)tid);
    R.load(0, min((uint32_t)tid, R.dim - 1u), nxt);
    double dn = at(R.dsrc, min((uint32_t)tid, R.dim - 1u));
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      const uint32_t r0 = (uint32_t)(k * T);
      if (r0 < R.dim) {
#pragma unroll
        for (int ch = 0; ch < NCH; ++ch) cur[ch] = nxt[ch];
        const double d = dn;
        const uint32_t r = r0 + (uint32_t)tid;
        if (k + 1 < RPT && r0 + (uint32_t)T < R.dim) {
          R.load(k + 1, min(r + (uint32_t)T, R.dim - 1u), nxt);
          dn = at(R.dsrc, min(r + (uint32_t)T, R.dim - 1u));
        }
        use(k, min(r, R.dim - 1u), r < R.dim, gather_row<NCH>(cur, cf, x), d);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
}

// Whether the sums of v x[r] over the steps, one per row, fit the registers
// beside the bond dots (rows kept in registers: always).
template <int RPT, int NCH>
constexpr bool kRowSums = RPT <= 16 || (RPT <= 26 && NCH <= 3);

// The product with its bond dots: D[b] += v x[P_b r] over the thread's rows, v =
// of(row, on).  Where the bond does not act the term is v x[r]: the same at every
// step, so with kRowSums it is left out here (the index gives a zero) and added at
// the end from the row's own sum.  Else the operand is picked by the row's bit of
// `off` (testing the index itself holds it, and 254 registers spilled at 38 rows
// of 32 bonds), which takes 10 to 20 % of a step: a gradient of 16 columns and 150
// steps, 1716 states and 32 bonds 1.52 ms, with the rows' sums 1.26; 12870 states
// and 8 bonds 6.0 and 5.1.
template <int NCH, bool kPick>
__device__ __forceinline__ double gather_dots(const uint4 (&q)[NCH], cptr<double> cf, const double* x, double v, double xr,
                                              uint32_t off, double (&D)[NCH * 8]) {
  double acc = 0.0;
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch) {
    const uint32_t w[4] = {q[ch].x, q[ch].y, q[ch].z, q[ch].w};
    double g[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) g[t] = x[(w[t >> 1] >> ((t & 1) * 16)) & 0xFFFFu];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      acc = fma(cf[ch * 8 + t], g[t], acc);
      D[ch * 8 + t] = fma(v, kPick && (off >> (ch * 8 + t) & 1u) ? xr : g[t], D[ch * 8 + t]);
    }
  }
  return acc;
}
template <int RPT, int NCH, typename V, typename F>
__device__ __forceinline__ void product_dots(const Rows<RPT, NCH>& R, cptr<double> cf, const double* x, int tid, int T,
                                             double (&D)[NCH * 8], V&& of, F&& use) {
  uint4 nxt[NCH];
  double dn = 0.0;
  uint32_t offn = 0u;
  constexpr bool kPick = !kRowSums<RPT, NCH>;
  tid = (int)fresh((uint32_t)tid);
  if constexpr (!Rows<RPT, NCH>::kKeep) {
    R.load(0, min((uint32_t)tid, R.dim - 1u), nxt);
    dn = at(R.dsrc, min((uint32_t)tid, R.dim - 1u));
    if constexpr (kPick) offn = R.osrc[min((uint32_t)tid, R.dim - 1u)];
  }
#pragma unroll
  for (int k = 0; k < RPT; ++k) {
    const uint32_t r0 = (uint32_t)(k * T);
    if (r0 < R.dim) {
      uint4 cur[NCH];
      const uint32_t r = r0 + (uint32_t)tid;
      const uint32_t rc = min(r, R.dim - 1u);
      const double v = of(rc, r < R.dim);
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch) {
        if constexpr (Rows<RPT, NCH>::kKeep)
          cur[ch] = make_uint4(fresh(R.q[k][ch].x), fresh(R.q[k][ch].y), fresh(R.q[k][ch].z), fresh(R.q[k][ch].w));
        else
          cur[ch] = nxt[ch];
      }
      double d = dn;
      const uint32_t off = offn;
      if constexpr (Rows<RPT, NCH>::kKeep) d = R.d[k];
      if constexpr (!Rows<RPT, NCH>::kKeep)
        if (k + 1 < RPT && r0 + (uint32_t)T < R.dim) {
          R.load(k + 1, min(r + (uint32_t)T, R.dim - 1u), nxt);
          dn = at(R.dsrc, min(r + (uint32_t)T, R.dim - 1u));
          if constexpr (kPick) offn = R.osrc[min(r + (uint32_t)T, R.dim - 1u)];
        }
      const double h = gather_dots<NCH, kPick>(cur, cf, x, v, kPick ? x[rc] : 0.0, off, D);
      use(k, rc, r < R.dim, h, d, v);
      if constexpr (!Rows<RPT, NCH>::kKeep) __builtin_amdgcn_sched_barrier(0);
    }
  }
}

template <int RPT, int NCH>
__device__ __forceinline__ void rows_init(Rows<RPT, NCH>& R, const ResArgs& a, const ResInfo& I, uint32_t dim, int tid,
                                          int T) {
  R.src = a.idx + I.idx_off;
  R.dsrc = a.diag + I.row_off;
  R.osrc = a.off + I.row_off;
  R.dim = dim;
  R.nch = I.nch;
  if constexpr (Rows<RPT, NCH>::kKeep) {
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      const uint32_t r = min((uint32_t)(tid + k * T), dim - 1u);
      R.load(k, r, R.q[k]);
      R.d[k] = at(R.dsrc, r);
    }
  }
}

// Start column of the job into x[0..dim), normalised as init_kernel does
// (mode 1: <r|r> = dim over the vector's columns; mode 2: unit norm); each
// thread writes and scales its own rows, and x[dim] = 0.  Returns the squared norm of the
// unscaled column.
__device__ __forceinline__ double start_rows(const ResArgs& a, const ProbDev& P, int kind, int col, int mode, int tid,
                                             int T, int lane, int wid, int nw, double* slot, double* x) {
  const int64_t dim = P.dim;
  double own = 0.0, pair = 0.0;
  if (tid == 0) x[dim] = 0.0;
#pragma unroll 1
  for (int64_t r = tid; r < dim; r += T) {
    const double v = start_value(kind, a.seed, P, col, r);
    x[r] = v;
    own = fma(v, v, own);
    if (kind == 1 && mode == 1) {
      const double o = start_value(kind, a.seed, P, col ^ 1, r);
      pair = fma(o, o, pair);
    }
  }
  const double n_own = group_sum(own, slot, lane, wid, nw);
  double scale = 1.0;
  if (mode == 2) {
    scale = 1.0 / sqrt(n_own);
  } else if (kind == 1 || kind == 2) {
    double n2 = n_own;
    if (kind == 1) n2 += group_sum(pair, slot + 16, lane, wid, nw);
    scale = sqrt((double)dim / n2);
  }
#pragma unroll 1
  for (int64_t r = tid; r < dim; r += T) x[r] *= scale;
  return n_own;
}

// ------------------------------------------------------------------ moments

// Dots of kResRing steps are kept in LDS before they are summed over the
// waves and written, so that the sum is not on every step's path.
constexpr int kResRing = 8;

template <int RPT, int NCH, bool KEEP>
__global__ __launch_bounds__(1024) void res_moments_kernel(const ResArgs a) {
  // a window of the call hangs on rounding: it is settled first, then the call
  // runs again
  if (*a.flag & 16) return;
  extern __shared__ __align__(16) double sm[];
  const int tid = threadIdx.x, T = group_threads<RPT>(1024), lane = tid & 63, nw = T >> 6;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const ResJob J = a.jobs[blockIdx.x];
  const ProbDev P = a.probs[J.prob];
  const ResInfo I = a.info[J.prob];
  const uint32_t dim = (uint32_t)P.dim;
  double* red = sm;                       // [kResRing][16][2]
  double* x = sm + kResRing * 32;         // [dim + 1]
  const double sa = a.scale[2 * J.prob], sb = a.scale[2 * J.prob + 1];
  const double inva = 1.0 / sa;
  const cptr<double> cf = cview(a.coef) + I.coef_off;
  Rows<RPT, NCH> R;
  rows_init(R, a, I, dim, tid, T);
  double y[RPT];
  start_rows(a, P, a.vec_kind, J.col, 1, tid, T, lane, wid, nw, red, x);
  double acc0 = 0.0;
#pragma unroll
  for (int k = 0; k < RPT; ++k) {
    const uint32_t r = (uint32_t)(tid + k * T);
    if (r < dim) acc0 = fma(x[r], x[r], acc0);
    y[k] = 0.0;
  }
  __syncthreads();                        // x complete; the slots of start_rows read
  {
    const double s0 = group_sum(acc0, red, lane, wid, nw);
    if (tid == 0) a.alpha[J.ocol] = s0;
    __syncthreads();
  }
  const int64_t TC = a.total_cols;
  // gradient calls: the whole trajectory (slot n holds v_n), or v_n and
  // v_{n+1} at every ckpt_every-th step
  const bool full = KEEP && a.ckpt == nullptr;
  double* kept = nullptr;
  if constexpr (KEEP) {
    kept = full ? a.seg + (a.K + 1) * a.col_elems[J.ocol] : a.ckpt + 2 * (int64_t)a.n_ckpt * a.col_elems[J.ocol];
    if (full)
      for (uint32_t r = tid; r < dim; r += T) kept[r] = x[r];
  }
  for (int n = 0; n < a.K; ++n) {
    double s2 = 0.0, s1 = 0.0;
    product<RPT, NCH>(R, cf, x, tid, T, [&](int k, uint32_t r, bool on, double h, double d) {
      const double xr = x[r];
      const double hx = fma(d - sb, xr, h) * inva;
      const double v = on ? (n == 0 ? hx : fma(2.0, hx, -y[k])) : 0.0;
      s2 = fma(v, v, s2);
      s1 = fma(v, xr, s1);
      y[k] = v;
    });
    const double f = wave_sum2(s2, s1, lane);
    if (lane < 2) red[(n & (kResRing - 1)) * 32 + wid * 2 + lane] = f;
    __syncthreads();                      // every read of v_n done
    const bool mark = KEEP && !full && n % a.ckpt_every == 0;
    double* k0 = nullptr;                 // where v_n goes (checkpoints) and v_{n+1}
    double* k1 = nullptr;
    if constexpr (KEEP) {
      k0 = kept + 2 * (int64_t)(n / a.ckpt_every) * dim;
      k1 = full ? kept + (int64_t)(n + 1) * dim : k0 + dim;
    }
    const uint32_t t0 = fresh((uint32_t)tid);
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      const uint32_t r = t0 + (uint32_t)(k * T);
      if (r < dim) {
        const double t = x[r];
        x[r] = y[k];
        if constexpr (KEEP) {
          if (mark) at(k0, r) = t;
          if (mark || full) at(k1, r) = y[k];
        }
        y[k] = t;
      }
    }
    if ((n & (kResRing - 1)) == kResRing - 1 || n == a.K - 1) {
      const int n0 = n & ~(kResRing - 1);
      const int st = n0 + (tid >> 1);
      if (tid < 2 * kResRing && st <= n) {
        const double* p = red + (st & (kResRing - 1)) * 32 + (tid & 1);
        double s = p[0];
        for (int w = 1; w < nw; ++w) s += p[2 * w];
        if (tid & 1) a.beta[(int64_t)st * TC + J.ocol] = s;
        else a.alpha[(int64_t)(st + 1) * TC + J.ocol] = s;
      }
    }
    __syncthreads();                      // v_{n+1} in place
  }
}

// ------------------------------------------------------------------ gradient

// Reverse sweep of one column (the recursion of kpm_adjoint.hip): with the
// adjoint vectors w_{n+1} in LDS and w_{n+2} in registers,
//   w_n = 2 abar_n v_n + bbar_n v_{n+1} + bbar_{n-1} v_{n-1} + 2 H' w_{n+1} - w_{n+2},
// and the gathers of w_{n+1} give the bond dots too: h_b = P_b / 2 - 1/4, so
//   <w_{n+1}, h_b v_n> = sum_r v_n[r] (w_{n+1}[P_b r] / 2 - w_{n+1}[r] / 4).
// A thread carries one sum per bond over all rows and steps; they are added
// over the workgroup once, at the end.  Vectors of v between checkpoints are
// made again, in the workgroup, by the forward step.
//
// 512 threads: a wave then has 256 registers, which hold w_{n+2} and the bond
// sums of up to 19456 rows without spills (1024 threads: 128).
template <int RPT, int NCH>
__global__ __launch_bounds__(kResAdjThreads) void res_adjoint_kernel(const ResArgs a) {
  extern __shared__ __align__(16) double sm[];
  const int tid = threadIdx.x, T = group_threads<RPT>(kResAdjThreads), lane = tid & 63, nw = T >> 6;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const ResJob J = a.jobs[blockIdx.x];
  const ProbDev P = a.probs[J.prob];
  const ResInfo I = a.info[J.prob];
  const uint32_t dim = (uint32_t)P.dim;
  double* red = sm;                       // [2][16]
  double* x = sm + 32;                    // [dim + 1]
  const double sa = a.scale[2 * J.prob], sb = a.scale[2 * J.prob + 1];
  if (tid == 0 && (!(sa > 0.0) || !isfinite(sa) || !isfinite(sb))) atomicOr(a.flag, 8);
  const double inva = 1.0 / sa;
  const cptr<double> cf = cview(a.coef) + I.coef_off;
  // dL/d<v_n, v_n> and dL/d<v_{n+1}, v_n> from dL/dmu through the estimator
  // and the doubling identities
  const double* lam = a.lambda + (int64_t)J.prob * a.M;
  double norm = a.alpha[J.ocol];
  if (a.vec_kind == 1) norm = a.alpha[J.ocol & ~1] + a.alpha[J.ocol | 1];
  const double est = (double)dim / ((a.R > 0 ? (double)a.R : (double)dim) * norm);
  double odd = 0.0;
  for (int n = 3 + 2 * tid; n < a.M; n += 2 * T) odd += lam[n];
  odd = group_sum(odd, red, lane, wid, nw);
  auto abar = [&](int n) { return 2 * n < a.M ? 2.0 * est * lam[2 * n] : 0.0; };            // n >= 1
  auto bbar = [&](int n) {
    if (n == 0) return est * (lam[1] - odd);
    return 2 * n + 1 < a.M ? 2.0 * est * lam[2 * n + 1] : 0.0;
  };
  Rows<RPT, NCH> R;
  rows_init(R, a, I, dim, tid, T);
  constexpr bool kSums = kRowSums<RPT, NCH>;
  double y[RPT], D[NCH * 8], S[kSums ? RPT : 1];              // S: sums of v_n w_{n+1}, by row or of all rows
#pragma unroll
  for (int k = 0; k < (kSums ? RPT : 1); ++k) S[k] = 0.0;
#pragma unroll
  for (int b = 0; b < NCH * 8; ++b) D[b] = 0.0;
#pragma unroll
  for (int k = 0; k < RPT; ++k) {
    const uint32_t r = (uint32_t)(tid + k * T);
    y[k] = 0.0;
    if (r < dim) x[r] = 0.0;
  }
  if (tid == 0) x[dim] = 0.0;
  const int64_t ce = a.col_elems[J.ocol];                    // rows of the columns before this one
  const bool full = a.ckpt == nullptr;
  const int C = a.ckpt_every, K = a.K;
  double* seg = a.seg + (int64_t)(full ? K + 1 : min(C, K) + 2) * ce;
  const double* ckpt = full ? nullptr : a.ckpt + 2 * (int64_t)a.n_ckpt * ce;
  double* wsave = full ? nullptr : a.wsave + 2 * ce;
  __syncthreads();
  auto swap_in = [&]() {                                     // x <-> y, own rows
    __syncthreads();
    const uint32_t t0 = fresh((uint32_t)tid);
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      const uint32_t r = t0 + (uint32_t)(k * T);
      if (r < dim) {
        const double t = x[r];
        x[r] = y[k];
        y[k] = t;
      }
    }
    __syncthreads();
  };
  for (int m = full ? 0 : a.n_ckpt - 1; m >= 0; --m) {
    const int j0 = full ? 0 : m * C;
    const int j1 = full ? K : min(j0 + C, K);
    if (!full) {
      const double* c = ckpt + 2 * (int64_t)m * dim;
      uint32_t t0 = fresh((uint32_t)tid);
#pragma unroll
      for (int k = 0; k < RPT; ++k) {
        const uint32_t r = t0 + (uint32_t)(k * T);
        if (r < dim) {
          at(wsave, r) = x[r];
          at(wsave + dim, r) = y[k];
        }
      }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < RPT; ++k) {
        const uint32_t r = t0 + (uint32_t)(k * T);
        if (r < dim) {
          y[k] = at(c, r);
          x[r] = at(c + dim, r);
          at(seg, r) = y[k];
          at(seg + dim, r) = x[r];
        }
      }
      __syncthreads();
      const int top = min(j1 + 1, K);                        // highest v index needed
      for (int t = 1; j0 + t + 1 <= top; ++t) {
        double* vt = seg + (int64_t)(t + 1) * dim;
        product<RPT, NCH>(R, cf, x, tid, T, [&](int k, uint32_t r, bool on, double h, double d) {
          const double v = on ? fma(2.0, fma(d - sb, x[r], h) * inva, -y[k]) : 0.0;
          if (on) at(vt, r) = v;
          y[k] = v;
        });
        swap_in();
      }
      __syncthreads();
      t0 = fresh((uint32_t)tid);
#pragma unroll
      for (int k = 0; k < RPT; ++k) {
        const uint32_t r = t0 + (uint32_t)(k * T);
        if (r < dim) {
          x[r] = at(wsave, r);
          y[k] = at(wsave + dim, r);
        }
      }
      __syncthreads();
    }
    for (int n = j1; n >= j0 + 1; --n) {
      const double ga = abar(n), gb = bbar(n), gbm = bbar(n - 1);
      const double* v0 = seg + (int64_t)(n - j0) * dim;
      const double* vm = v0 - dim;
      const double* vp = n + 1 <= K ? v0 + dim : v0;         // bbar_K = 0
      product_dots<RPT, NCH>(R, cf, x, tid, T, D, [&](uint32_t r, bool on) { return on ? 2.0 * at(v0, r) : 0.0; },
                             [&](int k, uint32_t r, bool on, double h, double d, double v2) {
                               const double wr = x[r];
                               double& s = S[kSums ? k : 0];
                               s = fma(v2, wr, s);
                               const double g = fma(gbm, at(vm, r), fma(gb, at(vp, r), ga * v2));
                               y[k] = on ? g + fma(2.0, fma(d - sb, wr, h) * inva, -y[k]) : 0.0;
                             });
      swap_in();
    }
  }
  // <w_1, h_b v_0> with weight 1 (slot 0 of segment 0 is v_0)
  product_dots<RPT, NCH>(R, cf, x, tid, T, D, [&](uint32_t r, bool on) { return on ? at(static_cast<const double*>(seg), r) : 0.0; },
                         [&](int k, uint32_t r, bool, double, double, double v) {
                           double& s = S[kSums ? k : 0];
                           s = fma(v, x[r], s);
                         });
  double s0 = S[0];
  if constexpr (kSums) {
    // the terms of the bonds that do not act, 0 past the last row
    s0 = 0.0;
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      const uint32_t r = (uint32_t)(tid + k * T);
      const uint32_t off = r < dim ? R.osrc[r] : 0u;
      s0 += S[k];
#pragma unroll
      for (int b = 0; b < NCH * 8; ++b) D[b] += off >> b & 1u ? S[k] : 0.0;
    }
  }
  const double sq = group_sum(s0, red, lane, wid, nw);
#pragma unroll
  for (int b = 0; b < NCH * 8; ++b) {
    const double t = group_sum(D[b], red + ((b + 1) & 1) * 16, lane, wid, nw);
    if (tid == 0) a.bond_part[(int64_t)J.ocol * kResMaxBonds + b] = inva * (0.5 * t - 0.25 * sq);
  }
}

// dL/dJ of problem blockIdx.x: its columns' parts, one bond per thread, the
// columns in order.
__global__ __launch_bounds__(64) void res_bond_sum_kernel(const ResArgs a, const UnitDev* units, double* dJ) {
  const ProbDev P = a.probs[blockIdx.x];
  const UnitDev U = units[blockIdx.x];
  const int b = threadIdx.x;
  if (b >= P.n_bonds) return;
  const double* p = a.bond_part + (int64_t)U.col_off * kResMaxBonds + b;
  double s = 0.0;
  for (int c = 0; c < U.ncols; ++c) s += p[(int64_t)c * kResMaxBonds];
  dJ[P.bond_off + b] = s;
}

// ------------------------------------------------------------------ Lanczos

// Eigenvalues of the symmetric tridiagonal (al[0..L), be2[0..L-1) = squared
// off-diagonals) below x, by the Sturm recurrence.
__device__ __forceinline__ int sturm_below(const double* al, const double* be2, int L, double x) {
  int cnt = 0;
  double q = 1.0;
  for (int i = 0; i < L; ++i) {
    // the quotient by the hardware reciprocal and two Newton steps
    double r = __builtin_amdgcn_rcp(q);
    r = fma(fma(-q, r, 1.0), r, r);
    r = fma(fma(-q, r, 1.0), r, r);
    q = al[i] - x - (i ? be2[i - 1] * r : 0.0);
    if (fabs(q) < 1e-140) q = -1e-140;   // its reciprocal times be2 stays finite up to 1e168
    cnt += q < 0.0;
  }
  return cnt;
}

// Plain Lanczos on H from the job's unit start column; the extreme Ritz
// values (cut at the first off-diagonal below 1e-12), widened as
// kpm_spectral_bounds documents, give the window and the problem's (a, b).
template <int RPT, int NCH>
__global__ __launch_bounds__(1024) void res_lanczos_kernel(const ResArgs a) {
  extern __shared__ __align__(16) double sm[];
  const int tid = threadIdx.x, T = group_threads<RPT>(1024), lane = tid & 63, nw = T >> 6;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const ResJob J = a.lz_jobs[blockIdx.x];
  const ProbDev P = a.probs[J.prob];
  const ResInfo I = a.info[J.prob];
  const uint32_t dim = (uint32_t)P.dim;
  double* red = sm;                       // [2][16]
  double* al = sm + 32;                   // [kResLanczos]
  double* be = al + kResLanczos;          // [kResLanczos]: beta_{j+1}^2
  double* x = be + kResLanczos;           // [dim + 1]
  const cptr<double> cf = cview(a.coef) + I.coef_off;
  Rows<RPT, NCH> R;
  rows_init(R, a, I, dim, tid, T);
  double y[RPT];
  start_rows(a, P, KPM_RES_GAUSSIAN, J.col, 2, tid, T, lane, wid, nw, red, x);
#pragma unroll
  for (int k = 0; k < RPT; ++k) y[k] = 0.0;
  __syncthreads();
  const int steps = (int)min((uint32_t)a.lz_steps, dim);
  double b = 0.0;
  int L = steps;
  for (int j = 0; j < steps; ++j) {
    double s = 0.0;
    product<RPT, NCH>(R, cf, x, tid, T, [&](int k, uint32_t r, bool on, double h, double d) {
      const double xr = x[r];
      const double w = on ? fma(d, xr, h) - b * y[k] : 0.0;
      s = fma(w, xr, s);
      y[k] = w;
    });
    const double alpha = group_sum(s, red, lane, wid, nw);
    s = 0.0;
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      const uint32_t r = (uint32_t)(tid + k * T);
      if (r < dim) {
        y[k] = fma(-alpha, x[r], y[k]);
        s = fma(y[k], y[k], s);
      }
    }
    const double b2 = group_sum(s, red + 16, lane, wid, nw);
    if (tid == 0) {
      al[j] = alpha;
      be[j] = b2;
    }
    b = sqrt(b2);
    if (j == steps - 1 || b < 1e-12) {    // the same for every thread
      L = j + 1;
      break;
    }
    const double inv = 1.0 / b;
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      const uint32_t r = (uint32_t)(tid + k * T);
      if (r < dim) {
        const double t = x[r];
        x[r] = y[k] * inv;
        y[k] = t;
      }
    }
    __syncthreads();
  }
  __syncthreads();
  // extreme eigenvalues by multisection: half of the threads cut the interval
  // of the smallest, half that of the largest, until no point falls inside
  double gl = INFINITY, gu = -INFINITY;
  for (int i = 0; i < L; ++i) {
    const double r = (i ? sqrt(be[i - 1]) : 0.0) + (i + 1 < L ? sqrt(be[i]) : 0.0);
    gl = fmin(gl, al[i] - r);
    gu = fmax(gu, al[i] + r);
  }
  const int half = T >> 1;
  const bool top = tid >= half;
  const int t = top ? tid - half : tid;
  double lo0 = gl, hi0 = gu, lo1 = gl, hi1 = gu;   // brackets of the smallest and the largest
  for (int it = 0; it < 60; ++it) {
    const double l = top ? lo1 : lo0, u = top ? hi1 : hi0;
    const double p = fma((u - l), (double)(t + 1) / (double)(half + 1), l);
    const bool below = sturm_below(al, be, L, p) <= (top ? L - 1 : 0);   // the eigenvalue is at or above p
    const int c0 = __syncthreads_count(!top && below);
    const int c1 = __syncthreads_count(top && below);
    auto point = [&](double lv, double uv, int i) { return fma((uv - lv), (double)(i + 1) / (double)(half + 1), lv); };
    const double nl0 = c0 > 0 ? point(lo0, hi0, c0 - 1) : lo0, nh0 = c0 < half ? point(lo0, hi0, c0) : hi0;
    const double nl1 = c1 > 0 ? point(lo1, hi1, c1 - 1) : lo1, nh1 = c1 < half ? point(lo1, hi1, c1) : hi1;
    const bool same = nl0 == lo0 && nh0 == hi0 && nl1 == lo1 && nh1 == hi1;
    lo0 = nl0;
    hi0 = nh0;
    lo1 = nl1;
    hi1 = nh1;
    const double m0 = 0.5 * (lo0 + hi0), m1 = 0.5 * (lo1 + hi1);
    if (same || ((m0 <= lo0 || m0 >= hi0) && (m1 <= lo1 || m1 >= hi1))) break;   // the same for every thread
  }
  if (tid == 0) {
    const double lo = 0.5 * (lo0 + hi0), hi = 0.5 * (lo1 + hi1);
    const double W = hi - lo;
    double e0 = lo - a.margin * W, e1 = hi + a.margin * W;
    if (W < 1e-8 * fmax(1.0, fmax(fabs(lo), fabs(hi)))) {
      e0 = lo - 0.5;
      e1 = hi + 0.5;
    }
    a.lohi[2 * J.prob] = e0;
    a.lohi[2 * J.prob + 1] = e1;
    const double sa = (e1 - e0) / (2.0 - a.eps), sb = 0.5 * (e1 + e0);
    a.scale[2 * J.prob] = sa;
    a.scale[2 * J.prob + 1] = sb;
    if (!(sa > 0.0) || !isfinite(sa) || !isfinite(sb)) atomicOr(a.flag, 8);
  }
  // Does the window hang on rounding?  A copy of the other, converged end takes
  // steps from an end that has not converged, from a point on that the last
  // bits decide.  An end's value of two steps less differs by c widths, and the
  // Lanczos vectors have lost their orthogonality by omega (Simon's recurrence
  // for omega_{j,k} = <q_j, q_k>, 1984): the order of summation moves the end
  // by about c omega^2.  Over 8640 sectors (six lattices of 8-16 sites) no
  // window with c under 1e-13 or c omega^2 under 3e-15 moved by more than 4e-15
  // of its width; a tenth of the sectors is above, most of them sawtooth chains.
  const double elo = 0.5 * (lo0 + hi0), ehi = 0.5 * (lo1 + hi1), width = ehi - elo;
  if (L < 3 || (L < steps && (uint32_t)L < dim)) return;       // the Krylov space is exhausted
  const int Ls = L - 2;
  auto converged = [&](double c) {
    return sturm_below(al, be, Ls, elo + c * width) > 0 && sturm_below(al, be, Ls, ehi - c * width) < Ls;
  };
  if (converged(kRoundingEnd)) return;
  __syncthreads();
  constexpr int S = kResLanczos + 2;
  double *prev = x, *cur = x + S, *nxt = x + 2 * S;            // omega_{j-1}, omega_j, omega_{j+1}
  for (int k = tid; k < 3 * S; k += T) x[k] = k == S ? 1.0 : 0.0;
  for (int k = tid; k < L; k += T) be[k] = sqrt(be[k]);
  __syncthreads();
  const double ulp = 1.1e-16;
  double top_w = 0.0, size = 0.0;
  for (int k = 0; k < L; ++k) size = fmax(size, fabs(al[k]));
  for (int j = 0; j + 1 < L; ++j) {
    for (int k = tid; k < j; k += T) {
      double v = be[k] * cur[k + 1] + (al[k] - al[j]) * cur[k] - be[j - 1] * prev[k];
      if (k > 0) v += be[k - 1] * cur[k - 1];
      v = (v + copysign(2.0 * ulp * size, v)) / be[j];
      nxt[k] = v;
      top_w = fmax(top_w, fabs(v));
    }
    if (tid == 0) {
      nxt[j] = 30.0 * ulp * be[0] / be[j];
      nxt[j + 1] = 1.0;
    }
    __syncthreads();
    double* t = prev;
    prev = cur;
    cur = nxt;
    nxt = t;
  }
  for (int k = tid; k < L; k += T) be[k] *= be[k];
  __syncthreads();
  const double w2 = fmin(top_w * top_w, 1.0);   // over this thread's entries
  if (w2 > kRoundingReach && !converged(fmax(kRoundingEnd, kRoundingReach / w2))) {
    a.unstable[J.prob] = 1;
    atomicOr(a.flag, 16);
  }
}

// ------------------------------------------------------------------ launches

hipError_t launch_res_tables(const ResArgs& a, int n_probs, uint32_t max_dim, hipStream_t st) {
  hipLaunchKernelGGL(res_tables_kernel, dim3((max_dim + kThreads - 1) / kThreads, n_probs), dim3(kThreads), 0, st, a);
  return hipGetLastError();
}

template <typename K>
static hipError_t launch_res(K kernel, const ResArgs& a, int grid, int threads, size_t lds, hipStream_t st) {
  if (lds > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), lds, st, a);
  return hipGetLastError();
}

template <int RPT, int NCH>
static hipError_t launch_res_t(const ResArgs& a, int what, int grid, int threads, size_t lds, hipStream_t st) {
  if constexpr (RPT <= 19 && RPT != 16) {
    if (what == kResLz) return launch_res(res_lanczos_kernel<RPT, NCH>, a, grid, threads, lds, st);
    if (what == kResMom)
      return a.seg ? launch_res(res_moments_kernel<RPT, NCH, true>, a, grid, threads, lds, st)
                   : launch_res(res_moments_kernel<RPT, NCH, false>, a, grid, threads, lds, st);
  }
  if constexpr (RPT != 13 && RPT != 19) {
    if (what == kResAdj) return launch_res(res_adjoint_kernel<RPT, NCH>, a, grid, threads, lds, st);
  }
  return hipErrorInvalidValue;
}

template <int RPT>
static hipError_t launch_res_n(const ResArgs& a, int what, int nch, int grid, int threads, size_t lds, hipStream_t st) {
  if (nch <= 2) return launch_res_t<RPT, 2>(a, what, grid, threads, lds, st);
  if (nch <= 3) return launch_res_t<RPT, 3>(a, what, grid, threads, lds, st);
  return launch_res_t<RPT, 4>(a, what, grid, threads, lds, st);
}

// Rows per thread: the smallest instantiation that covers the largest sector
// with at most 1024 threads (the gradient: kResAdjThreads).
static hipError_t launch_res_any(const ResArgs& a, int what, int nch, int grid, uint32_t max_dim, hipStream_t st) {
  if (max_dim > (uint32_t)kResMaxDim || nch > kResMaxBonds / 8 || grid < 1) return hipErrorInvalidValue;
  // the bounds end on three rows of omega in the vector's place
  const size_t rows = (size_t)max_dim + 1;
  const size_t lds = what == kResLz ? (std::max<size_t>(rows, 3 * (kResLanczos + 2)) + 32 + 2 * kResLanczos) * 8
                                    : (rows + (what == kResMom ? kResRing * 32 : 32)) * 8;
  const uint32_t most = what == kResAdj ? (uint32_t)kResAdjThreads : 1024u;
  const int threads = (int)std::min<uint32_t>(most, std::max(64u, (max_dim + 63u) / 64u * 64u));
  const int rpt = (int)((max_dim + threads - 1) / threads);
  if (rpt <= 1) return launch_res_n<1>(a, what, nch, grid, threads, lds, st);
  if (rpt <= 2) return launch_res_n<2>(a, what, nch, grid, threads, lds, st);
  if (rpt <= 4) return launch_res_n<4>(a, what, nch, grid, threads, lds, st);
  if (rpt <= 8) return launch_res_n<8>(a, what, nch, grid, threads, lds, st);
  if (what == kResAdj) {
    if (rpt <= 16) return launch_res_n<16>(a, what, nch, grid, threads, lds, st);
    if (rpt <= 26) return launch_res_n<26>(a, what, nch, grid, threads, lds, st);
    return launch_res_n<38>(a, what, nch, grid, threads, lds, st);
  }
  if (rpt <= 13) return launch_res_n<13>(a, what, nch, grid, threads, lds, st);
  return launch_res_n<19>(a, what, nch, grid, threads, lds, st);
}

hipError_t launch_resident(const ResArgs& a, int what, int nch, int n_jobs, uint32_t max_dim, hipStream_t st) {
  return launch_res_any(a, what, nch, n_jobs, max_dim, st);
}

hipError_t launch_res_bond_sum(const ResArgs& a, const UnitDev* units, int n_probs, double* dJ, hipStream_t st) {
  hipLaunchKernelGGL(res_bond_sum_kernel, dim3(n_probs), dim3(64), 0, st, a, units, dJ);
  return hipGetLastError();
}

}  // namespace kpm
