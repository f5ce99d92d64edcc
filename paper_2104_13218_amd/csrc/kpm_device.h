// Device helpers shared by the gfx950 kernels: basis unranking and ranking in
// the combinatorial number system of an S^z sector.
#pragma once

#include <hip/hip_runtime.h>

#include "kpm_internal.h"

namespace kpm {

// Word of rank r among N-bit words with k set bits (combinatorial number
// system, colex order = ascending integer order): greedily take the highest
// position p with C(p, j) <= remaining rank, for j = k .. 1.
__device__ __forceinline__ uint32_t unrank(uint32_t r, int N, int k, const uint32_t* binom) {
  uint32_t s = 0;
  int j = k;
  for (int p = N - 1; p >= 0 && j > 0; --p) {
    const uint32_t cv = binom[p * kBinomN + j];
    if (cv <= r) {
      s |= 1u << p;
      r -= cv;
      --j;
    }
  }
  return s;
}

// Rank of word s: the bits split as x0 (B0 low bits), x1 (next B1), x2 (rest);
// rank = T0[x0] + T1[x1][popcount(x0)] + T2[x2] (T2 already knows the sector's
// popcount, so the number of set bits below x2 is implied).
struct RankTables {
  const uint32_t* T0;
  const uint32_t* T1;
  const uint32_t* T2;
  uint32_t m0, m1;
  int B0, sh2;
  __device__ __forceinline__ uint32_t rank(uint32_t s) const {
    const uint32_t x0 = s & m0;
    const uint32_t x1 = (s >> B0) & m1;
    const uint32_t x2 = s >> sh2;
    return T0[x0] + T1[x1 * (uint32_t)(B0 + 1) + __popc(x0)] + T2[x2];
  }
};

__device__ __forceinline__ RankTables make_tables(const uint32_t* tab, const ProbDev& P) {
  RankTables R;
  R.T0 = tab;
  R.T1 = tab + (1u << P.B0);
  R.T2 = R.T1 + (1u << P.B1) * (uint32_t)(P.B0 + 1);
  R.m0 = (1u << P.B0) - 1u;
  R.m1 = (1u << P.B1) - 1u;
  R.B0 = P.B0;
  R.sh2 = P.B0 + P.B1;
  return R;
}

// Colex (= ascending-integer) rank of word s among the words of its popcount.
__device__ __forceinline__ uint32_t word_rank(uint32_t s, const uint32_t* binom) {
  uint32_t r = 0;
  int j = 0;
  for (uint32_t x = s; x; x &= x - 1u) {
    ++j;
    r += binom[(__ffs(x) - 1) * kBinomN + j];
  }
  return r;
}

// Relabelled sites: the word with bit i moved to bit perm[i] (to_kernel) or
// back (from the kernels' labels to the problem's).
__device__ __forceinline__ uint32_t relabel_word(uint32_t w, const uint8_t* perm, int N, bool to_kernel) {
  uint32_t o = 0;
  for (int i = 0; i < N; ++i) {
    if (to_kernel) o |= ((w >> i) & 1u) << perm[i];
    else o |= ((w >> perm[i]) & 1u) << i;
  }
  return o;
}

// Spin-s sites: rank of the digit string dg (4 bits per site, digit sum n)
// in its sector, from the table P[i][r][d] (strings of sites 0..i with sum r
// and digit < d at site i): the entries of each site's digit, from the most
// significant site down, with r the sum still left.
__device__ __forceinline__ uint32_t spin_rank(uint64_t dg, int N, int n, int R1, int B,
                                              const uint32_t* tab) {
  uint32_t rank = 0;
  int r = n;
  for (int i = N - 1; i >= 0; --i) {
    const int d = (int)((dg >> (4 * i)) & 15u);
    rank += tab[(i * R1 + r) * B + d];
    r -= d;
  }
  return rank;
}

// Counter-based SplitMix64 (Steele, Lea, Flood 2014): output ctr+1 of the
// sequential generator started at `seed`.
__device__ __forceinline__ uint64_t splitmix(uint64_t seed, uint64_t ctr) {
  uint64_t z = seed + 0x9E3779B97F4A7C15ull * (ctr + 1ull);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
__device__ __forceinline__ double unit_open(uint64_t u) {
  return ((double)(u >> 11) + 0.5) * 0x1.0p-53;
}


// Unnormalised start value of column pc (of the problem) at row rho.
__device__ __forceinline__ double start_value(int kind, uint64_t seed, const ProbDev& P, int pc,
                                              int64_t rho) {
  if (kind == 3) return rho == (int64_t)pc ? 1.0 : 0.0;
  const int r = kind == 1 ? (pc >> 1) : pc;
  const uint64_t stream = ((uint64_t)P.cluster << 16) | ((uint64_t)P.n_up << 10) | (uint64_t)r;
  if (kind == 0) {
    const uint64_t u = splitmix(seed, (stream << 32) | (uint64_t)rho);
    return (u >> 63) ? -1.0 : 1.0;
  }
  const uint64_t i1 = (uint64_t)(2 * rho), i2 = (uint64_t)(2 * rho + 1);
  const double u1 = unit_open(splitmix(seed, (stream << 32) | i1));
  const double u2 = unit_open(splitmix(seed, (stream << 32) | i2));
  const double rad = sqrt(-2.0 * log(u1));
  const double ang = 2.0 * M_PI * u2;
  return (kind == 1 && (pc & 1)) ? rad * sin(ang) : rad * cos(ang);
}

}  // namespace kpm
