// Sums over moments (the kernel polynomial reconstruction) and their transposes.
#include <hip/hip_runtime.h>

#include "internal.h"

namespace gpuqt {

namespace {

// T_n(x) = Re z^n of the sums over moments, z = x + i sqrt(1 - x^2).  Powers of z come from squarings with 106 bits
// (c + cl, s + sl), so what a kernel starts from is rounded once: cos(n acos x) carries n times the error of a
// rounded angle, and the sums of 1000 moments that started from it were 35 times less exact than one three-term recurrence over
// all of them (r.m.s. against extended precision, random moments, energies up to 0.95 of the band: recurrence
// 1.5e-15, angles 5.3e-14, powers 4.3e-16 by k_kpm and 1.1e-15 by k_kpm_rows; 64 moments 3.7e-16, 4.4e-15, 1.7e-16, 3.0e-16).
struct Unit { double c, s; };
struct Unit2 { double c, cl, s, sl; };

__device__ __forceinline__ Unit times(Unit a, Unit b) {
  return {fma(a.c, b.c, -(a.s * b.s)), fma(a.c, b.s, a.s * b.c)};
}

// h + l, |l| <= |h| / 2^53, of a + b and a small e
__device__ __forceinline__ void sum2(double a, double b, double e, double* h, double* l) {
#pragma clang fp contract(off)
  const double s = a + b, v = s - a, r = ((a - (s - v)) + (b - v)) + e;
  *h = s + r;
  *l = r - (*h - s);
}

__device__ __forceinline__ Unit2 unit_of(double x) {
#pragma clang fp contract(off)
  const double p = x * x;
  double w, wl;   // 1 - x^2
  sum2(1.0, -p, -fma(x, x, -p), &w, &wl);
  const double s = sqrt(w);
  return {x, 0.0, s, (fma(-s, s, w) + wl) / (2.0 * s)};   // (NaN past the band; not used)
}

// 2 c^2 - 1, 2 s c.  The low parts grow fourfold (c^2 - 1/2 is exact from 1/4 on, else its error is taken): normal()
// every few squarings.
__device__ __forceinline__ Unit2 squared(Unit2 z) {
#pragma clang fp contract(off)
  const double p = z.c * z.c, h = p - 0.5, m = z.s * z.c;
  const double pl = fma(z.c, z.c, -p) + (p - (h + 0.5)), ml = fma(z.s, z.c, -m);
  return {2.0 * h, 2.0 * fma(2.0 * z.c, z.cl, pl), 2.0 * m, 2.0 * fma(z.s, z.cl, fma(z.sl, z.c, ml))};
}

__device__ __forceinline__ Unit2 normal(Unit2 z) {
#pragma clang fp contract(off)
  const double c = z.c + z.cl, s = z.s + z.sl;
  return {c, z.cl - (c - z.c), s, z.sl - (s - z.s)};
}

__device__ __forceinline__ Unit rounded(Unit2 z) { return {z.c + z.cl, z.s + z.sl}; }

__device__ __forceinline__ double product(double x, double xl, double y, double yl, double* e) {
#pragma clang fp contract(off)
  const double p = x * y;
  *e = fma(x, y, -p) + (x * yl + xl * y);
  return p;
}

__device__ __forceinline__ Unit2 times(Unit2 a, Unit2 b) {
#pragma clang fp contract(off)
  Unit2 q;
  double e1, e2;
  double p1 = product(a.c, a.cl, b.c, b.cl, &e1), p2 = product(a.s, a.sl, b.s, b.sl, &e2);
  sum2(p1, -p2, e1 - e2, &q.c, &q.cl);
  p1 = product(a.c, a.cl, b.s, b.sl, &e1), p2 = product(a.s, a.sl, b.c, b.cl, &e2);
  sum2(p1, p2, e1 + e2, &q.s, &q.sl);
  return q;
}

// KPM sum of Section 3.3, one (row r, energy) per wavefront and kKpmEnergies of them in turn:
// s = sum_n 2 g_n c_n T_n(x), the damped coefficients of kKpmTile moments at a time in LDS (g_n and its
// sincospi once a workgroup, not once an energy).  Lane l takes the moments l + 64 i of a tile: z^l from the bits of
// l, then turned by z^64, at most 16 times before a tile starts from its own power.
// Bound by latency: 1001 energies, 1000 moments, one row: 200 us with a thread per energy and one chain
// over all moments, 8 us so.
constexpr int kKpmTile = 1024, kKpmEnergies = 2, kKpmWaves = 4;

__global__ __launch_bounds__(64 * kKpmWaves) void k_kpm(int R, int M, const double* __restrict__ C, int n_E,
                                                        const double* __restrict__ E, double inv_dE,
                                                        double pref_base, int jackson, double cot_pa,
                                                        double* __restrict__ out) {
  __shared__ double wc[kKpmTile];
  const int r = blockIdx.y;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int e0 = (blockIdx.x * kKpmWaves + wave) * kKpmEnergies;
  const double a = 1.0 / (M + 1);
  const double* c = C + (int64_t)r * M;
  double x[kKpmEnergies], s[kKpmEnergies];
  Unit zl[kKpmEnergies], z64[kKpmEnergies];   // z^lane, z^64
  Unit2 tile[kKpmEnergies], start[kKpmEnergies];   // z^kKpmTile, z^n0
#pragma unroll
  for (int q = 0; q < kKpmEnergies; ++q) {
    x[q] = e0 + q < n_E ? E[e0 + q] * inv_dE : 0.0;
    s[q] = 0.0;
    Unit2 z = unit_of(x[q]);
    zl[q] = {1.0, 0.0};
    for (int j = 0; j < 6; ++j) {
      if (lane >> j & 1) zl[q] = times(zl[q], rounded(z));
      z = squared(z);
    }
    z64[q] = rounded(z);
    if (M > kKpmTile) {
      z = normal(z);
      for (int j = 64; j < kKpmTile; j *= 2) z = squared(z);
      z = normal(z);
    }
    tile[q] = start[q] = z;
  }
  for (int n0 = 0; n0 < M; n0 += kKpmTile) {
    const int m = min(kKpmTile, M - n0);
    __syncthreads();
    for (int i = threadIdx.x; i < m; i += 64 * kKpmWaves) {
      const int n = n0 + i;
      double g = n == 0 ? 1.0 : 2.0;
      if (jackson && n > 0) {
        double sn, cs;
        sincospi(n * a, &sn, &cs);
        g *= (1.0 - n * a) * cs + a * sn * cot_pa;
      }
      wc[i] = g * c[n];
    }
    __syncthreads();
    Unit t[kKpmEnergies];   // z^n
#pragma unroll
    for (int q = 0; q < kKpmEnergies; ++q) {
      t[q] = zl[q];
      if (n0 > 0) t[q] = times(t[q], rounded(start[q]));
      if (n0 > 0 && n0 + kKpmTile < M) start[q] = times(start[q], tile[q]);
    }
    for (int i = lane; i < m; i += 64) {
      const double w = wc[i];
#pragma unroll
      for (int q = 0; q < kKpmEnergies; ++q) {
        s[q] = fma(w, t[q].c, s[q]);
        t[q] = times(t[q], z64[q]);
      }
    }
  }
#pragma unroll
  for (int q = 0; q < kKpmEnergies; ++q) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) s[q] += __shfl_xor(s[q], off);
    if (lane == 0 && e0 + q < n_E)
      out[(int64_t)r * n_E + e0 + q] =
          fabs(x[q]) < 1.0 ? pref_base / sqrt(1.0 - x[q] * x[q]) * s[q] : __builtin_nan("");
  }
}

// The same sum for many rows and energies: one energy and RQ rows a thread, 2^lE energies and 256 >> lE such
// groups of rows a workgroup, kKpmRowTile moments of its rows in LDS.  Chains T_{n+1} = 2 x T_n - T_{n-1} of eight moments, two
// at a time and each for all RQ rows, start from z^n0 turned by z^8 and z^16, that from turns by z^64, and
// every kKpmTile moments from its own power.
constexpr int kKpmRowTile = 64, kKpmRowsMinE = 4;   // (at least 2^kKpmRowsMinE energies)

template <int RQ>
__global__ __launch_bounds__(256) void k_kpm_rows(int R, int M, const double* __restrict__ C, int n_E,
                                                  const double* __restrict__ E, double inv_dE, double pref_base,
                                                  int jackson, double cot_pa, int lE, double* __restrict__ out) {
  constexpr int STRIDE = kKpmRowTile * RQ + 2;   // of a group of rows (+ 2: groups start in other banks)
  extern __shared__ double wr[];                 // [256 >> lE][STRIDE]
  const int e = (int)((blockIdx.x << lE) | (threadIdx.x & ((1u << lE) - 1))), g = threadIdx.x >> lE, G = 256 >> lE;
  const int64_t row0 = (int64_t)blockIdx.y * G * RQ;
  const double a = 1.0 / (M + 1), x = e < n_E ? E[e] * inv_dE : 0.0;
  Unit2 z = unit_of(x);
  const double sx = z.s;
  z = squared(squared(squared(z)));
  const Unit z8 = rounded(z);
  z = squared(z);
  const Unit z16 = rounded(z);
  z = squared(squared(z));
  const Unit z64 = rounded(z);
  if (M > kKpmTile) {
    z = normal(z);
    for (int j = kKpmRowTile; j < kKpmTile; j *= 2) z = squared(z);
    z = normal(z);
  }
  Unit2 tile = z;         // z^kKpmTile, and its power at the next multiple of kKpmTile
  Unit at = {1.0, 0.0};   // z^n0
  double s[RQ];
#pragma unroll
  for (int r = 0; r < RQ; ++r) s[r] = 0.0;
  for (int n0 = 0; n0 < M; n0 += kKpmRowTile) {
    const int i = threadIdx.x & (kKpmRowTile - 1), n = n0 + i;   // the moment this thread brings, of every row
    double w = n == 0 ? 1.0 : 2.0;
    if (jackson && n > 0) {
      double sn, cs;
      sincospi(n * a, &sn, &cs);
      w *= (1.0 - n * a) * cs + a * sn * cot_pa;
    }
    __syncthreads();
    for (int q = threadIdx.x / kKpmRowTile; q < G * RQ; q += 256 / kKpmRowTile)
      wr[q / RQ * STRIDE + i * RQ + q % RQ] = n < M && row0 + q < R ? w * C[(row0 + q) * M + n] : 0.0;
    __syncthreads();
    const double* wg = wr + g * STRIDE;
    Unit v = at;
    for (int c = n0; c < min(M, n0 + kKpmRowTile); c += 16) {
      const Unit v8 = times(v, z8);
      double t[2] = {v.c, v8.c}, u[2] = {fma(v.c, x, v.s * sx), fma(v8.c, x, v8.s * sx)};   // T_n, T_{n-1}
      const double* wc = wg + (c - n0) * RQ;
      // weights of two moments of both chains, read while the two before are taken (left to itself the compiler waits
      // for each pair of weights: 256 rows, 1000 moments, 1001 energies 82 us instead of 42)
      double w[2][2][2][RQ];
      auto read = [&](int k) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int r = 0; r < RQ; ++r) w[k / 2 & 1][h][i][r] = wc[(8 * h + k + i) * RQ + r];
      };
      read(0);
#pragma unroll
      for (int k = 0; k < 8; k += 2) {
        if (k + 2 < 8) read(k + 2);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int r = 0; r < RQ; ++r) s[r] = fma(w[k / 2 & 1][h][i][r], t[h], s[r]);
            const double next = fma(2.0 * x, t[h], -u[h]);
            u[h] = t[h];
            t[h] = next;
          }
      }
      v = times(v, z16);
    }
    at = times(at, z64);
    if ((n0 + kKpmRowTile) % kKpmTile == 0 && n0 + kKpmRowTile < M) {
      at = rounded(tile);
      tile = times(tile, z);
    }
  }
  if (e >= n_E) return;
#pragma unroll
  for (int r = 0; r < RQ; ++r) {
    const int64_t row = row0 + g * RQ + r;
    if (row < R)
      out[row * n_E + e] = fabs(x) < 1.0 ? pref_base / sqrt(1.0 - x * x) * s[r] : __builtin_nan("");
  }
}

// Transpose of k_kpm: out[r][n] = sum_e g[r][e] pref(E_e) w_n T_n(E~_e).  kKpmMoments moments of a row to 2^lS
// threads, which share the energies; energies outside the band contribute nothing.  acos, the square root, cosine and sine once
// for all of a group's moments.  A chain of eight from two cosines keeps the difference of their angles' errors, one from the
// cosine and the sine of one angle does not: 96 rows, 1000 moments, up to 0.9999 of the band, r.m.s. 2.5e-13 (computed on
// the host) and 3.3e-14; 6.9e-14 by a cosine per moment.  Powers of z leave 4e-16 and take twice as long at 1001 energies.
constexpr int kKpmMoments = 8;

// cosine and sine of n th, the product's rounding taken back
__device__ __forceinline__ Unit multiple(int n, double th) {
#pragma clang fp contract(off)
  const double p = n * th, e = fma((double)n, th, -p);
  double c, s;
  sincos(p, &s, &c);
  return {fma(-s, e, c), fma(c, e, s)};
}

__global__ __launch_bounds__(256) void k_kpm_adjoint(int R, int M, const double* __restrict__ g, int n_E,
                                                     const double* __restrict__ E, double inv_dE,
                                                     double pref_base, int jackson, double cot_pa, int lS,
                                                     double* __restrict__ out) {
  extern __shared__ double part[];   // [256 / in_wave][kKpmMoments]
  const int share = 1 << lS, in_wave = min(share, 64), l = threadIdx.x & (share - 1);
  const int groups = (M + kKpmMoments - 1) / kKpmMoments;   // of a row
  const int64_t q = (int64_t)blockIdx.x * (256 >> lS) + (threadIdx.x >> lS), r = q / groups;
  const int n0 = (int)(q - r * groups) * kKpmMoments;
  double s[kKpmMoments];
#pragma unroll
  for (int i = 0; i < kKpmMoments; ++i) s[i] = 0.0;
  for (int e = r < R ? l : n_E; e < n_E; e += share) {
    const double x = E[e] * inv_dE;
    if (!(fabs(x) < 1.0)) continue;
    const double sx = sqrt(1.0 - x * x), f = g[r * n_E + e] * pref_base / sx;
    const Unit z = multiple(n0, acos(x));
    double t = z.c, u = fma(t, x, z.s * sx);   // T_n0, T_{n0-1}
#pragma unroll
    for (int i = 0; i < kKpmMoments; ++i) {
      s[i] = fma(f, t, s[i]);
      const double v = fma(2.0 * x, t, -u);
      u = t;
      t = v;
    }
  }
  for (int off = in_wave >> 1; off >= 1; off >>= 1)
#pragma unroll
    for (int i = 0; i < kKpmMoments; ++i) s[i] += __shfl_xor(s[i], off);
  if ((threadIdx.x & (in_wave - 1)) == 0)
#pragma unroll
    for (int i = 0; i < kKpmMoments; ++i) part[threadIdx.x / in_wave * kKpmMoments + i] = s[i];
  __syncthreads();
  if (r >= R) return;
  const double a = 1.0 / (M + 1);
  const int w0 = (threadIdx.x - l) / in_wave, w1 = w0 + share / in_wave;   // the group's wavefronts, in order
#pragma unroll 1
  for (int i = l; i < kKpmMoments && n0 + i < M; i += share) {
    const int n = n0 + i;
    double wn = n == 0 ? 1.0 : 2.0, sum = 0.0;
    for (int w = w0; w < w1; ++w) sum += part[w * kKpmMoments + i];
    if (jackson && n > 0) {
      double sn, cs;
      sincospi(n * a, &sn, &cs);
      wn *= (1.0 - n * a) * cs + a * sn * cot_pa;
    }
    out[r * M + n] = wn * sum;
  }
}

}  // namespace

hipError_t launch_kpm(int R, int M, const double* C, int n_E, const double* E, double inv_dE,
                      double pref_base, int jackson, double* out, hipStream_t s) {
  if (R <= 0 || n_E <= 0) return hipSuccess;
  const double a = 1.0 / (M + 1);
  const double cot_pa = cos(M_PI * a) / sin(M_PI * a);
  // Estimated times beyond a launch's 6 us: k_kpm 0.5 ns + 0.65 ps a moment for each (row, energy), eight energies a
  // workgroup; k_kpm_rows the latency of its tiles, a moment 30 ns and 3 more for each of a workgroup's groups of rows, and 2
  // us.  331 sizes measured, 1 to 4096 rows, 8 to 4000 moments, 1 to 1001 energies: the one taken is at most 15 %
  // slower than the other.  k_kpm alone took 2313 us for 4096 rows, 8 moments and 1001 energies, where k_kpm_rows takes
  // 25; one row and 1000 moments take 7.8 and 20.
  int lE = kKpmRowsMinE;
  while (lE < 8 && (1 << lE) < n_E) ++lE;
  const int G = 256 >> lE;
  if (8.0 * R * ((n_E + 7) / 8) * (0.5e-3 + 6.5e-7 * M) > M * (0.03 + 0.003 * G) + 2.0) {
    const int rq = R >= 4 ? 4 : 1;
    const dim3 grid((n_E + (1 << lE) - 1) >> lE, (R + G * rq - 1) / (G * rq));
    const size_t lds = (size_t)G * (kKpmRowTile * rq + 2) * sizeof(double);
    auto* k = rq == 4 ? k_kpm_rows<4> : k_kpm_rows<1>;
    k<<<grid, 256, lds, s>>>(R, M, C, n_E, E, inv_dE, pref_base, jackson, cot_pa, lE, out);
    return hipGetLastError();
  }
  constexpr int per = kKpmWaves * kKpmEnergies;
  k_kpm<<<dim3((n_E + per - 1) / per, R), 64 * kKpmWaves, 0, s>>>(R, M, C, n_E, E, inv_dE, pref_base, jackson, cot_pa,
                                                   out);
  return hipGetLastError();
}

hipError_t launch_kpm_adjoint(int R, int M, const double* g, int n_E, const double* E, double inv_dE,
                              double pref_base, int jackson, double* out, hipStream_t s) {
  if (R <= 0 || M <= 0) return hipSuccess;
  const double a = 1.0 / (M + 1);
  const double cot_pa = cos(M_PI * a) / sin(M_PI * a);
  // threads sharing a group's energies: as many as there are energies, until the groups fill the chip (2^18
  // threads), and above 2^16 threads no fewer than four energies each.  Within 15 % of the best of 1 to 256 threads at the
  // 284 sizes of launch_kpm; 256 threads always took 2730 us for 4096 rows, 1000 moments and one energy, one takes 26.
  const int64_t groups = (int64_t)R * ((M + kKpmMoments - 1) / kKpmMoments);
  int lS = 8;
  while (lS > 0 && ((groups << lS) > (1 << 18) || (1 << lS) > n_E || ((groups << lS) > (1 << 16) && (4 << lS) > n_E))) --lS;
  const int per = 256 >> lS;   // groups a workgroup
  const size_t lds = sizeof(double) * kKpmMoments * (256 >> (lS < 6 ? lS : 6));
  k_kpm_adjoint<<<dim3((unsigned)((groups + per - 1) / per)), 256, lds, s>>>(R, M, g, n_E, E, inv_dE, pref_base, jackson,
                                                                           cot_pa, lS, out);
  return hipGetLastError();
}

}  // namespace gpuqt
