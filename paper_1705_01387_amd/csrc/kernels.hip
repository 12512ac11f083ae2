// HIP kernels for gfx950 (CDNA4): the sparse Chebyshev steps of the
// linear-scaling Kubo method and their helpers.
//
// Every sparse kernel streams the sliced-ELL Hamiltonian once per launch:
// one row (for B > 1, one (row, column) pair per lane with the B lanes of a
// row adjacent) per lane, slot-major entries so that a wavefront reading one
// slot of consecutive rows touches consecutive addresses, 16-byte loads of
// complex128 vector elements, FP64 throughout (no MFMA: a step moves about
// 20 bytes per FP64 multiply-add pair, far below the matrix-core balance).
//
// Schedule: G workgroups of 256 threads.  The hardware hands workgroups to
// the 8 XCDs round-robin, so physical workgroup p becomes logical workgroup
// (p % 8) * (G / 8) + p / 8; the logical workgroups of one XCD that work on
// one segment form a group owning a contiguous row range, and walk it in
// tiles of 256/B rows with stride "group size".  All workgroups resident on
// an XCD therefore sweep one compact window of rows together: a neighbour
// gather (e.g. one lattice plane away) finds the line its neighbours fetched
// moments ago in that XCD's L2 or in the last-level cache, instead of
// re-reading it from HBM.
//
// NT variants mark the once-read streams (indices, hoppings, position
// differences, on-site terms, v_{n-2}, phi_L) non-temporal so that they do
// not push the gathered vector out of the caches.
//
// Moment reductions are deterministic: wavefront butterfly, then a fixed
// order over the four wavefronts, one partial per workgroup and step, and a
// fixed-shape final reduction over workgroups.
#include <hip/hip_runtime.h>

#include <algorithm>

#include <type_traits>

#include "bessel.h"
#include "internal.h"

#include "device_common.h"

namespace gpuqt {

using namespace dev;

namespace {

// ---------------------------------------------------------------------------
// Chebyshev moment step (Sections 3.2-3.3): v_n = 2 H~ v_{n-1} - v_{n-2}
// (v_1 = H~ v_0) and the workgroup's part of <phiL|v_n> (and <phiL|v_0>).
// ---------------------------------------------------------------------------
template <int B, int HOP, int K, bool NT>
__global__ __launch_bounds__(kBlock) void k_moment_step(DevMat A, StepIO io,
                                                        const double2* __restrict__ phiL,
                                                        double2* __restrict__ part_n,
                                                        double2* __restrict__ part_0) {
  const int lb = logical_block(A.G);
  const BlkPlan P = A.plan[lb];
  const double hu = (HOP == HOP_UNIFORM) ? A.seg_hop[P.seg] : 0.0;
  const int b = threadIdx.x & (B - 1);
  const double2* __restrict__ x = io.x;
  const double2* __restrict__ w = io.w;
  double2* __restrict__ out = io.out;
  const bool first = io.first;
  // per-row operands that need no column index are loaded first (w is read
  // from x on the first step, where it is unused, to keep the load unconditional)
  const double2* __restrict__ wsrc = first ? x : w;
  double dr = 0.0, di = 0.0, zr = 0.0, zi = 0.0;
  for_rows_pf<B, HOP, K, NT>(A, P, [&](int64_t r, const int32_t* kc) {
    const int64_t idx = r * B + b;
    const double2 xr = x[idx];
    const double2 wv = ld2<NT>(wsrc + idx);
    double2 p = make_double2(0.0, 0.0);
    if (phiL) p = ld2<NT>(phiL + idx);   // plain recurrence step (no moment) when phiL is NULL
    double2 ha, hb, da;
    row_apply<B, HOP, K, NT, false, false, true>(A, r, b, hu, x, nullptr, xr, xr, ha, hb, da, kc);
    const double2 y = first ? ha : twice_minus(ha, wv);
    out[idx] = y;
    if (phiL) {
      cdot_acc(dr, di, p, y);
      if (first) cdot_acc(zr, zi, p, xr);
    }
  });
  if (!phiL) return;
  block_reduce_store<B>(dr, di, part_n + (int64_t)lb * B);
  if (first) {
    __syncthreads();
    block_reduce_store<B>(zr, zi, part_0 + (int64_t)lb * B);
  }
}

// ---------------------------------------------------------------------------
// Moment step for a Hermitian moment set (phiL = phiR = v_0): the same
// recurrence, but the moments come from the product identities
//   T_{2k} = 2 T_k T_k - T_0,   T_{2k-1} = 2 T_k T_{k-1} - T_1,
// so step k yields the raw dots <v_k|v_{k-1}> (row 2k-1) and <v_k|v_k>
// (row 2k); the first step also <v_0|v_0> (row 0) and <v_0|v_1> (row 1).
// k_reduce turns raw rows n >= 2 into 2 raw_n - mu_{n mod 2}.  Half the
// steps of the plain recurrence, and no phi_L stream.
// ---------------------------------------------------------------------------
template <int B, int HOP, int K, bool NT>
__global__ __launch_bounds__(kBlock) void k_moment_step_sym(DevMat A, StepIO io,
                                                            double2* __restrict__ part_a,
                                                            double2* __restrict__ part_b,
                                                            double2* __restrict__ part_c) {
  const int lb = logical_block(A.G);
  const BlkPlan P = A.plan[lb];
  const double hu = (HOP == HOP_UNIFORM) ? A.seg_hop[P.seg] : 0.0;
  const int b = threadIdx.x & (B - 1);
  const double2* __restrict__ x = io.x;
  const double2* __restrict__ w = io.w;
  double2* __restrict__ out = io.out;
  const bool first = io.first;
  // first: a = <v0|v0>, b = <v0|v1>, c = <v1|v1>;  else: a = <vk|vk-1>, c = <vk|vk>
  const double2* __restrict__ wsrc = first ? x : w;   // w unused on the first step
  double ar = 0.0, ai = 0.0, br = 0.0, bi = 0.0, cr = 0.0, ci = 0.0;
  for_rows_pf<B, HOP, K, NT>(A, P, [&](int64_t r, const int32_t* kc) {
    const int64_t idx = r * B + b;
    const double2 xr = x[idx];
    double2 ha, hb, da;
    row_apply<B, HOP, K, NT, false, false, true>(A, r, b, hu, x, nullptr, xr, xr, ha, hb, da, kc);
    const double2 wv = ld2<NT>(wsrc + idx);
    const double2 y = first ? ha : twice_minus(ha, wv);
    out[idx] = y;
    if (first) {
      cdot_acc(ar, ai, xr, xr);
      cdot_acc(br, bi, xr, y);
    } else {
      cdot_acc(ar, ai, y, xr);
    }
    cdot_acc(cr, ci, y, y);
  });
  block_reduce_store<B>(ar, ai, part_a + (int64_t)lb * B);
  __syncthreads();
  block_reduce_store<B>(cr, ci, part_c + (int64_t)lb * B);
  if (first) {
    __syncthreads();
    block_reduce_store<B>(br, bi, part_b + (int64_t)lb * B);
  }
}

// ---------------------------------------------------------------------------
// Moment step for <a|T_n|b> with a != b: both chains a_k = T_k a, b_k = T_k b
// advance in one launch (one matrix read, the two gathers share the indices)
// and the identities give
//   <a|T_{2k}|b> = 2 <a_k|b_k> - <a|b>,  <a|T_{2k-1}|b> = 2 <a_k|b_{k-1}> - <a|T_1 b>,
// so step k yields <a_k|b_{k-1}> (row 2k-1) and <a_k|b_k> (row 2k); the first
// step also <a|b> (row 0) and <a|b_1> (row 1).
// ---------------------------------------------------------------------------
template <int B, int HOP, int K, bool NT>
__global__ __launch_bounds__(kBlock) void k_moment_step_pair(DevMat A, ChainIO io,
                                                             double2* __restrict__ part_a,
                                                             double2* __restrict__ part_b,
                                                             double2* __restrict__ part_c) {
  const int lb = logical_block(A.G);
  const BlkPlan P = A.plan[lb];
  const double hu = (HOP == HOP_UNIFORM) ? A.seg_hop[P.seg] : 0.0;
  const int b = threadIdx.x & (B - 1);
  const bool first = io.first;
  const double2* __restrict__ wa = first ? io.xa : io.wa;   // unused on the first step
  const double2* __restrict__ wb = first ? io.xb : io.wb;
  double ar = 0.0, ai = 0.0, br = 0.0, bi = 0.0, cr = 0.0, ci = 0.0;
  for_rows_pf<B, HOP, K, NT>(A, P, [&](int64_t r, const int32_t* kc) {
    const int64_t idx = r * B + b;
    const double2 xa = io.xa[idx];
    const double2 xb = io.xb[idx];
    const double2 wav = ld2<NT>(wa + idx);
    const double2 wbv = ld2<NT>(wb + idx);
    double2 ha, hb, da;
    row_apply<B, HOP, K, NT, true, false, true>(A, r, b, hu, io.xa, io.xb, xa, xb, ha, hb, da, kc);
    const double2 ya = first ? ha : twice_minus(ha, wav);
    const double2 yb = first ? hb : twice_minus(hb, wbv);
    io.oa[idx] = ya;
    io.ob[idx] = yb;
    if (first) {
      cdot_acc(ar, ai, xa, xb);
      cdot_acc(br, bi, xa, yb);
    } else {
      cdot_acc(ar, ai, ya, xb);
    }
    cdot_acc(cr, ci, ya, yb);
  });
  block_reduce_store<B>(ar, ai, part_a + (int64_t)lb * B);
  __syncthreads();
  block_reduce_store<B>(cr, ci, part_c + (int64_t)lb * B);
  if (first) {
    __syncthreads();
    block_reduce_store<B>(br, bi, part_b + (int64_t)lb * B);
  }
}

// ---------------------------------------------------------------------------
// One term m of U(dt) psi = sum_m c_m T_m(H~) psi (Section 3.2):
// a_m by the recurrence, acc += c_m a_m; c_m = J[seg][m] * phase_m with the
// table holding (2 - delta_m0) J_m(DeltaE_seg |dt|).
// ---------------------------------------------------------------------------
template <int B, int HOP, int K, bool NT>
__global__ __launch_bounds__(kBlock) void k_evolve_term(DevMat A, StepIO io, double2* __restrict__ acc,
                                                        const double* __restrict__ Jtab, int ldJ,
                                                        int m, double2 ph_m, double2 ph_0) {
  const BlkPlan P = A.plan[logical_block(A.G)];
  const double hu = (HOP == HOP_UNIFORM) ? A.seg_hop[P.seg] : 0.0;
  const double2 cm = cscale(Jtab[(int64_t)P.seg * ldJ + m], ph_m);
  const double2 c0 = cscale(Jtab[(int64_t)P.seg * ldJ], ph_0);
  const int b = threadIdx.x & (B - 1);
  const double2* __restrict__ x = io.x;
  const double2* __restrict__ w = io.w;
  double2* __restrict__ out = io.out;
  const bool first = io.first;
  // w and acc are unused on the first step: read x there instead, so that the
  // loads stay unconditional and ahead of the gathers
  const double2* __restrict__ wsrc = first ? x : w;
  const double2* __restrict__ asrc = first ? x : acc;
  for_rows_pf<B, HOP, K, NT>(A, P, [&](int64_t r, const int32_t* kc) {
    const int64_t idx = r * B + b;
    const double2 xr = x[idx];
    const double2 wv = ld2<NT>(wsrc + idx);
    const double2 av = ld2<NT>(asrc + idx);
    double2 ha, hb, da;
    row_apply<B, HOP, K, NT, false, false, true>(A, r, b, hu, x, nullptr, xr, xr, ha, hb, da, kc);
    if (first) {
      out[idx] = ha;
      acc[idx] = cadd(cmul(c0, xr), cmul(cm, ha));
    } else {
      const double2 y = twice_minus(ha, wv);
      out[idx] = y;
      acc[idx] = cadd(av, cmul(cm, y));
    }
  });
}

// ---------------------------------------------------------------------------
// One term m of U(dt) applied to two vectors at once (both VAC states advance
// with the same U(-dt), Section 3.3): chains a_m = T_m psi_a, b_m = T_m psi_b
// share the matrix read and the gather indices; acc_a += c_m a_m,
// acc_b += c_m b_m.
// ---------------------------------------------------------------------------
template <int B, int HOP, int K, bool NT>
__global__ __launch_bounds__(kBlock) void k_evolve_pair_term(DevMat A, ChainIO io, double2* __restrict__ acc_a,
                                                             double2* __restrict__ acc_b,
                                                             const double* __restrict__ Jtab, int ldJ, int m,
                                                             double2 ph_m, double2 ph_0) {
  const BlkPlan P = A.plan[logical_block(A.G)];
  const double hu = (HOP == HOP_UNIFORM) ? A.seg_hop[P.seg] : 0.0;
  const double2 cm = cscale(Jtab[(int64_t)P.seg * ldJ + m], ph_m);
  const double2 c0 = cscale(Jtab[(int64_t)P.seg * ldJ], ph_0);
  const int b = threadIdx.x & (B - 1);
  const bool first = io.first;
  // the w and acc operands are unused on the first step (read x there instead)
  const double2* __restrict__ wa = first ? io.xa : io.wa;
  const double2* __restrict__ wb = first ? io.xb : io.wb;
  const double2* __restrict__ sa = first ? io.xa : acc_a;
  const double2* __restrict__ sb = first ? io.xb : acc_b;
  for_rows_pf<B, HOP, K, NT>(A, P, [&](int64_t r, const int32_t* kc) {
    const int64_t idx = r * B + b;
    const double2 xa = io.xa[idx];
    const double2 xb = io.xb[idx];
    const double2 wav = ld2<NT>(wa + idx);
    const double2 wbv = ld2<NT>(wb + idx);
    const double2 aav = ld2<NT>(sa + idx);
    const double2 abv = ld2<NT>(sb + idx);
    double2 ha, hb, da;
    row_apply<B, HOP, K, NT, true, false, true>(A, r, b, hu, io.xa, io.xb, xa, xb, ha, hb, da, kc);
    if (first) {
      io.oa[idx] = ha;
      io.ob[idx] = hb;
      acc_a[idx] = cadd(cmul(c0, xa), cmul(cm, ha));
      acc_b[idx] = cadd(cmul(c0, xb), cmul(cm, hb));
    } else {
      const double2 ya = twice_minus(ha, wav);
      const double2 yb = twice_minus(hb, wbv);
      io.oa[idx] = ya;
      io.ob[idx] = yb;
      acc_a[idx] = cadd(aav, cmul(cm, ya));
      acc_b[idx] = cadd(abv, cmul(cm, yb));
    }
  });
}

// ---------------------------------------------------------------------------
// One term m of the fused evolution + commutator series (Section 3.2):
//   a_m = T_m psi:                a_1 = H~ a_0,  a_m = 2 H~ a_{m-1} - a_{m-2}
//   b_m = [X,T_m] psi + T_m chi:  b_0 = chi, b_1 = [X,H~] a_0 + H~ b_0,
//                                 b_m = 2 [X,H~] a_{m-1} + 2 H~ b_{m-1} - b_{m-2}
// (the sum of the paper's [X,T_m] recurrence and the T_m recurrence applied to
// chi); acc_a += c_m a_m, acc_b += c_m b_m.  [X,H~]_rj = -dx_rj H~_rj.
// ---------------------------------------------------------------------------
template <int B, int HOP, int K, bool NT>
__global__ __launch_bounds__(kBlock) void k_msd_term(DevMat A, ChainIO io, double2* __restrict__ acc_a,
                                                     double2* __restrict__ acc_b,
                                                     const double* __restrict__ Jtab, int ldJ, int m,
                                                     double2 ph_m, double2 ph_0) {
  const BlkPlan P = A.plan[logical_block(A.G)];
  const double hu = (HOP == HOP_UNIFORM) ? A.seg_hop[P.seg] : 0.0;
  const double2 cm = cscale(Jtab[(int64_t)P.seg * ldJ + m], ph_m);
  const double2 c0 = cscale(Jtab[(int64_t)P.seg * ldJ], ph_0);
  const int b = threadIdx.x & (B - 1);
  const bool first = io.first;
  // the w and acc operands are unused on the first step (read x there instead)
  const double2* __restrict__ wa = first ? io.xa : io.wa;
  const double2* __restrict__ wb = first ? io.xb : io.wb;
  const double2* __restrict__ sa = first ? io.xa : acc_a;
  const double2* __restrict__ sb = first ? io.xb : acc_b;
  for_rows_pf<B, HOP, K, NT>(A, P, [&](int64_t r, const int32_t* kc) {
    const int64_t idx = r * B + b;
    const double2 xa = io.xa[idx];
    const double2 xb = io.xb[idx];
    const double2 wav = ld2<NT>(wa + idx);
    const double2 wbv = ld2<NT>(wb + idx);
    const double2 aav = ld2<NT>(sa + idx);
    const double2 abv = ld2<NT>(sb + idx);
    double2 ha, hb, da;
    row_apply<B, HOP, K, NT, true, true, true>(A, r, b, hu, io.xa, io.xb, xa, xb, ha, hb, da, kc);
    const double2 g = make_double2(hb.x - da.x, hb.y - da.y);   // [X,H~] a + H~ b
    if (first) {
      io.oa[idx] = ha;
      io.ob[idx] = g;
      acc_a[idx] = cadd(cmul(c0, xa), cmul(cm, ha));
      acc_b[idx] = cadd(cmul(c0, xb), cmul(cm, g));
    } else {
      const double2 ya = twice_minus(ha, wav);
      const double2 yb = twice_minus(g, wbv);
      io.oa[idx] = ya;
      io.ob[idx] = yb;
      acc_a[idx] = cadd(aav, cmul(cm, ya));
      acc_b[idx] = cadd(abv, cmul(cm, yb));
    }
  });
}

// ---------------------------------------------------------------------------
// Velocity V x (i sum dx H x) or [X,H] x (-sum dx H x), unscaled H
// (Section 4.2).  Stored values are H~ = H / DeltaE_seg, so multiply back.
// ---------------------------------------------------------------------------
template <int B, int HOP>
__global__ __launch_bounds__(kBlock) void k_commutator(DevMat A, int which, const double2* __restrict__ x,
                                                       double2* __restrict__ out) {
  const BlkPlan P = A.plan[logical_block(A.G)];
  const double hu = (HOP == HOP_UNIFORM) ? A.seg_hop[P.seg] : 0.0;
  const double e = A.seg_dE[P.seg];
  const int b = threadIdx.x & (B - 1);
  for_rows<B>(A, P, [&](int64_t r) {
    double2 ha, hb, da;
    const double2 z = make_double2(0.0, 0.0);   // no diagonal term: own element unused
    row_apply<B, HOP, 0, false, false, true, false>(A, r, b, hu, x, nullptr, z, z, ha, hb, da);
    const int64_t idx = r * B + b;
    double2 y;
    if ((which & 1) == GPUQT_VELOCITY) {
      y = make_double2(-e * da.y, e * da.x);   // i * e * da
    } else {
      y = make_double2(-e * da.x, -e * da.y);
    }
    out[idx] = (which & kAccumulate) ? cadd(out[idx], y) : y;
  });
}

// out = J_0(seg) * in, or zero when in is NULL.
template <int B>
__global__ __launch_bounds__(kBlock) void k_scale(DevMat A, const double2* __restrict__ in,
                                                  double2* __restrict__ out,
                                                  const double* __restrict__ Jtab, int ldJ) {
  const BlkPlan P = A.plan[logical_block(A.G)];
  const double j0 = Jtab ? Jtab[(int64_t)P.seg * ldJ] : 0.0;
  const int b = threadIdx.x & (B - 1);
  for_rows<B>(A, P, [&](int64_t r) {
    const int64_t idx = r * B + b;
    out[idx] = in ? cscale(j0, in[idx]) : make_double2(0.0, 0.0);
  });
}

// out = exp(i theta) with theta = 2 pi frac(0.618... idx + 0.414... b): a
// deterministic unit-modulus test vector (used only to time kernel variants).
template <int B>
__global__ __launch_bounds__(kBlock) void k_fill_phase(DevMat A, double2* __restrict__ out) {
  const BlkPlan P = A.plan[logical_block(A.G)];
  const int b = threadIdx.x & (B - 1);
  for_rows<B>(A, P, [&](int64_t r) {
    const double t = (double)r * 0.6180339887498949 + (double)b * 0.4142135623730951;
    double s, c;
    sincospi(2.0 * (t - floor(t)), &s, &c);
    out[r * B + b] = make_double2(c, s);
  });
}

__global__ void k_bessel_table(const double* __restrict__ seg_dE, int n_seg, double abs_dt, int Np,
                               int ldJ, double* __restrict__ J) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n_seg) return;
  double* row = J + (int64_t)s * ldJ;
  bessel_miller(seg_dE[s] * abs_dt, Np, row);
  for (int m = 1; m < Np; ++m) row[m] *= 2.0;
}

// Sum of one partial row over the segment's workgroups, fixed order.
__device__ __forceinline__ double2 reduce_row(const double2* __restrict__ part, int k, int G, int B, int b,
                                              int g0, int g1) {
  double re = 0.0, im = 0.0;
  for (int g = g0 + (int)threadIdx.x; g < g1; g += 64) {
    const double2 v = part[((int64_t)k * G + g) * B + b];
    re += v.x;
    im += v.y;
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    re += __shfl_xor(re, off);
    im += __shfl_xor(im, off);
  }
  return make_double2(re, im);
}

// One wavefront per (moment k, segment*B + b): sum the segment's workgroup
// partials in a fixed order.  sym: rows hold the raw dots of
// k_moment_step_sym, and moment k >= 2 is 2 raw_k - mu_{k mod 2}.
__global__ __launch_bounds__(64) void k_reduce(const double2* __restrict__ part, int M, int G, int B,
                                               const int32_t* __restrict__ seg_blk0, int sym,
                                               double2* __restrict__ out, double* __restrict__ out_real) {
  const int k = blockIdx.x;
  const int sb = blockIdx.y;
  const int seg = sb / B, b = sb - seg * B;
  const int g0 = seg_blk0[seg], g1 = seg_blk0[seg + 1];
  const double2 v = reduce_row(part, k, G, B, b, g0, g1);
  double re = v.x, im = v.y;
  if (sym && k >= 2) {
    const double2 u = reduce_row(part, k & 1, G, B, b, g0, g1);
    re = 2.0 * re - u.x;
    im = 2.0 * im - u.y;
  }
  if (threadIdx.x == 0) {
    const int64_t o = (int64_t)sb * M + k;
    if (out) out[o] = make_double2(re, im);
    if (out_real) out_real[o] = re;
  }
}

// Transport regimes of Section 2.2 (e = hbar = 1), one energy per thread:
// sigma_sc = max over the rows of the running conductivity (NaN rows skipped),
// v = sqrt(C_vv(E, 0)), tau = sigma_sc / (rho v^2), mfp = v tau,
// L(t) = 2 sqrt(DeltaX^2(t)), xi = L(t_last) / (2 pi); C_vv and DeltaX^2 are the
// reconstructed rows (rho C_vv, rho DeltaX^2) divided by rho.  NaN where rho <= 0,
// C_vv(E, 0) < 0 (v), rho v^2 <= 0 (tau, mfp) or DeltaX^2 < 0 (L, xi).
__global__ __launch_bounds__(256) void k_transport(TransportIO io) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= io.n_E) return;
  const double nan = __longlong_as_double(0x7ff8000000000000ll);
  const double r = io.rho[e];
  const bool ok = r > 0.0;
  double sc = nan;
  if (io.sigma) {
    for (int k = 0; k < io.n_t; ++k) {
      const double x = io.sigma[(int64_t)k * io.n_E + e];
      if (x == x && (sc != sc || x > sc)) sc = x;
    }
    if (io.sigma_sc) io.sigma_sc[e] = sc;
  }
  if (io.vac0) {
    const double c0 = io.vac0[e];
    const double cvv = ok ? c0 / r : nan;
    const double v = cvv >= 0.0 ? sqrt(cvv) : nan;
    if (io.v) io.v[e] = v;
    if (io.sigma) {
      const double tau = (ok && c0 > 0.0) ? sc / c0 : nan;
      if (io.tau) io.tau[e] = tau;
      if (io.mfp) io.mfp[e] = v * tau;
    }
  }
  if (io.msd) {
    double L = nan;
    for (int k = 0; k < io.n_t; ++k) {
      const double dx2 = ok ? io.msd[(int64_t)k * io.n_E + e] / r : nan;
      L = dx2 >= 0.0 ? 2.0 * sqrt(dx2) : nan;
      if (io.L) io.L[(int64_t)k * io.n_E + e] = L;
    }
    if (io.xi) io.xi[e] = io.n_t > 0 ? L / (2.0 * M_PI) : nan;
  }
}

// Running conductivity (Section 2.2) over the time rows, one energy per thread:
// mode 0 (VAC): trapezoid integral of rows at t_k = sum_{j<k} dt_j, sigma_0 = 0;
// mode 1 (MSD): (y_k - y_{k-1}) / (2 dt_k), y_{-1} = 0 (NaN for dt_k = 0).
__global__ __launch_bounds__(256) void k_sigma(int mode, int n_t, const double* __restrict__ dt, int n_E,
                                               const double* __restrict__ y, double* __restrict__ out) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n_E) return;
  if (mode == 0) {
    double acc = 0.0, prev = y[e];
    out[e] = 0.0;
    for (int k = 1; k < n_t; ++k) {
      const double cur = y[(int64_t)k * n_E + e];
      acc += 0.5 * dt[k - 1] * (prev + cur);
      out[(int64_t)k * n_E + e] = acc;
      prev = cur;
    }
  } else {
    double prev = 0.0;
    for (int k = 0; k < n_t; ++k) {
      const double cur = y[(int64_t)k * n_E + e];
      out[(int64_t)k * n_E + e] = dt[k] != 0.0 ? (cur - prev) / (2.0 * dt[k]) : __builtin_nan("");
      prev = cur;
    }
  }
}

// Bandwidth probe: one 16-byte element per thread over a grid that covers the
// whole buffer (every element's load is in flight at once, as far as the chip
// holds them; no loop-carried address arithmetic).
__global__ __launch_bounds__(256) void k_copy(const double2* __restrict__ src, double2* __restrict__ dst,
                                              size_t n) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = src[i];
}

}  // namespace


// ----------------------------------------------------------------------------
// launchers
// ----------------------------------------------------------------------------

int kernel_occupancy(int family, const DevMat& A, int hop_mode, int B, int nt) {
  int nb = 0;
  auto q = [&](auto fn) {
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fn, kBlock, 0) != hipSuccess) nb = 0;
  };
  (void)dispatch_sparse(A, hop_mode, B, nt, [&](auto Bc, auto Hc, auto Kc, auto NTc) {
    constexpr int b = decltype(Bc)::value, hm = decltype(Hc)::value, k = decltype(Kc)::value;
    constexpr bool n = decltype(NTc)::value;
    switch (family) {
      case FAM_MOMENT: q(k_moment_step<b, hm, k, n>); break;
      case FAM_SYM: q(k_moment_step_sym<b, hm, k, n>); break;
      case FAM_PAIR: q(k_moment_step_pair<b, hm, k, n>); break;
      case FAM_EVOLVE: q(k_evolve_term<b, hm, k, n>); break;
      case FAM_EVOLVE_PAIR: q(k_evolve_pair_term<b, hm, k, n>); break;
      default: q(k_msd_term<b, hm, k, n>); break;
    }
  });
  (void)hipGetLastError();
  return nb;
}

hipError_t launch_moment_step(const DevMat& A, int hop_mode, int B, const StepIO& io,
                              const double2* phiL, double2* part_n, double2* part_0, hipStream_t s) {
  return dispatch_sparse(A, hop_mode, B, A.nt, [&](auto Bc, auto Hc, auto Kc, auto NTc) {
    k_moment_step<decltype(Bc)::value, decltype(Hc)::value, decltype(Kc)::value, decltype(NTc)::value>
        <<<dim3(A.G), kBlock, 0, s>>>(A, io, phiL, part_n, part_0);
  });
}

hipError_t launch_evolve_term(const DevMat& A, int hop_mode, int B, const StepIO& io, double2* acc,
                              const double* Jtab, int ldJ, int m, double2 phase_m, double2 phase_0,
                              hipStream_t s) {
  return dispatch_sparse(A, hop_mode, B, A.nt, [&](auto Bc, auto Hc, auto Kc, auto NTc) {
    k_evolve_term<decltype(Bc)::value, decltype(Hc)::value, decltype(Kc)::value, decltype(NTc)::value>
        <<<dim3(A.G), kBlock, 0, s>>>(A, io, acc, Jtab, ldJ, m, phase_m, phase_0);
  });
}

hipError_t launch_msd_term(const DevMat& A, int hop_mode, int B, const ChainIO& io, double2* acc_a,
                           double2* acc_b, const double* Jtab, int ldJ, int m, double2 phase_m,
                           double2 phase_0, hipStream_t s) {
  return dispatch_sparse(A, hop_mode, B, A.nt, [&](auto Bc, auto Hc, auto Kc, auto NTc) {
    k_msd_term<decltype(Bc)::value, decltype(Hc)::value, decltype(Kc)::value, decltype(NTc)::value>
        <<<dim3(A.G), kBlock, 0, s>>>(A, io, acc_a, acc_b, Jtab, ldJ, m, phase_m, phase_0);
  });
}

hipError_t launch_evolve_pair_term(const DevMat& A, int hop_mode, int B, const ChainIO& io, double2* acc_a,
                                   double2* acc_b, const double* Jtab, int ldJ, int m, double2 phase_m,
                                   double2 phase_0, hipStream_t s) {
  return dispatch_sparse(A, hop_mode, B, A.nt, [&](auto Bc, auto Hc, auto Kc, auto NTc) {
    k_evolve_pair_term<decltype(Bc)::value, decltype(Hc)::value, decltype(Kc)::value, decltype(NTc)::value>
        <<<dim3(A.G), kBlock, 0, s>>>(A, io, acc_a, acc_b, Jtab, ldJ, m, phase_m, phase_0);
  });
}

hipError_t launch_commutator(const DevMat& A, int hop_mode, int B, int which, const double2* x,
                             double2* out, hipStream_t s) {
  return dispatch_bh(B, hop_mode, [&](auto Bc, auto Hc) {
    k_commutator<decltype(Bc)::value, decltype(Hc)::value><<<dim3(A.G), kBlock, 0, s>>>(A, which, x, out);
  });
}

hipError_t launch_scale(const DevMat& A, int B, const double2* in, double2* out, const double* Jtab,
                        int ldJ, hipStream_t s) {
  return dispatch_bh(B, HOP_UNIFORM, [&](auto Bc, auto) {
    k_scale<decltype(Bc)::value><<<dim3(A.G), kBlock, 0, s>>>(A, in, out, Jtab, ldJ);
  });
}

hipError_t launch_fill_phase(const DevMat& A, int B, double2* out, hipStream_t s) {
  return dispatch_bh(B, HOP_UNIFORM, [&](auto Bc, auto) {
    k_fill_phase<decltype(Bc)::value><<<dim3(A.G), kBlock, 0, s>>>(A, out);
  });
}

hipError_t launch_bessel_table(const double* seg_dE, int n_seg, double abs_dt, int Np, int ldJ,
                               double* J, hipStream_t s) {
  const int threads = 64;
  const int blocks = (n_seg + threads - 1) / threads;
  k_bessel_table<<<blocks, threads, 0, s>>>(seg_dE, n_seg, abs_dt, Np, ldJ, J);
  return hipGetLastError();
}

hipError_t launch_reduce_moments(const double2* part, int M, int G, int B, int n_seg,
                                 const int32_t* seg_blk0_dev, int sym, double2* out, double* out_real,
                                 hipStream_t s) {
  if (M <= 0) return hipSuccess;
  k_reduce<<<dim3(M, n_seg * B), 64, 0, s>>>(part, M, G, B, seg_blk0_dev, sym, out, out_real);
  return hipGetLastError();
}

hipError_t launch_moment_step_pair(const DevMat& A, int hop_mode, int B, const ChainIO& io,
                                   double2* part_a, double2* part_b, double2* part_c, hipStream_t s) {
  return dispatch_sparse(A, hop_mode, B, A.nt, [&](auto Bc, auto Hc, auto Kc, auto NTc) {
    k_moment_step_pair<decltype(Bc)::value, decltype(Hc)::value, decltype(Kc)::value,
                       decltype(NTc)::value><<<dim3(A.G), kBlock, 0, s>>>(A, io, part_a, part_b, part_c);
  });
}

hipError_t launch_moment_step_sym(const DevMat& A, int hop_mode, int B, const StepIO& io,
                                  double2* part_a, double2* part_b, double2* part_c, hipStream_t s) {
  return dispatch_sparse(A, hop_mode, B, A.nt, [&](auto Bc, auto Hc, auto Kc, auto NTc) {
    k_moment_step_sym<decltype(Bc)::value, decltype(Hc)::value, decltype(Kc)::value,
                      decltype(NTc)::value><<<dim3(A.G), kBlock, 0, s>>>(A, io, part_a, part_b, part_c);
  });
}

hipError_t launch_transport(const TransportIO& io, hipStream_t s) {
  if (io.n_E <= 0) return hipSuccess;
  k_transport<<<dim3((io.n_E + 255) / 256), 256, 0, s>>>(io);
  return hipGetLastError();
}

hipError_t launch_sigma(int mode, int n_t, const double* dt, int n_E, const double* y, double* out,
                        hipStream_t s) {
  if (n_t <= 0 || n_E <= 0) return hipSuccess;
  k_sigma<<<dim3((n_E + 255) / 256), 256, 0, s>>>(mode, n_t, dt, n_E, y, out);
  return hipGetLastError();
}

hipError_t launch_copy(const double2* src, double2* dst, size_t n16, hipStream_t s) {
  if (n16 == 0) return hipSuccess;
  const size_t blocks = (n16 + 255) / 256;
  if (blocks > 0x7fffffffu) return hipErrorInvalidValue;
  k_copy<<<dim3((unsigned)blocks), 256, 0, s>>>(src, dst, n16);
  return hipGetLastError();
}

}  // namespace gpuqt
