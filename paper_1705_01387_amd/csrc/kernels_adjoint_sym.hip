// Reverse steps of the Hermitian moments (kernels_adjoint.hip has the recurrence and the single chain).
#include <hip/hip_runtime.h>

#include "device_common.h"
#include "reverse_core.h"

namespace gpuqt {

using namespace dev;

namespace {

// Reverse step of the Hermitian form (phiL = phiR, one chain a_k = T_k phi):
// with both chains equal the two adjoints only enter through their sum
// cbar_k = abar_k + bbar_k,
//   cbar_k = 2 om_2k a_k + om_2k-1 a_{k-1} + om_2k+1 a_{k+1} + f_rec H~ cbar_{k+1} - cbar_{k+2},
// and the parameter terms are Re sum_k f_k <cbar_k| dH~/dp a_{k-1}>: one chain
// gathered instead of two.  At k = 0 the output is cbar_0 / 2 = sum_n w_n T_n phi
// (abar_0 = bbar_0).  Fields of io: xa, wa, oa, acc_a, a_m1, a_k, a_p1 and the
// weights; the b fields are unused.
template <int B, int HOP, int K, int NC, bool TR>
__global__ __launch_bounds__(kBlock) void k_adjoint_sym_step(DevMat A, AdjPairIO io) {
  const int lb = logical_block(A.G);
  const BlkPlan P = A.plan[lb];
  const double hu = (HOP == HOP_UNIFORM) ? A.seg_hop[P.seg] : 0.0;
  const double inv_dE = 1.0 / A.seg_dE[P.seg];
  const int b = threadIdx.x & (B - 1);
  const double* om = io.om + ((int64_t)P.seg * B + b) * io.R;
  const int k2 = 2 * io.k;
  const double w0 = 2.0 * om[k2];
  const double wm = io.k >= 1 ? om[k2 - 1] : 0.0;
  const double wp = (io.a_p1 && k2 + 1 < io.R) ? om[k2 + 1] : 0.0;
  const double out_scale = io.k == 0 ? 0.5 : 1.0;
  const bool grad = io.gU != nullptr && (TR ? io.xa != nullptr : io.k >= 1);
  const int S = 1 << A.S_log2;
  double gc[NC > 0 ? NC : 1];
#pragma unroll
  for (int c = 0; c < (NC > 0 ? NC : 1); ++c) gc[c] = 0.0;
  for_rows<B>(A, P, [&](int64_t r) {
    const int64_t idx = r * B + b;
    const int64_t sl = r >> A.S_log2;
    const int64_t p0 = A.slice_ptr[sl];
    const int64_t e0 = p0 + (r & (S - 1));
    const int w = K > 0 ? K : (int)((A.slice_ptr[sl + 1] - p0) >> A.S_log2);
    double2 h = make_double2(0.0, 0.0);
    double2 hv[NC > 0 ? NC : 1];
#pragma unroll
    for (int c = 0; c < (NC > 0 ? NC : 1); ++c) hv[c] = make_double2(0.0, 0.0);
    constexpr bool AHEAD = TR || NC == 0;   // gU read ahead of the products
    double gu0 = 0.0;
    if (AHEAD && grad && b == 0) gu0 = io.gU[r];
    auto mul = [](double2 he, double2 y) {
      return (HOP == HOP_COMPLEX || HOP == HOP_DICT) ? cmul(he, y) : cscale(he.x, y);
    };
    auto add_class = [&](int64_t e, bool ok, double2 y) {
      const double2 t = mul(hop0_entry<HOP>(A, e, ok, P.seg), y);
      const int cls = NC > 1 && (TR || ok) ? io.cls[HOP == HOP_DICT ? (int64_t)A.hidx[e] : e] : 0;   // (padding adds zero)
#pragma unroll
      for (int q = 0; q < (NC > 0 ? NC : 1); ++q) {
        if constexpr (TR) {
          hv[q].x += q == cls ? t.x : 0.0;
          hv[q].y += q == cls ? t.y : 0.0;
        } else if (q == cls) {
          hv[q] = cadd(hv[q], t);
        }
      }
    };
    if constexpr (NC > 0 && !TR) {
      if (io.xa) h = cscale(A.diag[r], io.xa[idx]);
      for (int j = 0; j < w; ++j) {
        const int64_t e = e0 + (int64_t)j * S;
        int64_t cc;
        const bool ok = col_entry<HOP>(A, r, e, &cc);
        const double2 he = hop_entry<HOP>(A, e, ok, hu);
        if (io.xa) h = cadd(h, mul(he, io.xa[cc * B + b]));
        if (grad) add_class(e, ok, io.a_m1[cc * B + b]);
      }
    } else if (io.xa) {   // (one block, so that the row's own loads are in flight with the gathers)
      h = cscale(A.diag[r], io.xa[idx]);
      for_entries<K>(w, [&](int j) {
        const int64_t e = e0 + (int64_t)j * S;
        int64_t cc;
        const bool ok = col_entry<HOP>(A, r, e, &cc);
        const double2 x = io.xa[cc * B + b];
        h = cadd(h, mul(hop_entry<HOP>(A, e, ok, hu), x));
        if constexpr (NC > 0) add_class(e, ok, x);
      });
    }
    // direct sensitivities of the raw dots
    double2 g = cscale(w0, io.a_k[idx]);
    if (io.k >= 1) g = cadd(g, cscale(wm, io.a_m1[idx]));
    if (io.a_p1) g = cadd(g, cscale(wp, io.a_p1[idx]));
    double2 c = make_double2(fma(io.f_rec, h.x, g.x), fma(io.f_rec, h.y, g.y));
    if (io.wa) {
      const double2 u = io.wa[idx];
      c = make_double2(c.x - u.x, c.y - u.y);
    }
    const double2 o = cscale(out_scale, c);
    io.oa[idx] = io.acc_a ? cadd(io.oa[idx], o) : o;
    if (grad) {
      const double2 v = TR ? io.a_k[idx] : io.a_m1[idx];
      const double2 p = TR ? io.xa[idx] : c, l = TR ? v : c;
      double gu = io.f * (p.x * v.x + p.y * v.y);
#pragma unroll
      for (int off = 1; off < B; off <<= 1) gu += __shfl_xor(gu, off);
      if (b == 0) io.gU[r] = (AHEAD ? gu0 : io.gU[r]) + gu * inv_dE;
#pragma unroll
      for (int q = 0; q < (NC > 0 ? NC : 1); ++q)
        if (NC > 0) gc[q] += io.f * (l.x * hv[q].x + l.y * hv[q].y);
    }
  });
  if (NC == 0 || !grad) return;
  __shared__ double sh[kBlock / 64][NC > 0 ? NC : 1];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int q = 0; q < (NC > 0 ? NC : 1); ++q) {
    double s = gc[q];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off);
    if (lane == 0) sh[wave][q] = s;
  }
  __syncthreads();
  if (threadIdx.x < (NC > 0 ? NC : 1)) {
    double s = 0.0;
#pragma unroll
    for (int wv = 0; wv < kBlock / 64; ++wv) s += sh[wv][threadIdx.x];
    io.gcp[(int64_t)lb * NC + threadIdx.x] += s;
  }
}

}  // namespace

hipError_t launch_adjoint_sym_step(const DevMat& A, int hop_mode, int B, int nc, const AdjPairIO& io, hipStream_t s) {
  return dispatch_reverse(A, hop_mode, B, nc, io.tr, [&](auto Bc, auto Hc, auto Kc, auto Nc, auto Tc) {
    k_adjoint_sym_step<decltype(Bc)::value, decltype(Hc)::value, decltype(Kc)::value, decltype(Nc)::value, decltype(Tc)::value == 1>
        <<<dim3(A.G), kBlock, 0, s>>>(A, io);
  });
}

}  // namespace gpuqt
