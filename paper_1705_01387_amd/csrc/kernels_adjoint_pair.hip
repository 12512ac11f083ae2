// Reverse steps of the two-chain moments (kernels_adjoint.hip has the recurrence and the single chain).
#include <hip/hip_runtime.h>

#include "device_common.h"
#include "reverse_core.h"

namespace gpuqt {

using namespace dev;

namespace {

// Where four waves a SIMD are asked for (TR): the unrolled forms take a few registers more than the 128 that those allow and run
// at three (six neighbours, a hopping an entry, 50^3, two vectors, 64 moments: 902 us instead of 1,177; eight neighbours, one
// class, 512 x 512, one vector: 836 instead of 1,105), but other forms of eight neighbours lose with the bound
// (two classes, one vector 881 instead of 754; one class, two vectors 1,618 instead of 1,518).
constexpr bool four_waves(int B, int K, int NC) { return K == 6 || (K == 8 && NC == 1 && B == 1); }

// Reverse step of the two-chain form (both adjoint chains in one launch, the
// matrix read once; abar_{k+1}, bbar_{k+1} and, for class gradients, a_{k-1},
// b_{k-1} gathered with the same indices).  Parameter terms, as for the
// single chain: dL/dp = Re sum_k f_k (<abar_k| dH~/dp a_{k-1}> + <bbar_k| dH~/dp b_{k-1}>).
template <int B, int HOP, int K, int NC, bool TR>
__device__ __forceinline__ void pair_step(const DevMat& A, const AdjPairIO& io) {
  const int lb = logical_block(A.G);
  const BlkPlan P = A.plan[lb];
  const double hu = (HOP == HOP_UNIFORM) ? A.seg_hop[P.seg] : 0.0;
  const double inv_dE = 1.0 / A.seg_dE[P.seg];
  const int b = threadIdx.x & (B - 1);
  const double* om = io.om + ((int64_t)P.seg * B + b) * io.R;
  const int k2 = 2 * io.k;
  const double w0 = om[k2];
  const double wm = io.k >= 1 ? om[k2 - 1] : 0.0;
  const double wp = (io.a_p1 && k2 + 1 < io.R) ? om[k2 + 1] : 0.0;
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
    double2 ha = make_double2(0.0, 0.0), hb = make_double2(0.0, 0.0);
    double2 hva[NC > 0 ? NC : 1], hvb[NC > 0 ? NC : 1];
#pragma unroll
    for (int c = 0; c < (NC > 0 ? NC : 1); ++c) {
      hva[c] = make_double2(0.0, 0.0);
      hvb[c] = make_double2(0.0, 0.0);
    }
    constexpr bool AHEAD = TR || NC == 0;   // gU read ahead of the products
    double gu0 = 0.0;
    if (AHEAD && grad && b == 0) gu0 = io.gU[r];
    auto mul = [](double2 he, double2 y) {
      return (HOP == HOP_COMPLEX || HOP == HOP_DICT) ? cmul(he, y) : cscale(he.x, y);
    };
    auto add_class = [&](int64_t e, bool ok, double2 ya, double2 yb) {
      const double2 he0 = hop0_entry<HOP>(A, e, ok, P.seg);
      const double2 ta = mul(he0, ya), tb = mul(he0, yb);
      const int cls = NC > 1 && (TR || ok) ? io.cls[HOP == HOP_DICT ? (int64_t)A.hidx[e] : e] : 0;   // (padding adds zero)
#pragma unroll
      for (int q = 0; q < (NC > 0 ? NC : 1); ++q) {
        if constexpr (TR) {
          hva[q].x += q == cls ? ta.x : 0.0;
          hva[q].y += q == cls ? ta.y : 0.0;
          hvb[q].x += q == cls ? tb.x : 0.0;
          hvb[q].y += q == cls ? tb.y : 0.0;
        } else if (q == cls) {
          hva[q] = cadd(hva[q], ta);
          hvb[q] = cadd(hvb[q], tb);
        }
      }
    };
    auto diagonal = [&]() {
      const double d = A.diag[r];
      ha = cscale(d, io.xa[idx]);
      hb = cscale(d, io.xb[idx]);
    };
    if constexpr (NC > 0 && !TR) {
      if (io.xa) diagonal();
      for (int j = 0; j < w; ++j) {
        const int64_t e = e0 + (int64_t)j * S;
        int64_t cc;
        const bool ok = col_entry<HOP>(A, r, e, &cc);
        const double2 he = hop_entry<HOP>(A, e, ok, hu);
        if (io.xa) {
          ha = cadd(ha, mul(he, io.xa[cc * B + b]));
          hb = cadd(hb, mul(he, io.xb[cc * B + b]));
        }
        if (grad) add_class(e, ok, io.a_m1[cc * B + b], io.b_m1[cc * B + b]);
      }
    } else if (io.xa) {   // (one block, so that the row's own loads are in flight with the gathers)
      diagonal();
      for_entries<K>(w, [&](int j) {
        const int64_t e = e0 + (int64_t)j * S;
        int64_t cc;
        const bool ok = col_entry<HOP>(A, r, e, &cc);
        const double2 he = hop_entry<HOP>(A, e, ok, hu);
        const double2 xa = io.xa[cc * B + b], xb = io.xb[cc * B + b];
        ha = cadd(ha, mul(he, xa));
        hb = cadd(hb, mul(he, xb));
        if constexpr (NC > 0) add_class(e, ok, xa, xb);
      });
    }
    // direct sensitivities of the raw dots
    double2 ga = cscale(w0, io.b_k[idx]);
    if (io.k >= 1) ga = cadd(ga, cscale(wm, io.b_m1[idx]));
    double2 gb = cscale(w0, io.a_k[idx]);
    if (io.a_p1) gb = cadd(gb, cscale(wp, io.a_p1[idx]));
    double2 la = make_double2(fma(io.f_rec, ha.x, ga.x), fma(io.f_rec, ha.y, ga.y));
    double2 lbv = make_double2(fma(io.f_rec, hb.x, gb.x), fma(io.f_rec, hb.y, gb.y));
    if (io.wa) {
      const double2 u = io.wa[idx], v = io.wb[idx];
      la = make_double2(la.x - u.x, la.y - u.y);
      lbv = make_double2(lbv.x - v.x, lbv.y - v.y);
    }
    io.oa[idx] = io.acc_a ? cadd(io.oa[idx], la) : la;
    io.ob[idx] = io.acc_b ? cadd(io.ob[idx], lbv) : lbv;
    if (grad) {
      const double2 va = TR ? io.a_k[idx] : io.a_m1[idx], vb = TR ? io.b_k[idx] : io.b_m1[idx];
      const double2 pa = TR ? io.xa[idx] : la, pb = TR ? io.xb[idx] : lbv;
      double gu = io.f * (pa.x * va.x + pa.y * va.y + pb.x * vb.x + pb.y * vb.y);
      const double2 qa = TR ? va : la, qb = TR ? vb : lbv;
#pragma unroll
      for (int off = 1; off < B; off <<= 1) gu += __shfl_xor(gu, off);
      if (b == 0) io.gU[r] = (AHEAD ? gu0 : io.gU[r]) + gu * inv_dE;
#pragma unroll
      for (int q = 0; q < (NC > 0 ? NC : 1); ++q)
        if (NC > 0)
          gc[q] += io.f * (qa.x * hva[q].x + qa.y * hva[q].y + qb.x * hvb[q].x + qb.y * hvb[q].y);
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

template <int B, int HOP, int K, int NC, bool TR>
__global__ __launch_bounds__(kBlock) void k_adjoint_pair_step(DevMat A, AdjPairIO io) {
  pair_step<B, HOP, K, NC, TR>(A, io);
}
template <int B, int HOP, int K, int NC>
__global__ __launch_bounds__(kBlock, 4) void k_adjoint_pair_step_4(DevMat A, AdjPairIO io) {
  pair_step<B, HOP, K, NC, true>(A, io);
}

}  // namespace

hipError_t launch_adjoint_pair_step(const DevMat& A, int hop_mode, int B, int nc, const AdjPairIO& io, hipStream_t s) {
  return dispatch_reverse(A, hop_mode, B, nc, io.tr, [&](auto Bc, auto Hc, auto Kc, auto Nc, auto Tc) {
    constexpr int Bv = decltype(Bc)::value, Hv = decltype(Hc)::value, Kv = decltype(Kc)::value, N = decltype(Nc)::value;
    constexpr bool TR = decltype(Tc)::value == 1;
    if constexpr (TR && four_waves(Bv, Kv, N)) k_adjoint_pair_step_4<Bv, Hv, Kv, N><<<dim3(A.G), kBlock, 0, s>>>(A, io);
    else k_adjoint_pair_step<Bv, Hv, Kv, N, TR><<<dim3(A.G), kBlock, 0, s>>>(A, io);
  });
}

}  // namespace gpuqt
