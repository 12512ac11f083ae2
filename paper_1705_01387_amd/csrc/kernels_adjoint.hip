// Reverse (adjoint) of the Chebyshev moment recurrence, for gradients of
// losses built on the moments of Section 3.3 with respect to the on-site
// energies and the hopping classes.
//
// Forward (Section 3.2): v_0 = phiR, v_1 = H~ v_0, v_n = 2 H~ v_{n-1} - v_{n-2},
// mu_n = <phiL|v_n>.  For L = sum_n w_n Re mu_n the adjoint vectors obey
//   lam_n = w_n phiL + 2 H~ lam_{n+1} - lam_{n+2},  lam_M = lam_{M+1} = 0,
// a Clenshaw-type recurrence run backwards, and
//   dL/dp = Re[ sum_{n>=2} 2 <lam_n| dH~/dp v_{n-1}> + <lam_1| dH~/dp v_0> ].
// With dH~/dU_i = e_i e_i^T / DeltaE and dH~/deps_c = H~_c (the class-c
// hoppings), one reverse step needs lam_{n+1} and v_{n-1} at the neighbours
// of each row: the kernel gathers both with the same neighbour indices, so a
// reverse step reads the matrix once.
#include <hip/hip_runtime.h>

#include "device_common.h"
#include "reverse_core.h"

namespace gpuqt {

using namespace dev;

namespace {

// Class gradients (TR, where every class's hoppings are Hermitian by themselves): <lam_{n+1}| H~_c v_n> =
// conj(<v_n| H~_c lam_{n+1}>), and H~_c lam_{n+1} is part of the product that gives lam_n.  So step n adds
// the terms of step n + 1 from the rows' own v_n, and only lam_{n+1} is gathered.  Bound by the gathers
// and the vectors' traffic (512 x 512 with next-nearest neighbours, two classes, us a step: two chains 20.5 with v gathered
// too and one entry's loads after another's, 16.3 so; one chain of the Hermitian form 16.5, 12.8; one
// chain 14.2, 10.8).  Otherwise the terms of step n, with v_{n-1}
// gathered.
template <int B, int HOP, int K, int NC, bool TR>
__global__ __launch_bounds__(kBlock) void k_adjoint_step(DevMat A, AdjIO io) {
  const int lb = logical_block(A.G);
  const BlkPlan P = A.plan[lb];
  const double hu = (HOP == HOP_UNIFORM) ? A.seg_hop[P.seg] : 0.0;
  const double inv_dE = 1.0 / A.seg_dE[P.seg];
  const int b = threadIdx.x & (B - 1);
  // source coefficient of phiL: a real loss weight, or a complex series
  // coefficient J[seg][n] * src_phase (already conjugated by the caller)
  const double2 wn = io.Jtab ? cscale(io.Jtab[(int64_t)P.seg * io.ldJ + io.n], io.src_phase)
                             : make_double2(io.wts ? io.wts[((int64_t)P.seg * B + b) * io.M + io.n] : 0.0,
                                            0.0);
  const double2* __restrict__ x = io.x;
  const double2* __restrict__ v = io.v;
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
    if (AHEAD && v && b == 0) gu0 = io.gU[r];
    // per-entry gradients: the neighbours' v ahead of lam_n
    constexpr bool ENT = NC == 0 && K > 0;
    double2 vn[ENT ? K : 1];
    if constexpr (ENT) {
      if (io.gH) {
#pragma unroll
        for (int j = 0; j < K; ++j) {
          int64_t cc;
          (void)col_entry<HOP>(A, r, e0 + (int64_t)j * S, &cc);
          vn[j] = v[cc * B + b];
        }
      }
    }
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
    if constexpr (NC > 0 && !TR) {   // x and v with one reading of the keys
      if (x) h = cscale(A.diag[r], x[idx]);
      for (int j = 0; j < w; ++j) {
        const int64_t e = e0 + (int64_t)j * S;
        int64_t cc;
        const bool ok = col_entry<HOP>(A, r, e, &cc);
        const double2 he = hop_entry<HOP>(A, e, ok, hu);
        if (x) h = cadd(h, mul(he, x[cc * B + b]));
        if (v) add_class(e, ok, v[cc * B + b]);
      }
    } else if (x) {   // (one block, so that the row's own loads are in flight with the gathers)
      h = cscale(A.diag[r], x[idx]);
      for_entries<K>(w, [&](int j) {
        const int64_t e = e0 + (int64_t)j * S;
        int64_t cc;
        const bool ok = col_entry<HOP>(A, r, e, &cc);
        const double2 xv = x[cc * B + b];
        h = cadd(h, mul(hop_entry<HOP>(A, e, ok, hu), xv));
        if constexpr (NC > 0) add_class(e, ok, xv);
      });
    }
    double2 lam = cmul(wn, io.phiL[idx]);
    lam = make_double2(fma(io.f_rec, h.x, lam.x), fma(io.f_rec, h.y, lam.y));
    if (io.w) {
      const double2 ww = io.w[idx];
      lam = make_double2(lam.x - ww.x, lam.y - ww.y);
    }
    io.out[idx] = io.accumulate ? cadd(io.out[idx], lam) : lam;
    if (v) {
      const double2 vr = v[idx];
      const double2 lg = TR ? x[idx] : lam;
      double gu = io.f * (lg.x * vr.x + lg.y * vr.y);     // f Re(conj(lam) v)
#pragma unroll
      for (int off = 1; off < B; off <<= 1) gu += __shfl_xor(gu, off);
      if (b == 0) io.gU[r] = (AHEAD ? gu0 : io.gU[r]) + gu * inv_dE;
#pragma unroll
      for (int q = 0; q < (NC > 0 ? NC : 1); ++q)
        if (NC > 0) {
          const double2 l = TR ? vr : lam;
          gc[q] += io.f * (l.x * hv[q].x + l.y * hv[q].y);
        }
      if constexpr (ENT) {
        if (io.gH) {
          double2 g[K];
#pragma unroll
          for (int j = 0; j < K; ++j) {
            g[j].x = row_lanes_sum<B>(lam.x * vn[j].x + lam.y * vn[j].y);   // conj(lam) v
            g[j].y = row_lanes_sum<B>(lam.x * vn[j].y - lam.y * vn[j].x);
          }
          double* p = io.gH + 2 * r * (int64_t)io.ldH;
          const double f = io.f * inv_dE;
          if (b == 0)
#pragma unroll
            for (int j = 0; j < K; ++j) {   // (K > 0: every row has K neighbours)
              p[2 * j] += f * g[j].x;
              p[2 * j + 1] -= f * g[j].y;
            }
        }
      } else if (!TR && io.gH) {
        row_entry_grads<B, HOP, K>(A, r, b, lam, v, io.f * inv_dE, io.gH, io.ldH);
      }
    }
  });
  if (NC == 0 || !v) return;
  // class partials: workgroup sum in a fixed order, accumulated per workgroup
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

// Whether the hoppings of every class are Hermitian by themselves: for each entry (r, c), the sums of
// the class's hoppings from r to c and back are conjugate to each other.
template <int HOP>
__global__ __launch_bounds__(kBlock) void k_check_classes(DevMat A, const int32_t* __restrict__ cls, int32_t* bad) {
  const BlkPlan P = A.plan[logical_block(A.G)];
  const int S = 1 << A.S_log2;
  auto klass = [&](int64_t e) { return cls ? cls[HOP == HOP_DICT ? (int64_t)A.hidx[e] : e] : 0; };
  // hoppings of class q from row r to row c
  auto sum = [&](int64_t r, int64_t c, int q) {
    const int64_t sl = r >> A.S_log2, p0 = A.slice_ptr[sl], e0 = p0 + (r & (S - 1));
    const int w = (int)((A.slice_ptr[sl + 1] - p0) >> A.S_log2);
    double2 t = make_double2(0.0, 0.0);
    for (int j = 0; j < w; ++j) {
      const int64_t e = e0 + (int64_t)j * S;
      int64_t cc;
      if (col_entry<HOP>(A, r, e, &cc) && cc == c && klass(e) == q) t = cadd(t, hop0_entry<HOP>(A, e, true, P.seg));
    }
    return t;
  };
  for_rows<1>(A, P, [&](int64_t r) {
    const int64_t sl = r >> A.S_log2, p0 = A.slice_ptr[sl], e0 = p0 + (r & (S - 1));
    const int w = (int)((A.slice_ptr[sl + 1] - p0) >> A.S_log2);
    for (int j = 0; j < w; ++j) {
      const int64_t e = e0 + (int64_t)j * S;
      int64_t c;
      if (!col_entry<HOP>(A, r, e, &c)) continue;
      const int q = klass(e);
      const double2 a = sum(r, c, q), t = sum(c, r, q);
      if (a.x != t.x || a.y != -t.y) *bad = 1;
    }
  });
}

// Raw-dot weights of the product identities, one wavefront per (segment,
// column) row: lane l sums w_n for n = 2 + l + 64 j (all of one parity, the
// parity of l), a butterfly over lanes of equal parity gives the even and odd
// tails in a fixed order, and the lanes write om[n] for n = l, l + 64, ...
__global__ __launch_bounds__(64) void k_raw_weights(const double* __restrict__ w, int M, int R,
                                                    double* __restrict__ om) {
  const int64_t i = blockIdx.x;
  const int lane = threadIdx.x;
  const double* wi = w + i * M;
  double* oi = om + i * R;
  double t = 0.0;
  for (int n = 2 + lane; n < M; n += 64) t += wi[n];
#pragma unroll
  for (int off = 2; off < 64; off <<= 1) t += __shfl_xor(t, off);
  const double even = __shfl(t, 0), odd = __shfl(t, 1);
  for (int n = lane; n < R; n += 64) {
    double v = 0.0;
    if (n == 0) v = (M > 0 ? wi[0] : 0.0) - even;
    else if (n == 1) v = (M > 1 ? wi[1] : 0.0) - odd;
    else if (n < M) v = 2.0 * wi[n];
    oi[n] = v;
  }
}

// gcp[lb][c] += Re sum_i conj(a_i) (V_c x)_i over the workgroup's rows, with
// V_c = i dx H_c the velocity restricted to the class-c hoppings (unscaled:
// the stored H~ is multiplied back by DeltaE).
template <int B, int HOP, int NC>
__global__ __launch_bounds__(kBlock) void k_velocity_class_grad(DevMat A, const double2* __restrict__ a,
                                                                const double2* __restrict__ x,
                                                                const int32_t* __restrict__ cls,
                                                                double* __restrict__ gcp) {
  const int lb = logical_block(A.G);
  const BlkPlan P = A.plan[lb];
  const double e = A.seg_dE[P.seg];
  const int b = threadIdx.x & (B - 1);
  const int S = 1 << A.S_log2;
  double gc[NC];
#pragma unroll
  for (int q = 0; q < NC; ++q) gc[q] = 0.0;
  for_rows<B>(A, P, [&](int64_t r) {
    const int64_t idx = r * B + b;
    const int64_t sl = r >> A.S_log2;
    const int64_t p0 = A.slice_ptr[sl];
    const int64_t e0 = p0 + (r & (S - 1));
    const int w = (int)((A.slice_ptr[sl + 1] - p0) >> A.S_log2);
    const double2 ar = a[idx];
    for (int j = 0; j < w; ++j) {
      const int64_t en = e0 + (int64_t)j * S;
      int64_t c;
      if (!col_entry<HOP>(A, r, en, &c)) continue;
      const double2 he = hop0_entry<HOP>(A, en, true, P.seg);
      const double2 t = cmul(he, x[c * B + b]);
      const double s = e * dx_entry<HOP>(A, en);
      const double2 vt = make_double2(-s * t.y, s * t.x);      // i e dx H~ x
      const double contrib = ar.x * vt.x + ar.y * vt.y;        // Re conj(a) vt
      const int q0 = (NC > 1) ? cls[HOP == HOP_DICT ? (int64_t)A.hidx[en] : en] : 0;
#pragma unroll
      for (int q = 0; q < NC; ++q)
        if (q == q0) gc[q] += contrib;
    }
  });
  __shared__ double sh[kBlock / 64][NC];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    double s = gc[q];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off);
    if (lane == 0) sh[wave][q] = s;
  }
  __syncthreads();
  if (threadIdx.x < NC) {
    double s = 0.0;
#pragma unroll
    for (int wv = 0; wv < kBlock / 64; ++wv) s += sh[wv][threadIdx.x];
    gcp[(int64_t)lb * NC + threadIdx.x] += s;
  }
}

// Per-entry share of a^+ V x, V_ij = i dx_ij H_ij (unscaled):
// g_ij = i dx_ij sum_b conj(a_ib) x_jb, gH[i*ldH + slot] += (Re g, -Im g).
template <int B, int HOP>
__global__ __launch_bounds__(kBlock) void k_velocity_entry_grad(DevMat A, const double2* __restrict__ a,
                                                                const double2* __restrict__ x,
                                                                double* __restrict__ gH, int ldH) {
  const BlkPlan P = A.plan[logical_block(A.G)];
  const int b = threadIdx.x & (B - 1);
  const int S = 1 << A.S_log2;
  for_rows<B>(A, P, [&](int64_t r) {
    const double2 ar = a[r * B + b];
    const int64_t sl = r >> A.S_log2;
    const int64_t p0 = A.slice_ptr[sl];
    const int64_t e0 = p0 + (r & (S - 1));
    const int w = (int)((A.slice_ptr[sl + 1] - p0) >> A.S_log2);
    for (int j = 0; j < w; ++j) {
      const int64_t en = e0 + (int64_t)j * S;
      int64_t c;
      const bool ok = col_entry<HOP>(A, r, en, &c);
      const double2 xv = x[c * B + b];
      double zr = ar.x * xv.x + ar.y * xv.y;   // z = conj(a) x
      double zi = ar.x * xv.y - ar.y * xv.x;
      zr = row_lanes_sum<B>(zr);
      zi = row_lanes_sum<B>(zi);
      if (ok && b == 0) {
        const double d = dx_entry<HOP>(A, en);   // g = i d z: (Re g, -Im g) = (-d Im z, -d Re z)
        double* p = gH + 2 * (r * (int64_t)ldH + j);
        p[0] -= d * zi;
        p[1] -= d * zr;
      }
    }
  });
}

// Hermitian tie of per-entry gradients, one thread per (row i, slot s): entry
// (i, s) -> j is the q-th of row i's entries pointing to j; its partner is the
// q-th entry of row j pointing to i.  out = (re_is + re_jp, im_is - im_jp), or
// the entry's own value without a partner (and for padding slots).
template <int HOP>
__global__ __launch_bounds__(256) void k_tie_entries(DevMat A, int64_t n, int ldH, const double* __restrict__ in,
                                                     double* __restrict__ out) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n * ldH) return;
  const int64_t i = t / ldH;
  const int s = (int)(t - i * ldH);
  const int S = 1 << A.S_log2;
  auto width = [&](int64_t r) { const int64_t sl = r >> A.S_log2; return (int)((A.slice_ptr[sl + 1] - A.slice_ptr[sl]) >> A.S_log2); };
  auto entry = [&](int64_t r, int j) { return A.slice_ptr[r >> A.S_log2] + (int64_t)j * S + (r & (S - 1)); };
  double re = in[2 * t], im = in[2 * t + 1];
  int64_t j = -1;
  if (s < width(i)) {
    int64_t c;
    if (col_entry<HOP>(A, i, entry(i, s), &c)) j = c;
  }
  if (j >= 0) {
    int q = 0;
    for (int u = 0; u < s; ++u) {
      int64_t c;
      if (col_entry<HOP>(A, i, entry(i, u), &c) && c == j) ++q;
    }
    const int wj = width(j);
    for (int u = 0; u < wj && u < ldH; ++u) {
      int64_t c;
      if (col_entry<HOP>(A, j, entry(j, u), &c) && c == i) {
        if (q == 0) {
          re += in[2 * (j * ldH + u)];
          im -= in[2 * (j * ldH + u) + 1];
          break;
        }
        --q;
      }
    }
  }
  out[2 * t] = re;
  out[2 * t + 1] = im;
}

// diag[r] = onsite[r] / DeltaE_seg (new on-site energies)
__global__ __launch_bounds__(kBlock) void k_set_onsite(DevMat A, const double* __restrict__ onsite,
                                                       double* __restrict__ diag) {
  const BlkPlan P = A.plan[logical_block(A.G)];
  const double inv = 1.0 / A.seg_dE[P.seg];
  for_rows<1>(A, P, [&](int64_t r) { diag[r] = onsite[r] * inv; });
}

// hop[e] = hop0[e] * scale[class of e]  (real: one double per entry, complex: two)
__global__ __launch_bounds__(256) void k_scale_hops(int64_t entries, int cplx, const double* __restrict__ hop0,
                                                    double* __restrict__ hop, const int32_t* __restrict__ cls,
                                                    ClassScale sc) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < entries;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int c = cls ? cls[e] : 0;
    const double f = c >= 0 ? sc.s[c] : 0.0;
    if (cplx) {
      hop[2 * e] = hop0[2 * e] * f;
      hop[2 * e + 1] = hop0[2 * e + 1] * f;
    } else {
      hop[e] = hop0[e] * f;
    }
  }
}

// bound[lb] = max over the workgroup's rows of |U~_r| + sum_j |H~_rj| (the
// Gershgorin bound of H / DeltaE, which must stay <= 1)
template <int HOP>
__global__ __launch_bounds__(kBlock) void k_row_bound(DevMat A, double* __restrict__ bound) {
  const int lb = logical_block(A.G);
  const BlkPlan P = A.plan[lb];
  const double hu = (HOP == HOP_UNIFORM) ? fabs(A.seg_hop[P.seg]) : 0.0;
  const int S = 1 << A.S_log2;
  double mx = 0.0;
  for_rows<1>(A, P, [&](int64_t r) {
    const int64_t sl = r >> A.S_log2;
    const int64_t p0 = A.slice_ptr[sl];
    const int64_t e0 = p0 + (r & (S - 1));
    const int w = (int)((A.slice_ptr[sl + 1] - p0) >> A.S_log2);
    double s = fabs(A.diag[r]);
    for (int j = 0; j < w; ++j) {
      const int64_t e = e0 + (int64_t)j * S;
      int64_t c;
      if (!col_entry<HOP>(A, r, e, &c)) continue;
      const double2 he = hop_entry<HOP>(A, e, true, hu);
      s += HOP == HOP_UNIFORM ? hu : (HOP == HOP_REAL ? fabs(he.x) : hypot(he.x, he.y));
    }
    mx = fmax(mx, s);
  });
  __shared__ double sh[kBlock / 64];
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) mx = fmax(mx, __shfl_xor(mx, off));
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = mx;
  __syncthreads();
  if (threadIdx.x == 0) {
    double m = 0.0;
    for (int q = 0; q < kBlock / 64; ++q) m = fmax(m, sh[q]);
    bound[lb] = m;
  }
}

__global__ __launch_bounds__(256) void k_zero(double* __restrict__ p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0.0;
}

// grad_class[c] += sum over workgroups of gcp[g][c], in a fixed order.
__global__ __launch_bounds__(64) void k_reduce_classes(const double* __restrict__ gcp, int G, int NC,
                                                       double* __restrict__ out) {
  const int c = blockIdx.x;
  double s = 0.0;
  for (int g = threadIdx.x; g < G; g += 64) s += gcp[(int64_t)g * NC + c];
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off);
  if (threadIdx.x == 0) out[c] += s;
}

}  // namespace

hipError_t launch_adjoint_step(const DevMat& A, int hop_mode, int B, int nc, const AdjIO& io, hipStream_t s) {
  return dispatch_reverse(A, hop_mode, B, nc, io.tr, [&](auto Bc, auto Hc, auto Kc, auto Nc, auto Tc) {
    k_adjoint_step<decltype(Bc)::value, decltype(Hc)::value, decltype(Kc)::value, decltype(Nc)::value, decltype(Tc)::value == 1>
        <<<dim3(A.G), kBlock, 0, s>>>(A, io);
  });
}

hipError_t launch_check_classes(const DevMat& A, int hop_mode, const int32_t* cls, int32_t* bad, hipStream_t s) {
  switch (hop_mode) {
    case HOP_UNIFORM: k_check_classes<HOP_UNIFORM><<<dim3(A.G), kBlock, 0, s>>>(A, cls, bad); break;
    case HOP_REAL: k_check_classes<HOP_REAL><<<dim3(A.G), kBlock, 0, s>>>(A, cls, bad); break;
    case HOP_COMPLEX: k_check_classes<HOP_COMPLEX><<<dim3(A.G), kBlock, 0, s>>>(A, cls, bad); break;
    default: k_check_classes<HOP_DICT><<<dim3(A.G), kBlock, 0, s>>>(A, cls, bad); break;
  }
  return hipGetLastError();
}

hipError_t launch_raw_weights(const double* w, int rows, int M, int R, double* om, hipStream_t s) {
  if (rows <= 0 || R <= 0) return hipSuccess;
  k_raw_weights<<<dim3(rows), 64, 0, s>>>(w, M, R, om);
  return hipGetLastError();
}

hipError_t launch_velocity_class_grad(const DevMat& A, int hop_mode, int B, int nc, const double2* a,
                                      const double2* x, const int32_t* cls, double* gcp, hipStream_t s) {
  return dispatch_bh(B, hop_mode, [&](auto Bc, auto Hc) {
    constexpr int Bv = decltype(Bc)::value, Hv = decltype(Hc)::value;
    switch (nc) {
      case 1: k_velocity_class_grad<Bv, Hv, 1><<<dim3(A.G), kBlock, 0, s>>>(A, a, x, cls, gcp); break;
      case 2: k_velocity_class_grad<Bv, Hv, 2><<<dim3(A.G), kBlock, 0, s>>>(A, a, x, cls, gcp); break;
      default: k_velocity_class_grad<Bv, Hv, 4><<<dim3(A.G), kBlock, 0, s>>>(A, a, x, cls, gcp); break;
    }
  });
}

hipError_t launch_velocity_entry_grad(const DevMat& A, int hop_mode, int B, const double2* a, const double2* x,
                                      double* gH, int ldH, hipStream_t s) {
  return dispatch_bh(B, hop_mode, [&](auto Bc, auto Hc) {
    k_velocity_entry_grad<decltype(Bc)::value, decltype(Hc)::value><<<dim3(A.G), kBlock, 0, s>>>(A, a, x, gH,
                                                                                                  ldH);
  });
}

hipError_t launch_tie_entries(const DevMat& A, int hop_mode, int64_t n, int ldH, const double* in, double* out,
                              hipStream_t s) {
  const int64_t total = n * (int64_t)ldH;
  if (total <= 0) return hipSuccess;
  const int64_t blocks = (total + 255) / 256;
  if (blocks > 0x7fffffff) return hipErrorInvalidValue;
  const dim3 g((unsigned)blocks);
  if (hop_mode == HOP_UNIFORM) k_tie_entries<HOP_UNIFORM><<<g, 256, 0, s>>>(A, n, ldH, in, out);
  else if (hop_mode == HOP_REAL) k_tie_entries<HOP_REAL><<<g, 256, 0, s>>>(A, n, ldH, in, out);
  else if (hop_mode == HOP_COMPLEX) k_tie_entries<HOP_COMPLEX><<<g, 256, 0, s>>>(A, n, ldH, in, out);
  else k_tie_entries<HOP_DICT><<<g, 256, 0, s>>>(A, n, ldH, in, out);
  return hipGetLastError();
}

hipError_t launch_set_onsite(const DevMat& A, const double* onsite, double* diag, hipStream_t s) {
  k_set_onsite<<<dim3(A.G), kBlock, 0, s>>>(A, onsite, diag);
  return hipGetLastError();
}

hipError_t launch_scale_hops(int64_t entries, int cplx, const double* hop0, double* hop,
                             const int32_t* cls, const ClassScale& sc, hipStream_t s) {
  if (entries <= 0) return hipSuccess;
  int64_t blocks = (entries + 255) / 256;
  if (blocks > 8192) blocks = 8192;
  k_scale_hops<<<dim3((unsigned)blocks), 256, 0, s>>>(entries, cplx, hop0, hop, cls, sc);
  return hipGetLastError();
}

hipError_t launch_row_bound(const DevMat& A, int hop_mode, double* bound, hipStream_t s) {
  if (hop_mode == HOP_UNIFORM) k_row_bound<HOP_UNIFORM><<<dim3(A.G), kBlock, 0, s>>>(A, bound);
  else if (hop_mode == HOP_REAL) k_row_bound<HOP_REAL><<<dim3(A.G), kBlock, 0, s>>>(A, bound);
  else if (hop_mode == HOP_COMPLEX) k_row_bound<HOP_COMPLEX><<<dim3(A.G), kBlock, 0, s>>>(A, bound);
  else k_row_bound<HOP_DICT><<<dim3(A.G), kBlock, 0, s>>>(A, bound);
  return hipGetLastError();
}

hipError_t launch_zero(double* p, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  k_zero<<<dim3((unsigned)blocks), 256, 0, s>>>(p, n);
  return hipGetLastError();
}

hipError_t launch_reduce_classes(const double* gcp, int G, int nc, int n_out, double* out, hipStream_t s) {
  if (nc <= 0 || n_out <= 0) return hipSuccess;
  k_reduce_classes<<<dim3(n_out), 64, 0, s>>>(gcp, G, nc, out);
  return hipGetLastError();
}

}  // namespace gpuqt
