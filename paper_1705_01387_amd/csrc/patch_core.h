// The patch kernel: the steps of march.h's launches for lattices too small for a
// march to fill the chip, for chains and for squares with next-nearest neighbours.  A
// workgroup holds a patch of cells with a margin of T cells on every side, one cell a lane,
// takes T steps of the recurrence on it in place and writes the two last ones.  Nothing moves between the steps but the
// cells' values through LDS (double-buffered: one barrier a step).
//
// What bounds it: on a small lattice the launch itself (about 4 us with its loads, stores
// and the dots' sums) and its barriers: 8 steps of the Hermitian set on 64 x 64 take 6.5 us in
// workgroups of 640 cells, where the march's run of 17 or more iterations takes 14 to 16.
// On a chain the vectors' traffic, two elements read and two written for 24 steps, and the
// double arithmetic: 8 M cells take 8.5 us a step (Hermitian set, 4 cells a lane) and 18
// (evolution + commutator, 2 cells a lane; 21 with 16 steps) where single steps take 81 and
// 268.  With next-nearest neighbours the LDS reads, eight a cell and step: 512 x 512 takes
// 4.7 us a step (Hermitian set) and 6.7 (two chains) where single steps take 7.6 and 9.9.
#pragma once

#include "march_core.h"

namespace gpuqt {
namespace march {

// C cells a lane (cell = lane + j LANES of the patch; C = 1 in two dimensions); io.steps steps,
// at most the margin A.T and a multiple of kPatchUnroll: the loop is unrolled that far and no
// further, since a workgroup runs its code once and longer code waits for instructions (8 steps
// of the Hermitian set on 64 x 64: 9.5 us unrolled, 7.1 us rolled).
template <int PAT, int FAM, int HOP, int LANES, int C, bool FIRST, bool KEEP>
__global__ __launch_bounds__(LANES) void k_patch(MarchMat A, MarchIO io) {
  constexpr int NC = two_chains(FAM) ? 2 : 1;
  constexpr bool DOTS = has_dots(FAM);
  constexpr bool FLAT = PAT == MARCH_CHAIN;
  constexpr bool DIAG = PAT == MARCH_NNN;   // diagonal neighbours too
  constexpr int K = FLAT ? 2 : PAT == MARCH_BRICK ? 3 : DIAG ? 8 : 4;
  constexpr bool ENTRY = HOP != HOP_UNIFORM;
  constexpr bool CPLX = HOP == HOP_COMPLEX || HOP == HOP_DICT;
  constexpr bool IM = NC == 2 || ENTRY;   // as in k_march
  using hv_t = std::conditional_t<CPLX, double2, double>;
  constexpr int MARGIN = FLAT ? 1 : kMaxTileX + 1;
  constexpr int SLOTS = C * LANES + 2 * MARGIN;
  constexpr int U = kPatchUnroll, NW = LANES / 64;
  // dots of a group of U steps: per step the real part of rows 2k - 1 and 2k, then (IM) the imaginary part of
  // row 2k - 1 and (two chains) of row 2k
  constexpr int PS = 2 + (IM ? 1 : 0) + (NC == 2 ? 1 : 0);
  constexpr int NV = PS * U <= 8 ? 8 : 16;
  __shared__ double2 lds[2][NC][SLOTS];
  __shared__ double red[DOTS ? kMarchMaxSteps / U : 1][NW][DOTS ? NV : 1], red0[NW][2];
  const int T = A.T;

  const int total = A.items * A.B, xcd = blockIdx.x & 7;
  const int lb = xcd * (total >> 3) + min(xcd, total & 7) + ((int)blockIdx.x >> 3);
  auto uni = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
  const int major = uni(lb / (KEEP ? A.B : A.items)), minor = lb - major * (KEEP ? A.B : A.items);
  const int col = KEEP ? minor : major, item = KEEP ? major : minor;
  const int64_t sb = KEEP ? A.B : 1;
  int sg = 0;
  for (int hi = A.n_seg - 1; sg < hi;) {
    const int mid = (sg + hi + 1) >> 1;
    if (A.segs[mid].item0 <= item) sg = mid;
    else hi = mid - 1;
  }
  const MarchSeg S = A.segs[sg];
  const int l = threadIdx.x, cells = S.tx * S.ty, up = FLAT ? 0 : S.tx;
  auto wrap = [](int v, int L) { v %= L; return v < 0 ? v + L : v; };

  const double hus = ENTRY ? 0.0 : 2.0 * A.seg_hop[sg];
  const int wave = l >> 6, lane = l & 63;
  for (int e = l; e < 2 * NC * SLOTS; e += LANES) (&lds[0][0][0])[e] = make_double2(0.0, 0.0);
  __syncthreads();

  // the work item's tiles: their dots add up in red.  (A tile's first write to LDS, to buffer 0, comes after
  // the barrier of the last step before it, which reads buffer 1.)
  const int q0 = (item - S.item0) * S.zc, q1 = min(q0 + S.zc, S.nx * S.ny);
#pragma unroll 1
  for (int q = q0; q < q1; ++q) {
  const int iy = uni(q / S.nx), ix = q - iy * S.nx;
  bool own[C], vert[C];
  int64_t at[C];
  double d2[C], hu[C], dxp[C], dxm[C];
  hv_t hop[C][ENTRY ? K : 1];
  double2 x[C][NC], w[C][NC], acc[C][DOTS ? 1 : NC];
#pragma unroll
  for (int j = 0; j < C; ++j) {
    const int p = l + j * LANES, tl = min(p, cells - 1);   // lanes past the patch repeat its last cell
    const int ty = FLAT ? 0 : tl / S.tx, tx = tl - ty * S.tx;
    const int X = ix * S.ux + tx - T, Y = FLAT ? 0 : iy * S.uy + ty - T;
    const int xw = wrap(X, S.Lx), yw = FLAT ? 0 : wrap(Y, S.Lm);
    own[j] = p < cells && tx >= T && tx < T + S.ux && X < S.Lx;
    if (!FLAT) own[j] = own[j] && ty >= T && ty < T + S.uy && Y < S.Lm;
    vert[j] = PAT == MARCH_BRICK && ((xw + yw + A.parity) & 1) == 0;
    const int64_t row = S.off + (int64_t)yw * S.Lx + xw;
    at[j] = KEEP ? row * sb + col : (int64_t)col * A.n + row;
    d2[j] = 2.0 * A.diag[row];
    // past the edge of a lattice that is open in x: elements start as zero, and no hopping keeps them so
    const bool out = PAT == MARCH_SQUARE && !ENTRY && A.open && (X < 0 || X >= S.Lx);
    hu[j] = out ? 0.0 : hus;
    if constexpr (ENTRY) {
      const int64_t e = (row >> A.S_log2) * ((int64_t)K << A.S_log2) + (row & ((1 << A.S_log2) - 1));
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const int64_t ek = e + ((int64_t)A.slot[k] << A.S_log2);
        if constexpr (HOP == HOP_REAL) hop[j][k] = 2.0 * A.hop[ek];
        else if constexpr (HOP == HOP_COMPLEX) hop[j][k] = cscale(2.0, reinterpret_cast<const double2*>(A.hop)[ek]);
        else hop[j][k] = cscale(2.0, A.htab[A.hidx[ek]]);
      }
    }
    dxp[j] = dxm[j] = 0.0;
    if constexpr (FAM == MF_MSD) {
      dxp[j] = FLAT ? A.dx : A.dxcol[S.dx0 + xw];
      dxm[j] = FLAT ? -A.dx : -A.dxcol[S.dx0 + (xw == 0 ? S.Lx - 1 : xw - 1)];
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const bool z = out || (FIRST && c == 1 && io.zero_b);
      x[j][c] = z ? make_double2(0.0, 0.0) : io.x[c][at[j]];
      w[j][c] = FIRST || out ? make_double2(0.0, 0.0) : io.w[c][at[j]];
      if constexpr (!DOTS)
        acc[j][c] = FIRST ? cscale(io.J[(int64_t)sg * io.ldJ], x[j][c]) : io.acc_in[c][at[j]];
    }
  }

  double v0[2] = {0.0, 0.0};   // dots of row 0
  auto axpy = [](double2& t, auto a, double2 b) {
    if constexpr (std::is_same_v<decltype(a), double2>) {
      t.x = fma(a.x, b.x, fma(-a.y, b.y, t.x));
      t.y = fma(a.x, b.y, fma(a.y, b.x, t.y));
    } else {
      t.x = fma(a, b.x, t.x);
      t.y = fma(a, b.y, t.y);
    }
  };
#pragma unroll 1
  for (int s0 = 0; s0 < io.steps; s0 += U) {
  double v[DOTS ? NV : 1];
#pragma unroll
  for (int d = 0; d < (DOTS ? NV : 1); ++d) v[d] = 0.0;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int s = s0 + u;
#pragma unroll
    for (int j = 0; j < C; ++j)
#pragma unroll
      for (int c = 0; c < NC; ++c) lds[u & 1][c][MARGIN + l + j * LANES] = x[j][c];
    __syncthreads();
    // c_m of step m = k0 + s: J_m (-i sgn)^m, none past the last term
    double2 cm = make_double2(0.0, 0.0);
    if constexpr (!DOTS) {
      const int m = io.k0 + s;
      const double jm = m <= io.k_end ? io.J[(int64_t)sg * io.ldJ + m] : 0.0;
      cm = (m & 3) == 0   ? make_double2(jm, 0.0)
           : (m & 3) == 1 ? make_double2(0.0, -io.sgn * jm)
           : (m & 3) == 2 ? make_double2(-jm, 0.0)
                          : make_double2(0.0, io.sgn * jm);
    }
#pragma unroll
    for (int j = 0; j < C; ++j) {
      double2 y[NC], sx = make_double2(0.0, 0.0);
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const double2* L = &lds[u & 1][c][MARGIN + l + j * LANES];
        const double2 xp = L[1], xm = L[-1];
        // t = 2 H~ x - w
        double2 t = make_double2(fma(d2[j], x[j][c].x, -w[j][c].x), fma(d2[j], x[j][c].y, -w[j][c].y));
        if constexpr (ENTRY) {
          if constexpr (FAM == MF_MSD) {
            double2 p = make_double2(0.0, 0.0), m = p;
            axpy(p, hop[j][0], xp);
            axpy(m, hop[j][1], xm);
            if constexpr (DIAG) {
              axpy(p, hop[j][K - 4], L[up + 1]);
              axpy(m, hop[j][K - 3], L[up - 1]);
              axpy(p, hop[j][K - 2], L[1 - up]);
              axpy(m, hop[j][K - 1], L[-1 - up]);
            }
            if (c == 0) sx = make_double2(fma(dxp[j], p.x, dxm[j] * m.x), fma(dxp[j], p.y, dxm[j] * m.y));
            t = cadd(t, cadd(p, m));
          } else {
            axpy(t, hop[j][0], xp);
            axpy(t, hop[j][1], xm);
            if constexpr (DIAG) {
              axpy(t, hop[j][K - 4], L[up + 1]);
              axpy(t, hop[j][K - 3], L[up - 1]);
              axpy(t, hop[j][K - 2], L[1 - up]);
              axpy(t, hop[j][K - 1], L[-1 - up]);
            }
          }
          if constexpr (PAT == MARCH_BRICK) {
            axpy(t, hop[j][K - 1], L[vert[j] ? up : -up]);
          } else if constexpr (!FLAT) {
            axpy(t, hop[j][DIAG ? 3 : K - 1], L[-up]);
            axpy(t, hop[j][DIAG ? 2 : K - 2], L[up]);
          }
        } else {
          const double hu2 = PAT == MARCH_SQUARE ? hu[j] : hus;
          double2 n = cadd(xp, xm), np = xp, nm = xm;   // (np, nm: neighbours at x + 1 and x - 1)
          if constexpr (DIAG) {
            np = cadd(np, cadd(L[up + 1], L[1 - up]));
            nm = cadd(nm, cadd(L[up - 1], L[-1 - up]));
            n = cadd(np, nm);
          }
          if constexpr (FAM == MF_MSD) {
            if (c == 0)
              sx = make_double2(hu2 * fma(dxp[j], np.x, dxm[j] * nm.x), hu2 * fma(dxp[j], np.y, dxm[j] * nm.y));
          }
          if constexpr (PAT == MARCH_BRICK) {
            n = cadd(n, L[vert[j] ? up : -up]);
          } else if constexpr (!FLAT) {
            n = cadd(n, L[-up]);
            n = cadd(n, L[up]);
          }
          t = make_double2(fma(hu2, n.x, t.x), fma(hu2, n.y, t.y));
        }
        if constexpr (FAM == MF_MSD) {   // + 2 [X, H~] a
          if (c == 1) t = make_double2(t.x - sx.x, t.y - sx.y);
        }
        y[c] = (FIRST && u == 0 && s0 == 0) ? cscale(0.5, t) : t;   // v_1 = H~ v_0
      }
      if constexpr (DOTS) {   // (a lane's cells that the patch does not own add nothing)
        const double2 ya = own[j] ? y[0] : make_double2(0.0, 0.0), yb = own[j] ? y[NC - 1] : make_double2(0.0, 0.0);
        const double2 xa = own[j] ? x[j][0] : make_double2(0.0, 0.0);
        const double2 xb = own[j] ? x[j][NC - 1] : make_double2(0.0, 0.0);
        double im = 0.0;
        if (FIRST && u == 0 && s0 == 0) {
          cdot_acc(v0[0], v0[1], xa, xb);      // <a0|b0>
          cdot_acc(v[0], im, xa, yb);          // <a0|b1>
        } else {
          cdot_acc(v[PS * u], im, ya, xb);
        }
        if constexpr (IM) v[PS * u + 2] += im;
        im = 0.0;
        cdot_acc(v[PS * u + 1], im, ya, yb);
        if constexpr (NC == 2) v[PS * u + 3] += im;
      } else {
#pragma unroll
        for (int c = 0; c < NC; ++c)
          if (io.k0 + s <= io.k_end) axpy(acc[j][c], cm, y[c]);
      }
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        if constexpr (KEEP) {
          if (own[j] && io.keepv[c][s]) io.keepv[c][s][at[j]] = y[c];
        }
        w[j][c] = x[j][c];
        x[j][c] = y[c];
      }
    }
  }
  if constexpr (DOTS) {
    const double z = wave_sums<NV>(v);
    double& r = red[s0 / U][wave][wave_slot<NV>(lane)];
    if ((lane & (64 / NV - 1)) == 0) r = q == q0 ? z : r + z;
  }
  }
#pragma unroll
  for (int j = 0; j < C; ++j)
    if (own[j]) {
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        if (!KEEP && io.o1[0]) {
          io.o1[c][at[j]] = w[j][c];
          io.o2[c][at[j]] = x[j][c];
        }
        if constexpr (!DOTS) io.acc_out[c][at[j]] = acc[j][c];
      }
    }
  if constexpr (DOTS && FIRST) {
    const double z0 = wave_sums<2>(v0);
    double& r = red0[wave][wave_slot<2>(lane)];
    if ((lane & 31) == 0) r = q == q0 ? z0 : r + z0;
  }
  }
  if constexpr (DOTS) {
    // one partial per dot and workgroup: the wavefronts' sums in order
    __syncthreads();
    const int64_t rs = (int64_t)A.items * A.B, o = (int64_t)item * A.B + col;
    if (l < 2 * io.steps) {
      const int s = l / 2, r = l & 1, k = io.k0 + s;
      const int ire = PS * (s % U) + r, iim = r == 0 ? (IM ? ire + 2 : -1) : (NC == 2 ? ire + 2 : -1);
      double re = 0.0, im = 0.0;
      for (int u = 0; u < NW; ++u) {
        re += red[s / U][u][ire];
        if (iim >= 0) im += red[s / U][u][iim];
      }
      if (k <= io.k_end) io.part[rs * (2 * k - 1 + r) + o] = make_double2(re, im);
    } else if (FIRST && l == 2 * io.steps) {
      double re = 0.0, im = 0.0;
      for (int u = 0; u < NW; ++u) {
        re += red0[u][0];
        if (IM) im += red0[u][1];
      }
      io.part[o] = make_double2(re, im);
    }
  }
}


// Workgroups: 640 or 1024 cells in two dimensions, eight or four steps; 256 lanes of four (one
// chain) or two cells on a chain, 24 steps (plan_patch).
constexpr int patch_cells(int fam) { return two_chains(fam) ? 2 : 4; }

template <int PAT, int HOP>
hipError_t launch_patch_pattern(int family, int lanes, const MarchMat& A, const MarchIO& io, hipStream_t s) {
  const dim3 grid((unsigned)(A.items * A.B));
  auto go = [&](auto Fc) -> hipError_t {
    constexpr int F = decltype(Fc)::value;
    auto with = [&](auto Lc) -> hipError_t {
      constexpr int L = decltype(Lc)::value, C = PAT == MARCH_CHAIN ? patch_cells(F) : 1;
      auto kept = [&](auto Kc) {
        constexpr bool KP = decltype(Kc)::value;
        if (io.first) k_patch<PAT, F, HOP, L, C, true, KP><<<grid, L, 0, s>>>(A, io);
        else k_patch<PAT, F, HOP, L, C, false, KP><<<grid, L, 0, s>>>(A, io);
        return hipGetLastError();
      };
      if constexpr (F == MF_SYM || F == MF_PAIR || F == MF_EVO2) {
        if (io.keep) return kept(std::true_type{});
      }
      return kept(std::false_type{});
    };
    if constexpr (PAT == MARCH_CHAIN) {
      return lanes == 256 ? with(IC<256>{}) : hipErrorInvalidValue;
    } else {
      return lanes == 640 ? with(IC<640>{}) : lanes == 1024 ? with(IC<1024>{}) : hipErrorInvalidValue;
    }
  };
  switch (family) {
    case MF_SYM: return go(IC<MF_SYM>{});
    case MF_PAIR: return go(IC<MF_PAIR>{});
    case MF_EVO: return go(IC<MF_EVO>{});
    case MF_EVO2: return go(IC<MF_EVO2>{});
    case MF_MSD: return go(IC<MF_MSD>{});
    default: return hipErrorInvalidValue;
  }
}

}  // namespace march
}  // namespace gpuqt
