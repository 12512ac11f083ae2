// The march kernel (see march.h): T Chebyshev steps per launch in one sweep over
// the lattice, instead of one sweep per step.
//
// What bounds a step of the general kernels is memory: three vectors move per step
// (v_{n-1} in, v_{n-2} in, v_n out) and the keys.  Here a workgroup holds a strip (a tile)
// of cells, with a margin of T cells on every side, and marches along the slowest
// direction.  Level s is step k0 + s - 2 of the recurrence (level 1 = v_{k0-1}); iteration i
// takes up row i of level 1 and computes row i - s + 1 of every level s = 2 .. T + 1, each
// from three rows of the level above, held in registers by the lane that owns the cell (the
// neighbours along the march), and from that row's neighbours across it, which the lanes
// staged in LDS one iteration before (double-buffered: one barrier an iteration).  So a
// launch reads two vectors and writes two for T steps; margins are computed twice, and
// their rows are read twice, mostly from a cache.  The next rows are loaded one iteration
// ahead.  Nothing is kept between launches but the two last elements of each chain.
//
// Measured per step (one MI355X, copy rate 6.2 TB/s), the kernel that took one step per
// launch before and this one: square 2000^2, one vector, Hermitian step 47 -> 9.9 us (T = 8,
// two waves a SIMD; T = 4 14.8, T = 6 11.3, T = 10 11.8 at one wave), two chains 91.5 -> 26.2
// (T = 5); brick 2000 x 1000 with complex hoppings, Hermitian 21 -> 9.4 (T = 5), two chains
// 34 -> 21 (T = 4); box 200^3, four vectors, Hermitian 277 -> 160 (T = 3; T = 2 232), MSD term
// 945 -> 684 (T = 2): there the counted traffic, 1.22 and 1.24 of two elements read and two
// written a chain, moves at 86 and 90 % of the copy rate.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "device_common.h"
#include "march.h"

namespace gpuqt {
namespace march {

using namespace dev;

constexpr bool two_chains(int fam) { return fam == MF_PAIR || fam == MF_EVO2 || fam == MF_MSD; }
constexpr bool has_dots(int fam) { return fam == MF_SYM || fam == MF_PAIR; }

// LDS elements of one staged row (plane): the tile's cells and a margin of one
// row of cells (at most kMaxTileX in a box) on either side, so that a neighbour
// index never leaves it.
constexpr int kMaxTileX = 64;
constexpr int margin_of(int pat) { return pat == MARCH_BOX ? kMaxTileX : 1; }

// Sums over the wavefront of N values a lane holds (N a power of two, at most 64): while
// more than one is left, a lane hands half of them to the lane `off` away and takes that
// lane's other half, so that N values cost N - 1 exchanges (not 6 N); the last steps add the
// copies up.  Afterwards lane l holds the sum of value wave_slot<N>(l) of all lanes.
// (A bit select, not a conditional: that becomes an index into v, a chain of compares.)
template <int N>
__device__ __forceinline__ double wave_sums(double (&v)[N]) {
  const int lane = threadIdx.x & 63;
  int off = 32;
#pragma unroll
  for (int half = N / 2; half >= 1; half >>= 1, off >>= 1) {
    const uint32_t m32 = (lane & off) ? 0xffffffffu : 0u;
    const uint64_t m = ((uint64_t)m32 << 32) | m32;
#pragma unroll
    for (int i = 0; i < half; ++i) {
      const uint64_t lo = __builtin_bit_cast(uint64_t, v[i]), hi = __builtin_bit_cast(uint64_t, v[i + half]);
      const double keep = __builtin_bit_cast(double, (hi & m) | (lo & ~m));
      const double give = __builtin_bit_cast(double, (lo & m) | (hi & ~m));
      v[i] = keep + __shfl_xor(give, off);
    }
  }
#pragma unroll
  for (; off >= 1; off >>= 1) v[0] += __shfl_xor(v[0], off);
  return v[0];
}
template <int N>
__device__ __forceinline__ int wave_slot(int lane) {
  int i = 0, off = 32;
#pragma unroll
  for (int half = N / 2; half >= 1; half >>= 1, off >>= 1) i |= (lane & off) ? half : 0;
  return i;
}

// One row (plane) of a vector as a buffer: its base is the same in every lane and
// stays in scalar registers, a lane adds a 32-bit byte offset, and an access past
// the row (offset kNoLane) reads zero and stores nothing, so that masked stores
// need no branch and the compiler's count of accesses in flight stays exact.
constexpr uint32_t kNoLane = 0xfffffff0u;
struct RowBuf {
  __amdgpu_buffer_rsrc_t r;
  __device__ __forceinline__ RowBuf(const void* base, int64_t off, uint32_t bytes)
      : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(static_cast<const char*>(base)) + off, 0, bytes, 0x00020000)) {}
  __device__ __forceinline__ double2 ld2(uint32_t o) const {
    typedef unsigned int u4 __attribute__((ext_vector_type(4)));
    const u4 v = __builtin_amdgcn_raw_buffer_load_b128(r, o, 0, 0);
    const d2v d = __builtin_bit_cast(d2v, v);
    return make_double2(d.x, d.y);
  }
  __device__ __forceinline__ double ld1(uint32_t o) const {
    typedef unsigned int u2 __attribute__((ext_vector_type(2)));
    const u2 v = __builtin_amdgcn_raw_buffer_load_b64(r, o, 0, 0);
    return __builtin_bit_cast(double, v);
  }
  template <int AUX = 0>
  __device__ __forceinline__ void st2(uint32_t o, double2 v) const {
    typedef unsigned int u4 __attribute__((ext_vector_type(4)));
    const d2v d = {v.x, v.y};
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, d), r, o, 0, AUX);
  }
};

// (two chains with their dots need more than the 256 registers of two waves a SIMD: spilled to fit them, the
// brick lattice's step costs 18.4 us instead of 16.5 at one wave)
template <int PAT, int FAM, int HOP, int T, int LANES, bool FIRST, bool KEEP>
__global__ __launch_bounds__(LANES, PAT == MARCH_BOX ? 4 : FAM == MF_PAIR ? 1 : 2) void k_march(MarchMat A, MarchIO io) {
  constexpr int NC = two_chains(FAM) ? 2 : 1;
  constexpr bool DOTS = has_dots(FAM);
  constexpr bool BOX = PAT == MARCH_BOX;
  constexpr int K = PAT == MARCH_BRICK ? 3 : PAT == MARCH_BOX ? 6 : 4;
  constexpr bool ENTRY = HOP != HOP_UNIFORM;
  constexpr bool CPLX = HOP == HOP_COMPLEX || HOP == HOP_DICT;
  constexpr int KE = ENTRY ? K : 1;
  // rows loaded ahead: two where the registers allow it (2 - 8 % on squares, none on boxes)
  constexpr int AHEAD = !ENTRY && PAT != MARCH_BOX && FAM != MF_PAIR ? 2 : 1;
  // outputs past the caches (bit 1: non-temporal): 4 % on the box MSD term, none or a loss elsewhere
  constexpr int NTS = BOX && FAM == MF_MSD ? 2 : 0;
  constexpr bool IM = NC == 2 || ENTRY;   // (one chain, one real hopping: H~ is real symmetric and every dot real)
  using hv_t = std::conditional_t<CPLX, double2, double>;
  constexpr int SLOTS = LANES + 2 * margin_of(PAT);
  __shared__ double2 lds[2 * NC * T * SLOTS];   // [2][NC][T][SLOTS]

  // consecutive work items to one XCD (workgroups go to the 8 XCDs round-robin), so that
  // tiles that share margins, or columns that share lines, meet in its L2
  const int total = A.items * A.B, xcd = blockIdx.x & 7;
  const int lb = xcd * (total >> 3) + min(xcd, total & 7) + ((int)blockIdx.x >> 3);
  // (the quotients are the same in every lane; readfirstlane keeps them and the
  // addresses built on them in scalar registers)
  auto uni = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
  // rows of B columns (KEEP): the columns of a tile run together, so that the lines they
  // share meet in one L2; planar vectors: the tiles of a column do, for their margins
  const int major = uni(lb / (KEEP ? A.B : A.items)), minor = lb - major * (KEEP ? A.B : A.items);
  const int col = KEEP ? minor : major, item = KEEP ? major : minor;
  const int64_t sb = KEEP ? A.B : 1;   // elements between two rows of a vector
  int sg = 0;
  for (int hi = A.n_seg - 1; sg < hi;) {
    const int mid = (sg + hi + 1) >> 1;
    if (A.segs[mid].item0 <= item) sg = mid;
    else hi = mid - 1;
  }
  const MarchSeg S = A.segs[sg];
  const int q = item - S.item0;
  const int row = uni(q / S.nx), ix = q - row * S.nx;
  const int iz = BOX ? uni(row / S.ny) : row, iy = row - iz * S.ny;
  const int z0 = iz * S.zc, z1 = min(z0 + S.zc, S.Lm);

  // this lane's cell: position in the tile, wrapped lattice position, and whether
  // the tile owns it (lanes past the tile repeat its last cell)
  const int l = threadIdx.x;
  const int tl = min(l, S.tx * S.ty - 1);
  const int tyi = BOX ? tl / S.tx : 0, txi = BOX ? tl - tyi * S.tx : tl;
  const int X = ix * S.ux + txi - T, Y = BOX ? iy * S.uy + tyi - T : 0;
  auto wrap = [](int v, int L) { v %= L; return v < 0 ? v + L : v; };
  const int xw = wrap(X, S.Lx), yw = BOX ? wrap(Y, S.Ly) : 0;
  bool own = l < S.tx * S.ty && txi >= T && txi < T + S.ux && X < S.Lx;
  if (BOX) own = own && tyi >= T && tyi < T + S.uy && Y < S.Ly;
  const uint32_t cell = (uint32_t)(yw * S.Lx + xw);
  // past the edge of a lattice that is open in x: elements read as zero, and no hopping keeps them so
  const bool out = PAT == MARCH_SQUARE && !ENTRY && A.open && (X < 0 || X >= S.Lx);
  const uint32_t vo = out ? kNoLane : (cell * (uint32_t)sb + (KEEP ? (uint32_t)col : 0u)) * (uint32_t)sizeof(double2), dof = cell * (uint32_t)sizeof(double);
  const uint32_t so = own ? vo : kNoLane;
  const int64_t plane = (int64_t)S.Lx * S.Ly;
  const uint32_t nv = (uint32_t)(plane * sb) * (uint32_t)sizeof(double2);   // bytes of a row of a vector
  const uint32_t nvo = io.o1[0] ? nv : 0;   // the last launch of a series keeps no chain elements
  const int me = margin_of(PAT) + l;
  const int up = BOX ? S.tx : 1;

  const double hu2 = ENTRY || out ? 0.0 : 2.0 * A.seg_hop[sg];
  // position differences of this lane's x neighbours
  const double hdx = FAM == MF_MSD && BOX ? hu2 * A.dx : 0.0;
  double dxp = 0.0, dxm = 0.0;
  if constexpr (FAM == MF_MSD && !BOX) {
    dxp = A.dxcol[S.dx0 + xw];
    dxm = -A.dxcol[S.dx0 + (xw == 0 ? S.Lx - 1 : xw - 1)];
  }
  const int64_t vbase = KEEP ? S.off * sb : (int64_t)col * A.n + S.off;
  const char* xs[NC];
  const char* ws[NC];
  char* o1s[NC];
  char* o2s[NC];
  const char* as[NC];
  char* aos[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    xs[c] = reinterpret_cast<const char*>(io.x[c] + vbase);
    ws[c] = reinterpret_cast<const char*>((FIRST ? io.x[c] : io.w[c]) + vbase);
    o1s[c] = reinterpret_cast<char*>(io.o1[c] + vbase);
    o2s[c] = reinterpret_cast<char*>(io.o2[c] + vbase);
    if (!DOTS) {
      as[c] = reinterpret_cast<const char*>((FIRST ? io.x[c] : io.acc_in[c]) + vbase);
      aos[c] = reinterpret_cast<char*>(io.acc_out[c] + vbase);
    }
  }
  const char* ds = reinterpret_cast<const char*>(A.diag + S.off);
  const bool bz = NC == 2 && FIRST && io.zero_b;   // chain b starts from zero

  // history: h[c][s][.] rows of level s + 1 (level 1 = x, level T + 1 = the last step),
  // a ring of three: the newest row, the one before and the one before that
  double2 h[NC][T][3];
  double2 wv[NC], av[DOTS ? 1 : NC];   // w of level 2's row, sums of level T + 1's
  double dq[T];                      // diagonal of the rows levels 2 .. T + 1 work on
  hv_t hq[ENTRY ? T : 1][KE];        // and their hoppings
  double ar[T], ai[T], cr[T], ci[T], zr = 0.0, zi = 0.0;   // dots
  double2 cm[DOTS ? 1 : T];
  double c0 = 0.0;
#pragma unroll
  for (int s = 0; s < T; ++s) {
    ar[s] = ai[s] = cr[s] = ci[s] = 0.0;
    dq[s] = 0.0;
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int p = 0; p < 3; ++p) h[c][s][p] = make_double2(0.0, 0.0);
    if constexpr (ENTRY)
#pragma unroll
      for (int j = 0; j < K; ++j) hq[s][j] = hv_t{};
    if constexpr (!DOTS) {
      // c_m of step m = k0 + s: J_m (-i sgn)^m, zero past the last term
      const int m = io.k0 + s;
      const double j = m <= io.k_end ? io.J[(int64_t)sg * io.ldJ + m] : 0.0;
      const double sg1 = io.sgn;
      cm[s] = (m & 3) == 0 ? make_double2(j, 0.0) : (m & 3) == 1 ? make_double2(0.0, -sg1 * j)
              : (m & 3) == 2 ? make_double2(-j, 0.0) : make_double2(0.0, sg1 * j);
    }
  }
  if constexpr (!DOTS) c0 = FIRST ? io.J[(int64_t)sg * io.ldJ] : 0.0;
#pragma unroll
  for (int c = 0; c < NC; ++c) wv[c] = make_double2(0.0, 0.0);
  for (int e = l; e < 2 * NC * T * SLOTS; e += LANES) lds[e] = make_double2(0.0, 0.0);

  // row (plane) offsets, wrapped: iteration i takes up row i of x and row i - 1 of w, the
  // diagonal, the hoppings and the sums, i = z0 - T, ...
  int rx = uni(wrap(z0 - T, S.Lm)), rw = uni(wrap(z0 - T - 1, S.Lm));   // rows to load next
  const int64_t pv = plane * sb * (int64_t)sizeof(double2);
  int64_t bx = rx * pv, bw = rw * pv;     // their byte offsets
  int ra = uni(wrap(z0 - 2 * T, S.Lm));   // row of the sums, level T + 1's
  int64_t ba = ra * pv;
  int64_t b1 = (z0 - 2 * T + 1) * pv;     // and that of the row level T computes next
  auto next = [&](int r) { return r + 1 == S.Lm ? 0 : r + 1; };
  double2 nx[3][NC], nw[3][NC], na[3][DOTS ? 1 : NC];   // rows on their way, by phase
  double nd[3];
  hv_t nh[3][KE];
  int32_t nk[KE];                         // table keys of the row after nh's
  auto entry0 = [&](int r) -> int64_t {   // first stored entry of the lane's row r
    const int64_t row = S.off + (int64_t)r * plane + cell;
    return (row >> A.S_log2) * ((int64_t)K << A.S_log2) + (row & ((1 << A.S_log2) - 1));
  };
  auto load_keys = [&](int r) {
    if constexpr (HOP == HOP_DICT) {
      const int64_t e = entry0(r);
#pragma unroll
      for (int j = 0; j < K; ++j) nk[j] = A.hidx[e + ((int64_t)A.slot[j] << A.S_log2)];
    }
  };
  auto load = [&](auto Qc) {
    constexpr int Q = decltype(Qc)::value;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      nx[Q][c] = RowBuf(xs[c], bx, nv).ld2(vo);
      if (!FIRST) nw[Q][c] = RowBuf(ws[c], bw, nv).ld2(vo);
      if (!DOTS) na[Q][c] = RowBuf(as[c], ba, nv).ld2(so);
    }
    nd[Q] = RowBuf(ds, rw * plane * (int64_t)sizeof(double), (uint32_t)plane * (uint32_t)sizeof(double)).ld1(dof);
    if constexpr (HOP == HOP_DICT) {
#pragma unroll
      for (int j = 0; j < K; ++j) nh[Q][j] = A.htab[nk[j]];
      load_keys(next(rw));
    } else if constexpr (ENTRY) {
      const int64_t e = entry0(rw);
#pragma unroll
      for (int j = 0; j < K; ++j) {
        const int64_t ej = e + ((int64_t)A.slot[j] << A.S_log2);
        if constexpr (HOP == HOP_REAL) nh[Q][j] = A.hop[ej];
        else nh[Q][j] = reinterpret_cast<const double2*>(A.hop)[ej];
      }
    }
    if (!DOTS) {
      ba = ra + 1 == S.Lm ? 0 : ba + pv;
      ra = next(ra);
    }
    bx = rx + 1 == S.Lm ? 0 : bx + pv;
    bw = rw + 1 == S.Lm ? 0 : bw + pv;
    rx = next(rx);
    rw = next(rw);
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  load_keys(rw);
  load(I0{});
  if constexpr (AHEAD == 2) load(I1{});
  __syncthreads();

  double2* rd = lds + NC * T * SLOTS + me;   // staged rows of the last iteration
  double2* wr = lds + me;                    // and of this one
  auto axpy_c = [](double2& t, double2 a, double2 b) {
    t.x = fma(a.x, b.x, fma(-a.y, b.y, t.x));
    t.y = fma(a.x, b.y, fma(a.y, b.x, t.y));
  };
  // t += a b
  auto axpy = [](double2& t, hv_t a, double2 b) {
    if constexpr (CPLX) {
      t.x = fma(a.x, b.x, fma(-a.y, b.y, t.x));
      t.y = fma(a.x, b.y, fma(a.y, b.x, t.y));
    } else {
      t.x = fma(a, b.x, t.x);
      t.y = fma(a, b.y, t.y);
    }
  };
  // Iteration i, P = (i - i0) mod 3: the newest rows at P, older ones at P + 2 and P + 1.
  // CHK: some level's row may lie outside [z0, z1); otherwise all are inside.
  auto iter = [&](int i, auto Pc, auto Cc) {
    constexpr int P = decltype(Pc)::value, P1 = (P + 2) % 3, P2 = (P + 1) % 3;
    constexpr bool CHK = decltype(Cc)::value;
    auto inside = [&](int r) { return !CHK || (r >= z0 && r < z1); };
    // take up the loaded rows, shift the queues, and load the next ones
#pragma unroll
    for (int s = T - 1; s > 0; --s) {
      dq[s] = dq[s - 1];
      if constexpr (ENTRY)
#pragma unroll
        for (int j = 0; j < K; ++j) hq[s][j] = hq[s - 1][j];
    }
    dq[0] = 2.0 * nd[P];
    if constexpr (ENTRY)
#pragma unroll
      for (int j = 0; j < K; ++j) {
        if constexpr (CPLX) hq[0][j] = cscale(2.0, nh[P][j]);
        else hq[0][j] = 2.0 * nh[P][j];
      }
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      h[c][0][P] = (c == 1 && bz) ? make_double2(0.0, 0.0) : nx[P][c];
      wv[c] = FIRST ? make_double2(0.0, 0.0) : nw[P][c];
      if constexpr (!DOTS) av[c] = (c == 1 && bz) ? make_double2(0.0, 0.0) : na[P][c];
    }
    load(std::integral_constant<int, AHEAD == 2 ? P1 : (P + 1) % 3>{});
#pragma unroll
    for (int s = 0; s < T; ++s) {         // level s + 2 from level s + 1; its row is i - 1 - s
      const int r = i - 1 - s;
      double2 y[NC], sx = make_double2(0.0, 0.0);
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const double2* L = rd + (c * T + s) * SLOTS;
        const double2 xp = L[1], xm = L[-1];
        const double2 xc = h[c][s][P1];
        const double2 zp = h[c][s][P], zm = h[c][s][P2];
        const double2 w2 = s == 0 ? wv[c] : h[c][s > 0 ? s - 1 : 0][P2];
        // t = 2 H~ x - w (the diagonal and the hoppings are held doubled); the newest row,
        // zp, comes from the level above in this very iteration and enters last
        double2 t = make_double2(fma(dq[s], xc.x, -w2.x), fma(dq[s], xc.y, -w2.y));
        if constexpr (ENTRY) {
          if constexpr (FAM == MF_MSD) {
            double2 p = make_double2(0.0, 0.0), m = p;
            axpy(p, hq[s][0], xp);
            axpy(m, hq[s][1], xm);
            if (c == 0) sx = make_double2(fma(dxp, p.x, dxm * m.x), fma(dxp, p.y, dxm * m.y));
            t = cadd(t, cadd(p, m));
          } else {
            axpy(t, hq[s][0], xp);
            axpy(t, hq[s][1], xm);
          }
          if constexpr (PAT == MARCH_BRICK) {
            axpy(t, hq[s][K - 1], ((xw + r + A.parity) & 1) == 0 ? zp : zm);
          } else {
            axpy(t, hq[s][K - 1], zm);
            axpy(t, hq[s][K - 2], zp);
          }
        } else {
          double2 n = cadd(xp, xm);
          if constexpr (FAM == MF_MSD) {
            if (c == 0) {
              if constexpr (BOX) sx = make_double2(hdx * (xp.x - xm.x), hdx * (xp.y - xm.y));
              else sx = make_double2(hu2 * fma(dxp, xp.x, dxm * xm.x), hu2 * fma(dxp, xp.y, dxm * xm.y));
            }
          }
          if constexpr (BOX) {
            n = cadd(n, L[up]);
            n = cadd(n, L[-up]);
          }
          if constexpr (PAT == MARCH_BRICK) {
            n = cadd(n, ((xw + r + A.parity) & 1) == 0 ? zp : zm);
          } else {
            n = cadd(n, zm);
            n = cadd(n, zp);
          }
          t = make_double2(fma(hu2, n.x, t.x), fma(hu2, n.y, t.y));
        }
        if constexpr (FAM == MF_MSD) {     // + 2 [X, H~] a, [X, H~]_rj = -dx_rj H~_rj
          if (c == 1) t = make_double2(t.x - sx.x, t.y - sx.y);
        }
        y[c] = (FIRST && s == 0) ? cscale(0.5, t) : t;   // v_1 = H~ v_0, half of 2 H~ v_0 - 0
        wr[(c * T + s) * SLOTS] = zp;      // staged for the next iteration
      }
      if constexpr (DOTS) {
        const double2 xa = h[0][s][P1], xb = h[NC - 1][s][P1];
        double a0 = ar[s], a1 = ai[s], b0 = cr[s], b1 = ci[s], d0 = zr, d1 = zi;
        if (FIRST && s == 0) {
          if constexpr (IM) {
            cdot_acc(d0, d1, xa, xb);                 // <a0|b0>
            cdot_acc(a0, a1, xa, y[NC - 1]);          // <a0|b1>
          } else {
            d0 = fma(xa.x, xa.x, fma(xa.y, xa.y, d0));
            a0 = fma(y[0].x, xa.x, fma(y[0].y, xa.y, a0));
          }
        } else if constexpr (IM) {
          cdot_acc(a0, a1, y[0], xb);
        } else {
          a0 = fma(y[0].x, xb.x, fma(y[0].y, xb.y, a0));
        }
        if constexpr (NC == 1) b0 = fma(y[0].x, y[0].x, fma(y[0].y, y[0].y, b0));
        else cdot_acc(b0, b1, y[0], y[NC - 1]);
        // lanes the tile does not own sum up whatever they hold; it is dropped at the end
        const bool in = inside(r);
        ar[s] = in ? a0 : ar[s];
        if constexpr (IM) ai[s] = in ? a1 : ai[s];
        cr[s] = in ? b0 : cr[s];
        if constexpr (NC == 2) ci[s] = in ? b1 : ci[s];
        if (FIRST && s == 0) {
          zr = in ? d0 : zr;
          zi = in ? d1 : zi;
        }
      }
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        if (s + 1 < T) h[c][s + 1 < T ? s + 1 : 0][P] = y[c];
        const bool out = s == T - 1, pre = s == T - 2;
        if (KEEP && !(out || pre))
          RowBuf(io.keepv[c][s] + vbase, b1 + (T - 2 - s) * pv, io.keepv[c][s] ? nv : 0).st2(inside(r) ? so : kNoLane, y[c]);
        if (out || pre) {
          const uint32_t o = inside(r) ? so : kNoLane;
          if (KEEP) RowBuf(io.keepv[c][s] + vbase, out ? b1 - pv : b1, io.keepv[c][s] ? nv : 0).st2(o, y[c]);
          else RowBuf(out ? o2s[c] : o1s[c], out ? b1 - pv : b1, nvo).template st2<NTS>(o, y[c]);
          if constexpr (!DOTS) {
            if (out) {
              // the sums of level T + 1's row: the steps before it are this row in the
              // levels below (T <= 3 of them, all still held)
              double2 a = av[c];
              if (FIRST) a = cscale(c0, a);       // c_0 v_0
#pragma unroll
              for (int m = 0; m < T; ++m) {
                double2 v = m == T - 1 ? y[c] : m == T - 2 ? h[c][T - 1][P1] : h[c][T > 2 ? T - 2 : 0][P2];
                if (io.k0 + m > io.k_end) v = make_double2(0.0, 0.0);
                axpy_c(a, cm[m], v);
              }
              RowBuf(aos[c], b1 - pv, nv).template st2<NTS>(o, a);
            }
          }
        }
      }
    }
    b1 += pv;
    double2* t = rd;
    rd = wr;
    wr = t;
    __syncthreads();
  };
  // level T + 1 has row z0 at i = z0 + T and row z1 - 1 at i = z1 - 1 + T
  int i = z0 - T;
  auto three = [&](auto Cc) {
    iter(i, I0{}, Cc);
    iter(i + 1, I1{}, Cc);
    iter(i + 2, I2{}, Cc);
    i += 3;
  };
  while (i < z0 + T) three(std::true_type{});
  while (i + 2 <= z1) three(std::false_type{});
  while (i < z1 + T) three(std::true_type{});
  if constexpr (DOTS) {
    // one partial per dot and workgroup: the wavefront's sums, then the wavefronts in order
    double* red = reinterpret_cast<double*>(lds);
    const int wave = l >> 6, lane = l & 63, nw2 = LANES >> 6;
    constexpr int ND = 4 * T + 2, N = ND <= 16 ? 16 : ND <= 32 ? 32 : 64;
    double v[N];
#pragma unroll
    for (int s = 0; s < N / 4; ++s) {
      v[4 * s] = s < T && own ? ar[s < T ? s : 0] : 0.0;
      v[4 * s + 1] = s < T && own ? ai[s < T ? s : 0] : 0.0;
      v[4 * s + 2] = s < T && own ? cr[s < T ? s : 0] : 0.0;
      v[4 * s + 3] = s < T && own ? ci[s < T ? s : 0] : 0.0;
    }
    v[4 * T] = own ? zr : 0.0;
    v[4 * T + 1] = own ? zi : 0.0;
    const double z = wave_sums<N>(v);
    const int d = wave_slot<N>(lane);
    if ((lane & (64 / N - 1)) == 0 && d < ND) red[wave * ND + d] = z;
    __syncthreads();
    if (l < 2 * T + 1) {
      double re = 0.0, im = 0.0;
      for (int w = 0; w < nw2; ++w) {
        re += red[w * ND + 2 * l];
        im += red[w * ND + 2 * l + 1];
      }
      const int64_t rs = (int64_t)A.items * A.B;
      const int64_t o = (int64_t)item * A.B + col;
      const int k = io.k0 + l / 2;
      if (l == 2 * T) {
        if (FIRST) io.part[o] = make_double2(re, im);
      } else if (k <= io.k_end) {
        io.part[rs * (2 * k - 1 + (l & 1)) + o] = make_double2(re, im);
      }
    }
  }
}


// Steps per launch of each kernel: more of them mean fewer bytes per step, more
// registers (12 per level and chain, and the hoppings of T rows) and wider margins.  The
// counts are the fastest that keep two waves a SIMD (a box: 16 waves of one workgroup; two chains with
// their dots run at one), measured as above; the sums of a series are formed where the last three
// levels meet, so T <= 3 there.
static_assert(kMarchMaxSteps >= 8, "the most steps of steps_of");
constexpr int steps_of(int pat, int hop, int fam) {
  const bool entry = hop != HOP_UNIFORM;
  if (pat == MARCH_BOX) return entry ? 0 : fam == MF_SYM ? 3 : fam == MF_EVO ? 3 : 2;
  if (!entry) return fam == MF_SYM ? 8 : fam == MF_PAIR ? 5 : 3;
  if (pat == MARCH_BRICK) return fam == MF_SYM ? 5 : fam == MF_PAIR ? 4 : 3;
  return fam == MF_SYM ? 4 : fam == MF_PAIR ? 3 : fam == MF_EVO ? 3 : 2;
}

template <int PAT, int HOP>
hipError_t launch_pattern(int family, int lanes, const MarchMat& A, const MarchIO& io, hipStream_t s) {
  const dim3 grid((unsigned)(A.items * A.B));
  auto go = [&](auto Fc) -> hipError_t {
    constexpr int F = decltype(Fc)::value, T = steps_of(PAT, HOP, F);
    auto with = [&](auto Lc) -> hipError_t {
      constexpr int L = decltype(Lc)::value;
      auto kept = [&](auto Kc) {
        constexpr bool KP = decltype(Kc)::value;
        if (io.first) k_march<PAT, F, HOP, T, L, true, KP><<<grid, L, 0, s>>>(A, io);
        else k_march<PAT, F, HOP, T, L, false, KP><<<grid, L, 0, s>>>(A, io);
        return hipGetLastError();
      };
      if constexpr (F == MF_SYM || F == MF_PAIR || F == MF_EVO2) {
        if (io.keep) return kept(std::true_type{});
      }
      return kept(std::false_type{});
    };
    if constexpr (PAT == MARCH_BOX) {
      return lanes == 1024 ? with(IC<1024>{}) : hipErrorInvalidValue;
    } else {
      return lanes == 64 ? with(IC<64>{}) : lanes == 128 ? with(IC<128>{}) : hipErrorInvalidValue;
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
