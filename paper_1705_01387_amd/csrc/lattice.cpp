// Lattices of the march kernels (march.h): recognising them in a descriptor and
// cutting them into the tiles of a launch.  Host code only.
#include <algorithm>
#include <cmath>

#include "internal.h"
#include "march.h"

namespace gpuqt {

namespace {

// The dims of a segment of n rows that is a BRICK lattice, from row 0's neighbours
// (1, Lx - 1 and Lx or (Ly - 1) Lx); every row must have its three neighbours in the
// slots of row 0.  slot = stored slots of (+x, -x, vertical).
bool brick_dims(const gpuqt_h_desc* d, int64_t off, int64_t n, int32_t dims[3], int32_t slot[3], int32_t* parity) {
  const int64_t k = d->max_nn;
  const int32_t* r0 = d->nbr + off * k;
  for (int cand = 0; cand < 3; ++cand) {
    const int64_t Lx = (int64_t)r0[cand] - off + 1;   // candidate: the -x neighbour of (0, 0) is Lx - 1
    if (Lx < 4 || Lx % 2 || n % Lx || Lx > (1 << 24)) continue;
    const int64_t Ly = n / Lx;
    if (Ly < 4 || Ly % 2 || Ly > INT32_MAX) continue;
    for (int par = 0; par < 2; ++par) {
      int32_t s[3] = {-1, cand, -1};
      for (int j = 0; j < 3; ++j) {
        const int64_t c = r0[j] - off;
        if (j == cand) continue;
        if (c == 1 && s[0] < 0) s[0] = j;
        else if (c == (par == 0 ? Lx : (Ly - 1) * Lx)) s[2] = j;
      }
      if (s[0] < 0 || s[2] < 0) continue;
      bool ok = true;
      for (int64_t y = 0; y < Ly && ok; ++y) {
        const int64_t up = off + (y + 1 == Ly ? 0 : y + 1) * Lx, dn = off + (y == 0 ? Ly - 1 : y - 1) * Lx;
        const int64_t row = off + y * Lx;
        for (int64_t x = 0; x < Lx; ++x) {
          const int32_t* c = d->nbr + (row + x) * k;
          if (d->nn[row + x] != 3 || c[s[0]] != row + (x + 1 == Lx ? 0 : x + 1) ||
              c[s[1]] != row + (x == 0 ? Lx - 1 : x - 1) || c[s[2]] != (((x + y + par) & 1) == 0 ? up : dn) + x) {
            ok = false;
            break;
          }
        }
      }
      if (!ok) continue;
      dims[0] = (int32_t)Lx;
      dims[1] = 1;
      dims[2] = (int32_t)Ly;
      std::copy(s, s + 3, slot);
      *parity = par;
      return true;
    }
  }
  return false;
}

// Lx of a segment of n rows that is a square open in x and periodic in y (each at least 3), its
// neighbours in any order; 0: it is not.
int64_t open_square(const gpuqt_h_desc* d, int64_t off, int64_t n) {
  const int64_t k = d->max_nn;
  if (n < 9 || d->nn[off] != 3) return 0;
  int64_t c[3] = {d->nbr[off * k] - off, d->nbr[off * k + 1] - off, d->nbr[off * k + 2] - off};
  std::sort(c, c + 3);   // 1, Lx, (Ly - 1) Lx
  const int64_t Lx = c[1];
  if (c[0] != 1 || Lx < 3 || n % Lx || n / Lx < 3) return 0;
  const int64_t Ly = n / Lx;
  for (int64_t y = 0; y < Ly; ++y) {
    const int64_t row = off + y * Lx, up = off + (y + 1 == Ly ? 0 : y + 1) * Lx, dn = off + (y == 0 ? Ly - 1 : y - 1) * Lx;
    for (int64_t x = 0; x < Lx; ++x) {
      const int edge = (x == 0 ? 2 : 0) | (x + 1 == Lx ? 1 : 0);
      int seen = edge;
      const int nn = d->nn[row + x];
      for (int j = 0; j < nn && j < 4; ++j) {
        const int64_t q = d->nbr[(row + x) * k + j];
        seen |= q == row + x + 1 && !(edge & 1) ? 1 : q == row + x - 1 && !(edge & 2) ? 2 : q == up + x ? 4 : q == dn + x ? 8 : 16;
      }
      if (seen != 15 || nn != (edge ? 3 : 4)) return 0;
    }
  }
  return Lx;
}

}  // namespace

bool detect_lattice(const gpuqt_h_desc* d, const HostLayout& L, const int32_t box[3],
                    const std::vector<int32_t>& sheets, MarchLattice* M) {
  *M = MarchLattice();
  const int n_seg = L.n_seg;
  bool chain = false;
  if (box[0] > 0) {
    M->pattern = MARCH_BOX;
    M->dims = {box[0], box[1], box[2]};
  } else if (!sheets.empty()) {
    M->pattern = MARCH_SQUARE;
    for (int s = 0; s < n_seg; ++s) M->dims.insert(M->dims.end(), {sheets[2 * s], 1, sheets[2 * s + 1]});
  } else if (L.uniform_width == 3 && d->nn && d->nbr) {
    for (int s = 0; s < n_seg; ++s) {
      int32_t dims[3], slot[3], par = 0;
      if (!brick_dims(d, L.seg_off[s], L.seg_off[s + 1] - L.seg_off[s], dims, slot, &par)) return false;
      if (s > 0 && (par != M->parity || !std::equal(slot, slot + 3, M->slot))) return false;
      M->parity = par;
      std::copy(slot, slot + 3, M->slot);
      M->dims.insert(M->dims.end(), dims, dims + 3);
    }
    M->pattern = MARCH_BRICK;
  } else if (L.uniform_width == 8 && d->nn && d->nbr) {
    // row 0's neighbours sorted: 1, Lx - 1, Lx, ...; the slots, the same on every row, are checked below
    for (int s = 0; s < n_seg; ++s) {
      const int64_t off = L.seg_off[s], n = L.seg_off[s + 1] - off;
      int32_t c[8];
      std::copy(d->nbr + off * d->max_nn, d->nbr + off * d->max_nn + 8, c);
      std::sort(c, c + 8);
      const int64_t Lx = c[2] - off;
      if (Lx < 3 || n % Lx || n / Lx < 3 || n > INT32_MAX) return false;
      M->dims.insert(M->dims.end(), {(int32_t)Lx, 1, (int32_t)(n / Lx)});
    }
    M->pattern = MARCH_NNN;
  } else if (L.uniform_width == 2 && d->nn && d->nbr) {
    // rings in natural order, at least three sites each (their neighbours are checked below)
    for (int s = 0; s < n_seg; ++s) {
      const int64_t n = L.seg_off[s + 1] - L.seg_off[s];
      if (n < 3 || n > (int64_t(1) << 30)) return false;
      M->dims.insert(M->dims.end(), {(int32_t)n, 1, 1});
    }
    chain = true;
  } else if (L.uniform_width == 0 && L.hop_mode == HOP_UNIFORM && d->max_nn >= 4 && d->nn && d->nbr) {
    for (int s = 0; s < n_seg; ++s) {
      const int64_t n = L.seg_off[s + 1] - L.seg_off[s], Lx = open_square(d, L.seg_off[s], n);
      if (Lx == 0 || n > INT32_MAX) return false;
      M->dims.insert(M->dims.end(), {(int32_t)Lx, 1, (int32_t)(n / Lx)});
    }
    M->pattern = MARCH_SQUARE;
    M->open = 1;
  } else {
    return false;
  }
  // rows (planes) of blocks of 16 vectors are addressed with 32-bit byte offsets
  for (int s = 0; s < n_seg; ++s)
    if (!chain && (int64_t)M->dims[3 * s] * M->dims[3 * s + 1] >= (int64_t(1) << 24)) {
      M->pattern = MARCH_NONE;
      return false;
    }
  // one pass over the rows: the stored slot of each square neighbour (needed where every
  // entry has its own hopping: it must be the same on every row) and the position steps
  const bool diag = M->pattern == MARCH_NNN;
  const bool slots = diag || ((M->pattern == MARCH_SQUARE || chain) && L.hop_mode != HOP_UNIFORM);
  const int nw = diag ? 8 : 4;
  const int K = M->open ? 4 : L.uniform_width, ls = __builtin_ctz((unsigned)L.S);
  auto entry = [&](int64_t r) { return L.slice_ptr[r >> ls] + (r & (L.S - 1)); };
  auto width = [&](int64_t r) { return M->open ? d->nn[r] : K; };
  auto diff = [&](int64_t e) { return L.hop_mode == HOP_DICT ? L.dxtab[L.hidx[e]] : L.dx[e]; };
  bool dx_ok = true;
  if (chain) {
    const int64_t S = L.S, e00 = entry(0);
    const bool first = L.col[e00] == 1;   // row 0 names +x first
    M->slot[0] = first ? 0 : 1;
    M->slot[1] = first ? 1 : 0;
    M->dx = diff(first ? e00 : e00 + S);
    const double* dx = L.hop_mode == HOP_DICT ? nullptr : L.dx.data();
    for (int s = 0; s < n_seg; ++s) {
      const int64_t off = L.seg_off[s], end = L.seg_off[s + 1];
      for (int64_t r = off; r < end; ++r) {
        const int64_t e0 = 2 * (r & -S) + (r & (S - 1)), e1 = e0 + S;   // (every row has two entries)
        const int64_t xp = r + 1 == end ? off : r + 1, xm = r == off ? end - 1 : r - 1;
        const bool fwd = L.col[e0] == xp && L.col[e1] == xm;
        if (!fwd && !(L.col[e0] == xm && L.col[e1] == xp)) return false;
        if (slots && fwd != first) return false;
        if (dx_ok) {
          const double d0 = dx ? dx[e0] : diff(e0), d1 = dx ? dx[e1] : diff(e1);
          dx_ok = (fwd ? d0 : d1) == M->dx && (fwd ? d1 : d0) == -M->dx;
        }
      }
    }
    M->pattern = MARCH_CHAIN;
    M->dx_ok = dx_ok ? 1 : 0;
    return true;
  }
  size_t col0 = 0;
  for (int s = 0; s < n_seg; ++s) {
    const int64_t Lx = M->dims[3 * s], Ly = M->dims[3 * s + 1], Lm = M->dims[3 * s + 2];
    const int64_t off = L.seg_off[s];
    M->dxcol.resize(col0 + Lx, 0.0);
    double* dxc = M->dxcol.data() + col0;
    col0 += Lx;
    for (int64_t x = 0; x < Lx; ++x)
      for (int j = 0, w = width(off + x); j < w; ++j) {
        const int64_t e = entry(off + x) + ((int64_t)j << ls);
        if (L.col[e] == off + (x + 1 == Lx ? 0 : x + 1)) dxc[x] = diff(e);
      }
    // where every row has row 0's positions, row 0's differences are every row's
    bool same = true;
    for (int64_t r = off + Lx, c = off, end = off + Lx * Ly * Lm; r < end && same; ++r, ++c) same = d->x[r] == d->x[c];
    for (int64_t z = 0, rows = same && !slots ? 1 : Ly * Lm; z < rows; ++z) {
      const int64_t row = off + z * Lx;
      const int64_t up = off + (z + 1 == Lm ? 0 : z + 1) * Lx, dn = off + (z == 0 ? Lm - 1 : z - 1) * Lx;
      for (int64_t x = 0; x < Lx; ++x) {
        const int64_t r = row + x, e0 = entry(r);
        const int64_t xp = row + (x + 1 == Lx ? 0 : x + 1), xm = row + (x == 0 ? Lx - 1 : x - 1);
        for (int j = 0, w = width(r); j < w; ++j) {
          const int64_t e = e0 + ((int64_t)j << ls), c = L.col[e];
          bool right = c == xp, left = c == xm;
          if (slots) {
            const int64_t want[8] = {xp, xm, up + x, dn + x, up + xp - row, up + xm - row, dn + xp - row, dn + xm - row};
            int q = 0;
            while (q < nw && want[q] != c) ++q;
            right = q == 0 || q == 4 || q == 6;
            left = q == 1 || q == 5 || q == 7;
            // the first row has to name each neighbour once, the others in its order
            const bool first = s == 0 && z == 0 && x == 0;
            if (q == nw || (first ? M->slot[q] >= 0 : M->slot[q] != j)) {
              M->pattern = MARCH_NONE;
              return false;
            }
            M->slot[q] = j;
          }
          if (!dx_ok || (same && z > 0)) continue;
          const double v = diff(e);
          if (right) {
            dx_ok = v == dxc[x];
          } else if (!left) {
            dx_ok = v == 0.0;
          } else {
            dx_ok = v == -dxc[x == 0 ? Lx - 1 : x - 1];
          }
        }
      }
    }
  }
  M->dx = M->dxcol[0];
  if (M->pattern == MARCH_BOX) {   // one value everywhere
    for (double v : M->dxcol) dx_ok = dx_ok && v == M->dx;
    M->dxcol.clear();
  }
  M->dx_ok = dx_ok ? 1 : 0;
  return true;
}

// The tiles and runs with the least estimated time: a run of zc rows (planes) takes zc + 2 T
// iterations, and an iteration costs the CU's wavefronts per SIMD and `idle` of a wavefront's
// time more per round of resident workgroups, which nothing hides (0.7 for the chain of eight
// steps, a tenth elsewhere, and at least 0.75 wavefronts' time; fitted to runs of 24 to 100 rows of 64 and 128 cells on 2000^2
// squares and a brick lattice, where it picks runs within 8 % of the best measured); a barrier
// between two wavefronts costs a twentieth.  A box,
// whose workgroups fill a CU, runs ceil(workgroups / CUs) of them in turn, and a fifth more for
// every time its planes are read (margins and cut lines).
bool plan_march(const MarchLattice& M, const std::vector<int64_t>& seg_off, int T, int B, int max_items, int cus,
                const std::vector<int>& lane_choices, int max_tile_x, MarchPlan* out) {
  const int n_seg = (int)seg_off.size() - 1;
  const bool box = M.pattern == MARCH_BOX;
  double best = 0.0;
  const double idle = T >= 8 ? 0.7 : 0.1;
  out->T = 0;
  auto ceil_div = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
  // tiles of one segment: as equal as the counts allow
  auto consider = [&](int lanes, const std::vector<MarchSeg>& tiles, int zmax) {
    int64_t last = -1;
    for (int64_t nz = 1; nz <= zmax; nz = nz < 64 ? nz + 1 : nz + nz / 16) {
      const int64_t zt = ceil_div(zmax, nz);
      if (zt == last) continue;
      last = zt;
      int64_t items = 0;
      int zc = 0;
      for (const MarchSeg& t : tiles) {
        const int64_t runs = ceil_div(t.Lm, std::min<int64_t>(zt, t.Lm));
        const int64_t z = ceil_div(t.Lm, runs);
        items += (int64_t)t.nx * t.ny * ceil_div(t.Lm, z);
        zc = std::max(zc, (int)z);
      }
      if (items > max_items) break;
      const int64_t per_cu = ceil_div(items * B, cus);
      // wavefronts per SIMD: of the fullest CU, and (several workgroups to a CU) of the average one
      const double waves = (box ? (double)per_cu : 0.5 * (per_cu + (double)(items * B) / cus)) * lanes / 256.0;
      const double rounds = (double)ceil_div(per_cu, box ? 1 : 512 / lanes);   // of resident workgroups
      // elements read per element: margins, and lines of 8 elements that a tile's rows cut
      double moved = 0.0, rows = 0.0;
      for (const MarchSeg& t : tiles) {
        moved += (double)t.nx * t.ny * (t.tx + 7) * t.ty * (t.Lm + 2.0 * T * ceil_div(t.Lm, std::min<int64_t>(zc, t.Lm)));
        rows += (double)t.Lx * t.Ly * t.Lm;
      }
      const double t = (ceil_div(zc + 2 * T, 3) * 3) * (std::max(waves, 0.75) + idle * rounds) *
                       (1.0 + (box ? 0.2 * moved / rows : lanes > 64 ? 0.05 : 0.0));
      if (best == 0.0 || t < best) {
        best = t;
        out->T = T;
        out->lanes = lanes;
        out->items = (int32_t)items;
        out->segs = tiles;
        int32_t first = 0;
        out->item0.assign(1, 0);
        for (MarchSeg& q : out->segs) {
          const int64_t runs = ceil_div(q.Lm, std::min<int64_t>(zt, q.Lm));
          q.zc = (int32_t)ceil_div(q.Lm, runs);
          q.item0 = first;
          first += (int32_t)(q.nx * q.ny * ceil_div(q.Lm, q.zc));
          out->item0.push_back(first);
        }
      }
    }
  };
  for (int lanes : lane_choices) {
    int zmax = 0;
    std::vector<MarchSeg> tiles(n_seg);
    for (int s = 0; s < n_seg; ++s) {
      MarchSeg& t = tiles[s];
      t = MarchSeg();
      t.off = seg_off[s];
      t.Lx = M.dims[3 * s];
      t.Ly = M.dims[3 * s + 1];
      t.Lm = M.dims[3 * s + 2];
      t.ny = t.ty = t.uy = 1;
      t.dx0 = s == 0 ? 0 : tiles[s - 1].dx0 + tiles[s - 1].Lx;
      zmax = std::max(zmax, t.Lm);
      if (!box) {
        const int u = lanes - 2 * T;
        t.nx = (int32_t)ceil_div(t.Lx, u);
        t.ux = (int32_t)ceil_div(t.Lx, t.nx);
        t.nx = (int32_t)ceil_div(t.Lx, t.ux);
        t.tx = t.ux + 2 * T;
      }
    }
    if (!box) {
      consider(lanes, tiles, zmax);
      continue;
    }
    // a box: every split of the plane whose tile (with its margins) has at most `lanes` cells
    MarchSeg& t = tiles[0];
    for (int nx = 1; nx <= t.Lx; ++nx) {
      const int ux = (int)ceil_div(t.Lx, nx);
      if (ux + 2 * T > max_tile_x) continue;
      const int uy_max = lanes / (ux + 2 * T) - 2 * T;
      if (uy_max < 1) continue;
      const int ny = (int)ceil_div(t.Ly, uy_max), uy = (int)ceil_div(t.Ly, ny);
      t.ux = ux;
      t.uy = uy;
      t.nx = (int32_t)ceil_div(t.Lx, ux);
      t.ny = (int32_t)ceil_div(t.Ly, uy);
      t.tx = ux + 2 * T;
      t.ty = uy + 2 * T;
      consider(lanes, tiles, zmax);
      if (ux <= 4) break;
    }
  }
  return out->T > 0;
}

// A CU holds one workgroup of 640 or 1024 cells at a time, so a launch costs rounds of
// workgroups.  Chains: 24 steps.  In two dimensions eight steps where one round does (64^2, us a step
// of one / two chains with dots in 640 cells 1.06 / 1.48, in 1024 1.28 / 1.95; 256^2 in 1024 cells 1.38 / 2.03 against
// 2.00 / 2.69 with four steps), else four, whose smaller margins mean fewer patches (512^2: 3.2 / 4.9
// against 4.0 / 6.2; next-nearest neighbours 4.7 / 6.7 against 6.1 / 9.3).  Where the lattice has marches
// they are the faster beyond two rounds (two rounds, 512^2: patches 3.2 / 4.9 and with sums 3.1 / 5.2, marches
// 3.3 / 4.8 and 3.9 / 6.1; four, 512^2 and two vectors: 5.6 / 8.9 and 4.9 / 9.5 against 4.3 / 5.8 and 5.5 / 9.4).
// Measured on squares with one hopping, which brick lattices and hoppings per entry follow: none of their patches
// measured was slower than the general kernels.  Next-nearest neighbours have no marches (four steps a
// launch against single ones, 1000^2: 14.4 / 21 against 22 / 33, with sums 12.5 / 20 against 28 / 45).
bool plan_patch(const MarchLattice& M, const std::vector<int64_t>& seg_off, int family, int B, int max_items, int cus,
                MarchPlan* out) {
  const int n_seg = (int)seg_off.size() - 1;
  const int chains = family == MF_SYM || family == MF_EVO ? 1 : 2;
  auto ceil_div = [](auto a, auto b) { return (a + b - 1) / b; };
  const int64_t n = seg_off[n_seg];
  // segment s in tiles of at most tx x ty cells with margins of T, several to a work item where a
  // tile each would be more items than a workspace has partial sums for
  auto cut = [&](int s, int T, int tx, int ty, MarchSeg* q) {
    q->off = seg_off[s];
    q->Lx = M.dims[3 * s];
    q->Ly = 1;
    q->Lm = M.dims[3 * s + 2];
    q->nx = (int32_t)ceil_div(q->Lx, tx - 2 * T);
    q->ux = (int32_t)ceil_div(q->Lx, q->nx);
    q->nx = (int32_t)ceil_div(q->Lx, q->ux);
    q->tx = q->ux + 2 * T;
    q->ny = (int32_t)ceil_div(q->Lm, ty == 1 ? 1 : ty - 2 * T);
    q->uy = (int32_t)ceil_div(q->Lm, q->ny);
    q->ny = (int32_t)ceil_div(q->Lm, q->uy);
    q->ty = ty == 1 ? 1 : q->uy + 2 * T;
    const int64_t tiles = (int64_t)q->nx * q->ny;
    const int64_t room = std::max<int64_t>(1, max_items * (seg_off[s + 1] - seg_off[s]) / n);
    q->zc = tiles <= room ? 1 : (int32_t)ceil_div(tiles, room);
    return tiles <= room ? tiles : ceil_div(tiles, (int64_t)q->zc);
  };
  int bT = 0, blanes = 0, btx = 0, bty = 0;
  int64_t brounds = 0, bitems = 0;
  auto consider = [&](int T, int lanes, int tx, int ty) {
    int64_t items = 0, per = 1;
    MarchSeg q = MarchSeg();
    for (int s = 0; s < n_seg; ++s) {
      items += cut(s, T, tx, ty, &q);
      per = std::max<int64_t>(per, q.zc);
      if (items > max_items) return;
    }
    const int64_t rounds = per * ceil_div(items * B, (int64_t)cus);
    // among equals the narrowest for one round (64^2: 4 x 16 owned cells 1.06 us a step, 6 x 13 cells 1.18), the fewest for more
    if (bT > 0 && (rounds > brounds || (rounds == brounds && (rounds == 1 || items >= bitems)))) return;
    bT = T;
    blanes = lanes;
    btx = tx;
    bty = ty;
    brounds = rounds;
    bitems = items;
  };
  if (M.pattern == MARCH_CHAIN) {
    consider(24, 256, 256 * (chains == 1 ? 4 : 2), 1);
  } else if (M.pattern != MARCH_BOX) {
    const int shapes[3][2] = {{8, 640}, {8, 1024}, {4, 1024}};
    for (const auto& sh : shapes) {
      if (bT > 0 && brounds == 1) break;
      bT = 0;
      for (int tx = 2 * sh[0] + 2; tx <= 64; tx += 2)
        if (sh[1] / tx > 2 * sh[0]) consider(sh[0], sh[1], tx, sh[1] / tx);
    }
    if (out->T > 0 && brounds > 2) return false;
  }
  if (bT == 0) return false;
  *out = MarchPlan();
  out->T = bT;
  out->patch = 1;
  out->lanes = blanes;
  out->item0.assign(1, 0);
  int32_t dx0 = 0;
  for (int s = 0; s < n_seg; ++s) {
    MarchSeg q = MarchSeg();
    q.item0 = out->items;
    out->items += (int32_t)cut(s, bT, btx, bty, &q);
    q.dx0 = dx0;
    dx0 += q.Lx;
    out->segs.push_back(q);
    out->item0.push_back(out->items);
  }
  return true;
}

// Estimates, from per-step times (events around 64 steps) of every family by marches or patches and by the general
// kernels: 901 pairs of lattice and block width on one MI355X (boxes of 125 to 4 M sites; squares, open squares,
// brick lattices and squares with next-nearest neighbours of 64 to 1.6 M sites, any shape down to strips of four columns;
// rings; one hopping and one an entry; B = 1, 2, 4, 16), 378 of them on tuned handles too.  A launch costs a constant and a
// time per iteration of a round of workgroups, less where few of a tile's lanes have work of their own, and its
// traffic.  Boxes come out within 9 %, r.m.s., the others within 7 to 17 %.
//
// Marches are slower by 5 % or more in 601 of 4,505 places (454 of 1,890 against tuned kernels), up to 19 times: small
// boxes, whose launch takes 14 us or more for three steps of 3.5 us (20^3, one vector: Hermitian step 4.65 us
// against 3.56 general, MSD term 10.8 against 3.6, two chains 15.3 against 3.8; 60^3: 5.6 / 6.1, 13.3 / 10.9 and
// 17.9 / 7.2), and strips, whose tiles own few of their cells (5 x 5 x 20,000, four vectors: 93 against
// 25; squares of 4 x 200,000, four vectors: 42 against 33).  By these estimates the slower one is taken in 101 (61) places,
// by 20 % or more in 48 (18).
double plan_launch_us(const MarchLattice& M, int hop_mode, int family, int B, int cus, const MarchPlan& p) {
  auto ceil_div = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
  const bool one = family == MF_SYM || family == MF_EVO, entry = hop_mode != HOP_UNIFORM;
  const int64_t per_cu = ceil_div((int64_t)p.items * B, cus);
  int zc = 0;
  double rows = 0.0, fill = 0.0;   // elements; the tiles' share of a workgroup's lanes
  for (const MarchSeg& q : p.segs) {
    zc = std::max(zc, (int)q.zc);
    const double r = (double)q.Lx * q.Ly * q.Lm * B;
    fill += r * (M.pattern == MARCH_BOX ? q.tx * q.ty : q.ux) / p.lanes;
    rows += r;
  }
  fill /= rows;
  if (p.patch) {
    if (M.pattern == MARCH_CHAIN) return 8.7 + (entry ? 9.0 : 7.0) * zc * per_cu;
    const double full = (one ? 4.5 : 6.6) * (entry ? 1.15 : 1.0) * (M.pattern == MARCH_NNN ? 1.5 : 1.0);
    return kPatchFixedUs + full * (p.T == 8 && p.lanes == 1024 ? 1.5 : 1.0) * zc * per_cu;
  }
  // constant; time of an iteration; bytes per us; share of the iteration that does not shrink with the fill
  struct Cost { double fixed, iter, rate, base; };
  static const Cost cost[3][kMarchFamilies] = {   // SYM, PAIR, EVO, EVO2, MSD
      {{5.9, 1.05, 7.1e6, 0.80}, {14.9, 3.39, 4.3e6, 0.66}, {5.3, 1.22, 6.3e6, 0.78}, {5.8, 2.70, 5.8e6, 0.80}, {4.6, 3.52, 5.1e6, 0.74}},   // box
      {{13.6, 0.34, 9.1e6, 0.89}, {6.4, 0.96, 8.1e6, 0.82}, {7.2, 0.28, 6.7e6, 1.0}, {9.3, 0.48, 6.2e6, 1.0}, {10.2, 0.51, 6.1e6, 1.0}},    // one hopping
      {{7.4, 0.63, 12.0e6, 0.68}, {3.7, 1.13, 9.7e6, 0.64}, {6.4, 0.49, 7.5e6, 0.80}, {3.9, 1.15, 7.9e6, 0.50}, {4.4, 1.19, 8.0e6, 0.53}},  // one an entry
  };
  const Cost& c = cost[M.pattern == MARCH_BOX ? 0 : entry ? 2 : 1][family];
  double w = (double)ceil_div(zc + 2 * p.T, 3) * 3;
  double bytes = 16.0 * rows * (one ? 1 : 2) * (family == MF_SYM || family == MF_PAIR ? 4 : 6);   // two elements in and out a chain, and sums
  if (M.pattern == MARCH_BOX) {
    w *= per_cu;
    bytes *= 1.24;   // (margins)
  } else {
    const double waves = 0.5 * (per_cu + (double)p.items * B / cus) * p.lanes / 256.0;   // as in plan_march
    const double rounds = (double)ceil_div(per_cu, 512 / p.lanes);
    w *= (std::max(waves, 0.75) + (p.T >= 8 ? 0.7 : 0.1) * rounds) * (p.lanes > 64 ? 1.05 : 1.0);
    const double hop[4] = {0, 8, 16, 2};
    bytes = 1.15 * bytes + hop[hop_mode] * rows * (M.pattern == MARCH_BRICK ? 3 : 4);
  }
  return std::hypot(c.fixed + c.iter * w * (c.base + (1.0 - c.base) * fill), bytes / c.rate);
}

// A step is a launch, at least, and 0.75 of that and its bytes at 5.2 TB/s (the measured steps lie within 15 %, r.m.s.);
// with the row order and caps that the autotuner chooses 6.7, while the step's bytes fit the last-level cache; the
// gathers of eight neighbours take longer than the bytes.
double general_step_us(int family, int hop_mode, int64_t n, int64_t nnz, int B, bool tuned) {
  static const double floor_us[kMarchFamilies] = {3.7, 3.7, 2.9, 3.1, 3.3}, vec[kMarchFamilies] = {48, 96, 80, 160, 160};
  const double key[4] = {4, 12, 20, 2};   // bytes of an entry: column and hopping, or a table index
  const double entry = key[hop_mode] + (family == MF_MSD && hop_mode != HOP_DICT ? 8.0 : 0.0);
  const double bytes = (double)n * (vec[family] * B + 8.0) + entry * (double)nnz;
  const double gather = nnz < 8 * n ? 1.0 : family == MF_SYM || family == MF_PAIR ? 1.4 : 1.25;
  return gather * std::max(floor_us[family] + 0.2 * (B - 1),
                           0.75 * floor_us[family] + bytes / (tuned && bytes < 380e6 ? 6.7e6 : 5.2e6));
}

double planar_us(int64_t n, int B) { return B == 1 ? 0.0 : 2.2 + 32.0 * (double)n * B / 5.5e6; }

}  // namespace gpuqt
