// Host build of the lattice recognition and of the launch plans for the CPU tests: what a recognised pattern
// says the matrix is, against the layout that the general kernels read.
#include <complex>
#include <cstring>
#include <map>

#include "../paper_1705_01387_amd/csrc/internal.h"
#include "../paper_1705_01387_amd/csrc/march.h"

using namespace gpuqt;

extern "C" {

// The recognised pattern of a descriptor (0: none), + 100 where some row of the pattern's matrix is not
// the layout's, -1 for a refused descriptor.  hop_mode (may be NULL) receives the storage mode.
int lattice_check(int64_t n, int max_nn, const int32_t* nn, const int32_t* nbr, const double* hop, int cplx,
                  const double* x, double length_x, int n_seg, const int64_t* seg_off, int no_dictionary,
                  int check_hermitian, int32_t* hop_mode) {
  gpuqt_h_desc d;
  std::memset(&d, 0, sizeof(d));
  d.n = n;
  d.max_nn = max_nn;
  d.nn = nn;
  d.nbr = nbr;
  d.hop = hop;
  d.hop_is_complex = cplx;
  d.x = x;
  d.length_x = length_x;
  d.n_segments = n_seg;
  d.seg_offsets = seg_off;
  d.no_dictionary = no_dictionary;
  d.check_hermitian = check_hermitian;
  HostLayout L;
  std::string msg;
  if (build_host_layout(&d, &L, &msg) != GPUQT_OK) return -1;
  if (hop_mode) *hop_mode = L.hop_mode;
  int32_t box[3] = {0, 0, 0};
  if (L.hop_mode == HOP_UNIFORM && L.n_seg == 1 && L.uniform_width == 6) (void)detect_box(&d, box);
  std::vector<int32_t> sheets;
  if (box[0] == 0 && L.uniform_width == 4) (void)detect_sheets(&d, L.seg_off, &sheets);
  MarchLattice M;
  if (!detect_lattice(&d, L, box, sheets, &M)) return 0;
  const int K = M.pattern == MARCH_CHAIN ? 2 : M.pattern == MARCH_BRICK ? 3 : M.pattern == MARCH_BOX ? 6 : M.pattern == MARCH_NNN ? 8 : 4;
  auto value = [&](int64_t e, int seg) -> std::complex<double> {
    switch (L.hop_mode) {
      case HOP_UNIFORM: return L.seg_hop[seg];
      case HOP_REAL: return L.hop[e];
      case HOP_COMPLEX: return {L.hop[2 * e], L.hop[2 * e + 1]};
      default: return {L.htab[2 * L.hidx[e]], L.htab[2 * L.hidx[e] + 1]};
    }
  };
  for (int s = 0; s < L.n_seg; ++s) {
    const int64_t off = L.seg_off[s], Lx = M.dims[3 * s], Ly = M.dims[3 * s + 1], Lm = M.dims[3 * s + 2];
    if (off + Lx * Ly * Lm != L.seg_off[s + 1]) return 100 + M.pattern;
    for (int64_t r = off; r < L.seg_off[s + 1]; ++r) {
      std::map<int64_t, std::complex<double>> want, got;
      const int64_t sl = r >> L.S_log2, p0 = L.slice_ptr[sl], w = (L.slice_ptr[sl + 1] - p0) >> L.S_log2;
      const int64_t e0 = p0 + (r & (L.S - 1));
      for (int64_t j = 0; j < w; ++j)
        if (L.col[e0 + j * L.S] >= 0) want[L.col[e0 + j * L.S]] += value(e0 + j * L.S, s);
      const int64_t X = (r - off) % Lx, Y = (r - off) / Lx % Ly, Z = (r - off) / (Lx * Ly);
      auto at = [&](int64_t a, int64_t b, int64_t c) {
        return off + (a + Lx) % Lx + Lx * ((b + Ly) % Ly + Ly * ((c + Lm) % Lm));
      };
      int64_t q[8];
      q[0] = at(X + 1, Y, Z);
      q[1] = at(X - 1, Y, Z);
      if (M.pattern == MARCH_BOX) {
        q[2] = at(X, Y + 1, Z);
        q[3] = at(X, Y - 1, Z);
        q[4] = at(X, Y, Z + 1);
        q[5] = at(X, Y, Z - 1);
      } else if (M.pattern == MARCH_BRICK) {
        q[2] = at(X, 0, ((X + Z + M.parity) & 1) == 0 ? Z + 1 : Z - 1);
      } else {
        q[2] = at(X, 0, Z + 1);
        q[3] = at(X, 0, Z - 1);
        q[4] = at(X + 1, 0, Z + 1);
        q[5] = at(X - 1, 0, Z + 1);
        q[6] = at(X + 1, 0, Z - 1);
        q[7] = at(X - 1, 0, Z - 1);
      }
      for (int j = 0; j < K; ++j) {
        if (M.open && ((j == 0 && X + 1 == Lx) || (j == 1 && X == 0))) continue;
        if (M.slot[j] < 0 && L.hop_mode != HOP_UNIFORM) return 100 + M.pattern;
        got[q[j]] += value(L.hop_mode == HOP_UNIFORM ? 0 : e0 + (int64_t)M.slot[j] * L.S, s);
      }
      if (want != got) return 100 + M.pattern;
    }
  }
  return M.pattern;
}

}  // extern "C"
