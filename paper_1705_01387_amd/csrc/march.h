// Lattice marches: several Chebyshev steps per launch on lattices whose rows have
// a fixed neighbour pattern (march_core.h has the marches' kernel, patch_core.h that of
// chains and small lattices; lattice.cpp recognises the lattices and cuts them into tiles).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

#include "../../include/gpuqt.h"

namespace gpuqt {

// Neighbour patterns.  Rows are (x, y[, z]) in natural order, periodic in every
// direction (SQUARE with one hopping: or open in x).  The slots of a row, in the order the kernels name them:
//   SQUARE  +x, -x, +y, -y                 (segments may be squares of any sizes)
//   BRICK   +x, -x, +y where x + y + parity is even, else -y   (honeycomb)
//   BOX     +x, -x, +y, -y, +z, -z         (one hopping)
//   CHAIN   +x, -x
//   NNN     +x, -x, +y, -y, +x+y, -x+y, +x-y, -x-y   (squares of any sizes)
enum MarchPattern { MARCH_NONE = 0, MARCH_SQUARE = 1, MARCH_BRICK = 2, MARCH_BOX = 3, MARCH_CHAIN = 4, MARCH_NNN = 5 };

// Families of the marches: one chain with its moment dots, two chains with
// theirs, one and two chains with their running sums (evolution), and the
// coupled chains of the evolution + commutator series.
enum MarchFamily { MF_SYM = 0, MF_PAIR = 1, MF_EVO = 2, MF_EVO2 = 3, MF_MSD = 4, kMarchFamilies = 5 };

constexpr int kMarchMaxSteps = 24;
constexpr int kPatchUnroll = 4;

// One segment's tiles.  The march runs along the slowest direction (Lm rows or
// planes); a workgroup holds tx x ty cells of the other directions (ty = 1 in two
// dimensions), the inner ux x uy of which it owns, for zc rows (planes).  Its work
// items are numbered x tile fastest, then y tile, then run, from item0.
struct MarchSeg {
  int64_t off;              // first row
  int32_t Lx, Ly, Lm;       // Ly = 1 in two dimensions
  int32_t tx, ty, ux, uy;   // cells of a tile and how many of them it owns
  int32_t nx, ny, zc;       // tiles in x and y; rows (planes) per run, or (patches) tiles per work item
  int32_t item0;            // first work item of the segment
  int32_t dx0;              // first column of the segment in dxcol (two dimensions)
};

// A launch plan of one family and block width: T steps per launch.
struct MarchPlan {
  int32_t T = 0;            // 0: no march for this family
  int32_t patch = 0;        // 1: patches (patch_core.h), 0: marches
  int32_t lanes = 0;        // threads per workgroup
  int32_t items = 0;        // work items of one vector; a launch has items x B workgroups
  double launch_us = 0.0;   // estimated time of a launch of T steps (plan_launch_us)
  std::vector<MarchSeg> segs;
  std::vector<int32_t> item0;   // [n_seg + 1] first item of each segment
};

// The lattice of a handle.
struct MarchLattice {
  int32_t pattern = MARCH_NONE;
  int32_t parity = 0;           // BRICK
  int32_t open = 0;             // 1: no bonds between the columns Lx - 1 and 0 (SQUARE, one hopping)
  int32_t slot[8] = {-1, -1, -1, -1, -1, -1, -1, -1};   // stored slot of each neighbour above (-1: not looked at)
  // position differences: that of the +x neighbour of each column (dxcol, [sum of the Lx], the
  // -x neighbour of the next column having its negative), the same on every row of a
  // segment, 0 for the other neighbours; in a box one value, dx
  std::vector<double> dxcol;
  double dx = 0.0;
  int32_t dx_ok = 0;
  std::vector<int32_t> dims;    // [3 n_seg] Lx, Ly, Lm
};

// What a march kernel reads of the Hamiltonian.
struct MarchMat {
  const MarchSeg* segs;
  int32_t n_seg, items, B;
  int32_t T;                    // steps per launch (patches)
  int32_t parity, open;
  int64_t n;                    // rows of all segments: the stride between two vectors
  const double* diag;
  const double* seg_hop;        // uniform hopping per segment
  const double* hop;            // per entry, real or complex
  const uint16_t* hidx;         // table index per entry
  const double2* htab;
  int32_t S_log2;
  int32_t slot[8];
  double dx;                    // BOX
  const double* dxcol;          // two dimensions
};

// One launch: steps k0 .. k0 + T - 1 of the recurrence, from the chain elements
// x = v_{k0 - 1} and w = v_{k0 - 2} (w unused when first: k0 = 1) to o1 = v_{k0 + T - 2}
// and o2 = v_{k0 + T - 1}.  Vectors are planar: column c of a block at c * n.
struct MarchIO {
  const double2* x[2];
  const double2* w[2];
  double2* o1[2];
  double2* o2[2];
  const double2* acc_in[2];     // running sums (evolution families)
  double2* acc_out[2];
  int32_t first, k0, k_end;     // steps past k_end leave no dots and no sums
  int32_t steps;                // patches: steps of this launch, a multiple of kPatchUnroll (<= T)
  int32_t zero_b;               // first launch: chain b starts from zero (xb not read)
  double2* part;                // dots: [row][items][B], rows 2k - 1 and 2k of step k (row 0 on the first)
  int32_t keep;                 // 1: every step's elements go to keep[chain][step - k0] (NULL: dropped)
                                // instead of o1 and o2, and all vectors are rows of B columns, [n][B]
  double2* keepv[2][kMarchMaxSteps];
  const double* J;              // sums: c_m = J[seg * ldJ + m] (-i sgn)^m
  int32_t ldJ;
  double sgn;
};

// lattice.cpp.  The lattice of a layout whose hoppings and neighbours allow a march:
// box = detect_box's dims (0: none), sheets = detect_sheets' (Lx, Ly) per segment (empty:
// none; with per-entry hoppings the neighbours' slots must be the same on every row);
// otherwise the BRICK pattern is looked for.
struct HostLayout;
bool detect_lattice(const gpuqt_h_desc* d, const HostLayout& L, const int32_t box[3],
                    const std::vector<int32_t>& sheets, MarchLattice* M);

// Tiles for T steps per launch of blocks of B vectors on `cus` compute units, at most
// max_items work items (the partial sums of a workspace), workgroups of one of
// lane_choices threads.  False when none fits.
bool plan_march(const MarchLattice& M, const std::vector<int64_t>& seg_off, int T, int B, int max_items, int cus,
                const std::vector<int>& lane_choices, int max_tile_x, MarchPlan* out);

// What a family's kernel is built for (0 steps: no march): steps per launch, and the
// workgroup sizes.
struct MarchShape {
  int T = 0;
  std::vector<int> lanes;
  int max_tile_x = 0;
};
MarchShape march_shape(int pattern, int hop_mode, int family);
hipError_t launch_march(int pattern, int hop_mode, int family, int lanes, int patch, const MarchMat& A,
                        const MarchIO& io, hipStream_t s);
// Patches instead of marches where they take less time (plan_march's answer in *out, or none), for
// two-dimensional patterns; chains and NNN have no marches.
bool plan_patch(const MarchLattice& M, const std::vector<int64_t>& seg_off, int family, int B, int max_items, int cus,
                MarchPlan* out);
// Estimated times (microseconds): a launch of the plan's T steps, a single step of a family by the general
// kernels (nnz: stored entries; tuned: with the autotuner's row order and caps), and the change of layout of a block of vectors.
double plan_launch_us(const MarchLattice& M, int hop_mode, int family, int B, int cus, const MarchPlan& p);
double general_step_us(int family, int hop_mode, int64_t n, int64_t nnz, int B, bool tuned);
double planar_us(int64_t n, int B);
constexpr double kPatchFixedUs = 2.3;   // of a patch launch's time, what does not shrink with its steps
// planar[c * n + r] = rows[r * B + c], and back
hipError_t launch_to_planar(int64_t n, int B, const double2* rows, double2* planar, hipStream_t s);
hipError_t launch_from_planar(int64_t n, int B, const double2* planar, double2* rows, hipStream_t s);

}  // namespace gpuqt
