// Dispatch of the march kernels (march_core.h; one file per pattern and hopping
// storage, so that they compile in parallel) and the change of layout between
// blocks of vectors [n][B] and planar vectors [B][n].
#include <hip/hip_runtime.h>

#include "internal.h"
#include "march.h"
#include "march_core.h"

namespace gpuqt {
namespace march {
hipError_t launch_square_uniform(int family, int lanes, const MarchMat& A, const MarchIO& io, hipStream_t s);
hipError_t launch_square_real(int family, int lanes, const MarchMat& A, const MarchIO& io, hipStream_t s);
hipError_t launch_square_complex(int family, int lanes, const MarchMat& A, const MarchIO& io, hipStream_t s);
hipError_t launch_square_dict(int family, int lanes, const MarchMat& A, const MarchIO& io, hipStream_t s);
hipError_t launch_brick_uniform(int family, int lanes, const MarchMat& A, const MarchIO& io, hipStream_t s);
hipError_t launch_brick_real(int family, int lanes, const MarchMat& A, const MarchIO& io, hipStream_t s);
hipError_t launch_brick_complex(int family, int lanes, const MarchMat& A, const MarchIO& io, hipStream_t s);
hipError_t launch_brick_dict(int family, int lanes, const MarchMat& A, const MarchIO& io, hipStream_t s);
hipError_t launch_box_uniform(int family, int lanes, const MarchMat& A, const MarchIO& io, hipStream_t s);
hipError_t patch_square_uniform(int family, int lanes, const MarchMat& A, const MarchIO& io, hipStream_t s);
hipError_t patch_square_real(int family, int lanes, const MarchMat& A, const MarchIO& io, hipStream_t s);
hipError_t patch_square_complex(int family, int lanes, const MarchMat& A, const MarchIO& io, hipStream_t s);
hipError_t patch_square_dict(int family, int lanes, const MarchMat& A, const MarchIO& io, hipStream_t s);
hipError_t patch_brick_uniform(int family, int lanes, const MarchMat& A, const MarchIO& io, hipStream_t s);
hipError_t patch_brick_real(int family, int lanes, const MarchMat& A, const MarchIO& io, hipStream_t s);
hipError_t patch_brick_complex(int family, int lanes, const MarchMat& A, const MarchIO& io, hipStream_t s);
hipError_t patch_brick_dict(int family, int lanes, const MarchMat& A, const MarchIO& io, hipStream_t s);
hipError_t patch_nnn_uniform(int family, int lanes, const MarchMat& A, const MarchIO& io, hipStream_t s);
hipError_t patch_chain_uniform(int family, int lanes, const MarchMat& A, const MarchIO& io, hipStream_t s);
hipError_t patch_nnn_real(int family, int lanes, const MarchMat& A, const MarchIO& io, hipStream_t s);
hipError_t patch_chain_real(int family, int lanes, const MarchMat& A, const MarchIO& io, hipStream_t s);
hipError_t patch_nnn_complex(int family, int lanes, const MarchMat& A, const MarchIO& io, hipStream_t s);
hipError_t patch_chain_complex(int family, int lanes, const MarchMat& A, const MarchIO& io, hipStream_t s);
hipError_t patch_nnn_dict(int family, int lanes, const MarchMat& A, const MarchIO& io, hipStream_t s);
hipError_t patch_chain_dict(int family, int lanes, const MarchMat& A, const MarchIO& io, hipStream_t s);
}  // namespace march

MarchShape march_shape(int pattern, int hop_mode, int family) {
  MarchShape m;
  if (pattern == MARCH_CHAIN || pattern == MARCH_NNN) return m;   // patches only
  m.T = march::steps_of(pattern, hop_mode, family);
  m.max_tile_x = march::kMaxTileX;
  if (pattern == MARCH_BOX) m.lanes = {1024};
  else m.lanes = {64, 128};
  return m;
}

hipError_t launch_march(int pattern, int hop_mode, int family, int lanes, int patch, const MarchMat& A,
                        const MarchIO& io, hipStream_t s) {
  if (patch) {
    switch (pattern * 4 + hop_mode) {
      case MARCH_SQUARE * 4 + HOP_UNIFORM: return march::patch_square_uniform(family, lanes, A, io, s);
      case MARCH_SQUARE * 4 + HOP_REAL: return march::patch_square_real(family, lanes, A, io, s);
      case MARCH_SQUARE * 4 + HOP_COMPLEX: return march::patch_square_complex(family, lanes, A, io, s);
      case MARCH_SQUARE * 4 + HOP_DICT: return march::patch_square_dict(family, lanes, A, io, s);
      case MARCH_BRICK * 4 + HOP_UNIFORM: return march::patch_brick_uniform(family, lanes, A, io, s);
      case MARCH_BRICK * 4 + HOP_REAL: return march::patch_brick_real(family, lanes, A, io, s);
      case MARCH_BRICK * 4 + HOP_COMPLEX: return march::patch_brick_complex(family, lanes, A, io, s);
      case MARCH_BRICK * 4 + HOP_DICT: return march::patch_brick_dict(family, lanes, A, io, s);
      case MARCH_NNN * 4 + HOP_UNIFORM: return march::patch_nnn_uniform(family, lanes, A, io, s);
      case MARCH_CHAIN * 4 + HOP_UNIFORM: return march::patch_chain_uniform(family, lanes, A, io, s);
      case MARCH_NNN * 4 + HOP_REAL: return march::patch_nnn_real(family, lanes, A, io, s);
      case MARCH_CHAIN * 4 + HOP_REAL: return march::patch_chain_real(family, lanes, A, io, s);
      case MARCH_NNN * 4 + HOP_COMPLEX: return march::patch_nnn_complex(family, lanes, A, io, s);
      case MARCH_CHAIN * 4 + HOP_COMPLEX: return march::patch_chain_complex(family, lanes, A, io, s);
      case MARCH_NNN * 4 + HOP_DICT: return march::patch_nnn_dict(family, lanes, A, io, s);
      case MARCH_CHAIN * 4 + HOP_DICT: return march::patch_chain_dict(family, lanes, A, io, s);
      default: return hipErrorInvalidValue;
    }
  }
  switch (pattern * 4 + hop_mode) {
    case MARCH_SQUARE * 4 + HOP_UNIFORM: return march::launch_square_uniform(family, lanes, A, io, s);
    case MARCH_SQUARE * 4 + HOP_REAL: return march::launch_square_real(family, lanes, A, io, s);
    case MARCH_SQUARE * 4 + HOP_COMPLEX: return march::launch_square_complex(family, lanes, A, io, s);
    case MARCH_SQUARE * 4 + HOP_DICT: return march::launch_square_dict(family, lanes, A, io, s);
    case MARCH_BRICK * 4 + HOP_UNIFORM: return march::launch_brick_uniform(family, lanes, A, io, s);
    case MARCH_BRICK * 4 + HOP_REAL: return march::launch_brick_real(family, lanes, A, io, s);
    case MARCH_BRICK * 4 + HOP_COMPLEX: return march::launch_brick_complex(family, lanes, A, io, s);
    case MARCH_BRICK * 4 + HOP_DICT: return march::launch_brick_dict(family, lanes, A, io, s);
    case MARCH_BOX * 4 + HOP_UNIFORM: return march::launch_box_uniform(family, lanes, A, io, s);
    default: return hipErrorInvalidValue;
  }
}

namespace {

// One element per thread; a wavefront's 64 elements are 64 / B rows, so the planar
// side moves B runs of 1024 / B bytes.
__global__ __launch_bounds__(kBlock) void k_planar(int64_t total, int64_t n, int lB, const double2* __restrict__ rows,
                                                   double2* __restrict__ planar) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < total) planar[(i & ((1 << lB) - 1)) * n + (i >> lB)] = rows[i];
}
__global__ __launch_bounds__(kBlock) void k_rows(int64_t total, int64_t n, int lB, const double2* __restrict__ planar,
                                                 double2* __restrict__ rows) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < total) rows[i] = planar[(i & ((1 << lB) - 1)) * n + (i >> lB)];
}

}  // namespace

hipError_t launch_to_planar(int64_t n, int B, const double2* rows, double2* planar, hipStream_t s) {
  const int64_t t = n * B;
  k_planar<<<dim3((unsigned)((t + kBlock - 1) / kBlock)), kBlock, 0, s>>>(t, n, Handle::log2B(B), rows, planar);
  return hipGetLastError();
}

hipError_t launch_from_planar(int64_t n, int B, const double2* planar, double2* rows, hipStream_t s) {
  const int64_t t = n * B;
  k_rows<<<dim3((unsigned)((t + kBlock - 1) / kBlock)), kBlock, 0, s>>>(t, n, Handle::log2B(B), planar, rows);
  return hipGetLastError();
}

}  // namespace gpuqt
