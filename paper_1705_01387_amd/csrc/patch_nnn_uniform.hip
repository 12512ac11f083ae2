// Patch kernels of the square pattern with next-nearest neighbours, one hopping per segment.
#include "patch_core.h"

namespace gpuqt {
namespace march {

hipError_t patch_nnn_uniform(int family, int lanes, const MarchMat& A, const MarchIO& io, hipStream_t s) {
  return launch_patch_pattern<MARCH_NNN, HOP_UNIFORM>(family, lanes, A, io, s);
}

}  // namespace march
}  // namespace gpuqt
