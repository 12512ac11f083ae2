// Patch kernels of the brick-wall (honeycomb) pattern, a complex hopping per entry.
#include "patch_core.h"

namespace gpuqt {
namespace march {

hipError_t patch_brick_complex(int family, int lanes, const MarchMat& A, const MarchIO& io, hipStream_t s) {
  return launch_patch_pattern<MARCH_BRICK, HOP_COMPLEX>(family, lanes, A, io, s);
}

}  // namespace march
}  // namespace gpuqt
