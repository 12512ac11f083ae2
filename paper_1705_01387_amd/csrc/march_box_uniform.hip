// March kernels of the box pattern, one hopping per segment.
#include "march_core.h"

namespace gpuqt {
namespace march {

hipError_t launch_box_uniform(int family, int lanes, const MarchMat& A, const MarchIO& io, hipStream_t s) {
  return launch_pattern<MARCH_BOX, HOP_UNIFORM>(family, lanes, A, io, s);
}

}  // namespace march
}  // namespace gpuqt
