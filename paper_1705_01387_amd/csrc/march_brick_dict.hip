// March kernels of the brick-wall (honeycomb) pattern, a table index per entry.
#include "march_core.h"

namespace gpuqt {
namespace march {

hipError_t launch_brick_dict(int family, int lanes, const MarchMat& A, const MarchIO& io, hipStream_t s) {
  return launch_pattern<MARCH_BRICK, HOP_DICT>(family, lanes, A, io, s);
}

}  // namespace march
}  // namespace gpuqt
