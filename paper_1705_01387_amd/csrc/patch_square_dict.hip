// Patch kernels of the square pattern, a table index per entry.
#include "patch_core.h"

namespace gpuqt {
namespace march {

hipError_t patch_square_dict(int family, int lanes, const MarchMat& A, const MarchIO& io, hipStream_t s) {
  return launch_patch_pattern<MARCH_SQUARE, HOP_DICT>(family, lanes, A, io, s);
}

}  // namespace march
}  // namespace gpuqt
