// March kernels of the square pattern, a real hopping per entry.
#include "march_core.h"

namespace gpuqt {
namespace march {

hipError_t launch_square_real(int family, int lanes, const MarchMat& A, const MarchIO& io, hipStream_t s) {
  return launch_pattern<MARCH_SQUARE, HOP_REAL>(family, lanes, A, io, s);
}

}  // namespace march
}  // namespace gpuqt
