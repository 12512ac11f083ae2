// Patch kernels of chains.
#include "patch_core.h"

namespace gpuqt {
namespace march {

hipError_t patch_chain_uniform(int family, int lanes, const MarchMat& A, const MarchIO& io, hipStream_t s) {
  return launch_patch_pattern<MARCH_CHAIN, HOP_UNIFORM>(family, lanes, A, io, s);
}

hipError_t patch_chain_real(int family, int lanes, const MarchMat& A, const MarchIO& io, hipStream_t s) {
  return launch_patch_pattern<MARCH_CHAIN, HOP_REAL>(family, lanes, A, io, s);
}

hipError_t patch_chain_complex(int family, int lanes, const MarchMat& A, const MarchIO& io, hipStream_t s) {
  return launch_patch_pattern<MARCH_CHAIN, HOP_COMPLEX>(family, lanes, A, io, s);
}

hipError_t patch_chain_dict(int family, int lanes, const MarchMat& A, const MarchIO& io, hipStream_t s) {
  return launch_patch_pattern<MARCH_CHAIN, HOP_DICT>(family, lanes, A, io, s);
}

}  // namespace march
}  // namespace gpuqt
