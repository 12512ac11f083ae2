// What the reverse steps share (kernels_adjoint.hip, and the two-chain and Hermitian forms in files of their own, so
// that they compile in parallel).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>

#include "device_common.h"

namespace gpuqt {
namespace dev {

// f(j) for the entries of a row: K of them unrolled, so that every index, table and gather load is in
// flight at once instead of one entry's chain after another's, or w.
template <int K, typename F>
__device__ __forceinline__ void for_entries(int w, F&& f) {
  if constexpr (K > 0) {
#pragma unroll
    for (int j = 0; j < K; ++j) f(j);
  } else {
    for (int j = 0; j < w; ++j) f(j);
  }
}

// f(B, HOP, K, NC, TR) of a reverse step with nc class sums.  (One hopping per segment: one class.)
template <typename F>
inline hipError_t dispatch_reverse(const DevMat& A, int hop_mode, int B, int nc, bool tr, F&& f) {
  if (hop_mode == HOP_UNIFORM && nc > 1) return hipErrorInvalidValue;
  return dispatch_bh(B, hop_mode, [&](auto Bc, auto Hc) {
    constexpr int Hv = decltype(Hc)::value;
    auto with = [&](auto Kc) {
      auto classes = [&](auto Nc) {
        if constexpr (Hv != HOP_UNIFORM || decltype(Nc)::value <= 1) {
          if (tr) f(Bc, Hc, Kc, Nc, IC<1>{});
          else f(Bc, Hc, Kc, Nc, IC<0>{});
        }
      };
      switch (nc) {
        case 0: f(Bc, Hc, Kc, IC<0>{}, IC<0>{}); break;
        case 1: classes(IC<1>{}); break;
        case 2: classes(IC<2>{}); break;
        default: classes(IC<4>{}); break;
      }
    };
    switch (A.K) {
      case 3: with(IC<3>{}); break;
      case 4: with(IC<4>{}); break;
      case 6: with(IC<6>{}); break;
      case 8: with(IC<8>{}); break;
      default: with(IC<0>{}); break;
    }
  });
}

}  // namespace dev
}  // namespace gpuqt
