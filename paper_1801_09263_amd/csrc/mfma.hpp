// mfma.hpp - the FP64 matrix-core instruction of the dense kernels.
//
// v_mfma_f64_16x16x4_f64: per wave D(16x16) += A(16x4) B(4x16), where lane
// l supplies A[l % 16][l / 16] and B[l / 16][l % 16] and holds
// D[l / 16 + 4 e][l % 16] in accumulator element e (rows interleaved; the
// layout was confirmed with a one-wave probe on gfx950).
#pragma once
#include <hip/hip_runtime.h>

namespace lace {

typedef double d4 __attribute__((ext_vector_type(4)));

__device__ inline d4 mfma(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

}  // namespace lace
