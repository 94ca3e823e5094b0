// Operands of the FP64 matrix instruction (v_mfma_f64_16x16x4f64) on gfx950:
//   lane l supplies A[l%16][l/16] and B[l/16][l%16];
//   accumulator register r of lane l is D[l/16 + 4r][l%16] (checked on the device),
// so register r of a product's accumulator is the B operand of k = 4r .. 4r + 3.
#pragma once

#include <hip/hip_runtime.h>

namespace dfjk {

typedef double f64x4 __attribute__((ext_vector_type(4)));

}  // namespace dfjk
