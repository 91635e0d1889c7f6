// GEMM kernels for fp16 operands: the register-staged configurations (see gemm_kernels.h).
#define MPX_GEMM_STAGED_SOURCE
#include "gemm_kernels.h"

namespace mpx {

MPX_GEMM_STAGED(, MPX_F16)

}  // namespace mpx
