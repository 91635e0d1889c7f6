// GEMM kernels for bf16 operands: the configurations that are only forced (see gemm_kernels.h).
#define MPX_GEMM_FORCED_SOURCE
#include "gemm_kernels.h"

namespace mpx {

MPX_GEMM_FORCED(, MPX_BF16)

}  // namespace mpx
