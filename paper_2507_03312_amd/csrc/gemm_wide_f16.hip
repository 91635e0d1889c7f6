// GEMM kernels for fp16 operands: the wide tiles (see gemm_kernels.h).
#define MPX_GEMM_WIDE_SOURCE
#include "gemm_kernels.h"

namespace mpx {

MPX_GEMM_WIDE(, MPX_F16)

}  // namespace mpx
