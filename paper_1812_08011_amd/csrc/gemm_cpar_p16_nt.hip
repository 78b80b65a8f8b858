// chunk_gemm_cpar instances with FP16 operands for one operand layout
// (kernel template in gemm_cpar_impl.h).
#include "gemm_cpar_impl.h"

namespace fp8t {

const void* cpar_p16_kernel_nt(int i) { return cpar::table<false, true, true>(i); }

}  // namespace fp8t
