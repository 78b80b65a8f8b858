// chunk_gemm_cpar instances for one operand layout (kernel template in
// gemm_cpar_impl.h; one file per layout so the builds run in parallel).
#include "gemm_cpar_impl.h"

namespace fp8t {

const void* cpar_kernel_nn(int i) { return cpar::table<false, false, false>(i); }

}  // namespace fp8t
