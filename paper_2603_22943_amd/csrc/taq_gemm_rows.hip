// to_q of the kernel-per-stage path on row-major weights (taq_gemm.hip has it on operand-ordered ones).
#include "taq_gemm_op.h"

namespace taq {

hipError_t launch_to_q_rows(const GemmOpArgs& a, hipStream_t st) { return launch_to_q_tiles<false>(a, st); }

}  // namespace taq
