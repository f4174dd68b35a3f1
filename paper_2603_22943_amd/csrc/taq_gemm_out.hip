// to_out of the kernel-per-stage path.
#include "taq_gemm_op.h"

namespace taq {

template <bool PACKED>
static hipError_t launch(const GemmOpArgs& a, hipStream_t st) {
    if (tile_cost(a, 8, 5) < tile_cost(a, 4, 4) && tile_cost(a, 8, 5) < tile_cost(a, 8, 8)) return launch_gemm_op_cfg<PACKED, 2, 5, 4, 1, 0>(a, st);
    return launch_gemm_op<PACKED, 0>(a, st);
}

hipError_t launch_to_out_tiles(const GemmOpArgs& a, bool packed, hipStream_t st) { return packed ? launch<true>(a, st) : launch<false>(a, st); }

}  // namespace taq
