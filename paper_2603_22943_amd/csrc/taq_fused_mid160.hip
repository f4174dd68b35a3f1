// Instantiations of the head-group variant of the fused block kernel for (head dimension, heads) = (160, 8): eight head groups of one head.
#include "taq_fused_kernel.h"

namespace taq {

hipError_t launch_fused_mid160(const FusedTable<1>& tab, const FusedDims& dm, int grid, hipStream_t st) {
    return launch_fused_cfg<160, 1, 1, 8, 16>(tab, dm, grid, st);
}

}  // namespace taq
