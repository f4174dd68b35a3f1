// Instantiations of the head-group variant of the fused block kernel for (head dimension, heads) = (64, 20): ten head groups of two heads.
#include "taq_fused_kernel.h"

namespace taq {

hipError_t launch_fused_mid64(const FusedTable<1>& tab, const FusedDims& dm, int grid, hipStream_t st) {
    return launch_fused_cfg<64, 2, 1, 10, 16>(tab, dm, grid, st);
}

}  // namespace taq
