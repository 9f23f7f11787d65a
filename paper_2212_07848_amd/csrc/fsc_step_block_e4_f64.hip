// fsc_step_block_e4_f64.hip -- instantiations of the block kernel (D2Q9, StencilE4_2D, double).
#include "fsc_block_kernel.h"

namespace fsc {

hipError_t launch_block_e4_f64(const BlockLaunch &P, hipStream_t s) {
    return launch_block_kind<StencilE4_2D, double>(P, s);
}

}  // namespace fsc
