// fsc_step_block_e4_f32.hip -- instantiations of the block kernel (D2Q9, StencilE4_2D, float).
#include "fsc_block_kernel.h"

namespace fsc {

hipError_t launch_block_e4_f32(const BlockLaunch &P, hipStream_t s) {
    return launch_block_kind<StencilE4_2D, float>(P, s);
}

}  // namespace fsc
