// fsc_step_block_e8_f32.hip -- instantiations of the block kernel (D2Q9, StencilE8_2D, float).
#include "fsc_block_kernel.h"

namespace fsc {

hipError_t launch_block_e8_f32(const BlockLaunch &P, hipStream_t s) {
    return launch_block_kind<StencilE8_2D, float>(P, s);
}

}  // namespace fsc
