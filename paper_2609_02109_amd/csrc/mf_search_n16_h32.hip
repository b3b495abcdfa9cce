// fp32 fast search kernels: up to 16 models, hidden width 32.
#include "mf_fast_kernel.h"

namespace mfi {

hipError_t launch_fast_n16_h32(const FastArgs &a, const FastConst &fc, int grid, int kp, int mode, hipStream_t s)
{
    return launch_fast_for<16, 32>(a, fc, grid, kp, mode, s);
}

}  // namespace mfi
