// fp32 fast search kernels: up to 8 models, hidden width 64.
#include "mf_fast_kernel.h"

namespace mfi {

hipError_t launch_fast_n8_h64(const FastArgs &a, const FastConst &fc, int grid, int kp, int mode, hipStream_t s)
{
    return launch_fast_for<8, 64>(a, fc, grid, kp, mode, s);
}

}  // namespace mfi
