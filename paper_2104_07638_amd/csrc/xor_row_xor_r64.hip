// xor_row_xor_r64.hip -- the register xor minors kernels (xor_row.h), fp64, 4 to 16 blocks.
#include "xor_row_launch.h"

namespace apm {

hipError_t xor_row_launch_r64(const LaunchXor& L, hipStream_t st)
{
    return xrow::launch_n<FR64, xrow::kXor, 2, 4>(L, st);
}

}  // namespace apm
