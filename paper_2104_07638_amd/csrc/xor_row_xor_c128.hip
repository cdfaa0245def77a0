// xor_row_xor_c128.hip -- the register xor minors kernels (xor_row.h), complex128, 4 to 16 blocks.
#include "xor_row_launch.h"

namespace apm {

hipError_t xor_row_launch_c128(const LaunchXor& L, hipStream_t st)
{
    return xrow::launch_n<FC128, xrow::kXor, 1, 4>(L, st);
}

}  // namespace apm
