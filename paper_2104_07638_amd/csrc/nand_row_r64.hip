// nand_row_r64.hip -- the register NAND minors kernels (nand_row.h), fp64, 7 to 13 blocks.
#include "nand_row.h"

namespace apm {

hipError_t nand_row_launch_r64(const LaunchXor& L, hipStream_t st)
{
    return nrow::launch_n<FR64, 2, 7>(L, st);
}

}  // namespace apm
