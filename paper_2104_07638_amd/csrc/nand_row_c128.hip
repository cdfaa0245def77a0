// nand_row_c128.hip -- the register NAND minors kernels (nand_row.h), complex128, 7 to 13 blocks.
#include "nand_row.h"

namespace apm {

hipError_t nand_row_launch_c128(const LaunchXor& L, hipStream_t st)
{
    return nrow::launch_n<FC128, 1, 7>(L, st);
}

}  // namespace apm
