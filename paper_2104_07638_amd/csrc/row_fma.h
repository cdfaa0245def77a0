// row_fma.h -- multiply-adds whose one factor is a value of another lane of the row of 16
// lanes: v_fmac_f64_dpp with a row_newbcast operand, for Schur updates of matrices held one
// column per lane.  It issues at the rate of a plain fp64 multiply-add (5.45 against 5.2 cycles
// per wavefront instruction), so the broadcast that row_bcast makes a move of its own is free.
// The compiler has no form of it to choose, hence the assembly.  Every block starts and ends
// with two wait states: a DPP operand must not be written by one of the two instructions
// before its use, and the compiler does not look for that inside (or right behind) a block.
// Within a block no DPP operand is written less than three instructions ahead.  The results
// are early-clobber: a block writes them before it has read all its operands.
//
// The rounding is that of F::upd, in its order: real a - c w; complex
// re: (a + c.y w.y) - c.x w.x, im: (a - c.y w.x) - c.x w.y.
#pragma once
#include "apm_device.h"

namespace apm {

#define APM_BC(P) " row_newbcast:%" #P " row_mask:0xf bank_mask:0xf\n\t"

// a[r] -= (lane P of a[r]) w, r = 0..3.  Complex: w must be zero in lane P, whose value the
// second half of the block reads again.
template <int P>
__device__ __forceinline__ void row_elim4(double& a0, double& a1, double& a2, double& a3, double w)
{
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, -%0, %4" APM_BC(5)
        "v_fmac_f64_dpp %1, -%1, %4" APM_BC(5)
        "v_fmac_f64_dpp %2, -%2, %4" APM_BC(5)
        "v_fmac_f64_dpp %3, -%3, %4" APM_BC(5)
        "s_nop 1"
        : "+&v"(a0), "+&v"(a1), "+&v"(a2), "+&v"(a3)
        : "v"(w), "n"(P));
}

template <int P>
__device__ __forceinline__ void row_elim2(double& a0, double& a1, double w)
{
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, -%0, %2" APM_BC(3)
        "v_fmac_f64_dpp %1, -%1, %2" APM_BC(3)
        "s_nop 1"
        : "+&v"(a0), "+&v"(a1)
        : "v"(w), "n"(P));
}

template <int P>
__device__ __forceinline__ void row_elim4(cd& a0, cd& a1, cd& a2, cd& a3, cd w)
{
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %1, %9" APM_BC(10)
        "v_fmac_f64_dpp %2, %3, %9" APM_BC(10)
        "v_fmac_f64_dpp %4, %5, %9" APM_BC(10)
        "v_fmac_f64_dpp %6, %7, %9" APM_BC(10)
        "v_fmac_f64_dpp %1, -%1, %8" APM_BC(10)
        "v_fmac_f64_dpp %3, -%3, %8" APM_BC(10)
        "v_fmac_f64_dpp %5, -%5, %8" APM_BC(10)
        "v_fmac_f64_dpp %7, -%7, %8" APM_BC(10)
        "v_fmac_f64_dpp %1, -%0, %9" APM_BC(10)
        "v_fmac_f64_dpp %3, -%2, %9" APM_BC(10)
        "v_fmac_f64_dpp %5, -%4, %9" APM_BC(10)
        "v_fmac_f64_dpp %7, -%6, %9" APM_BC(10)
        "v_fmac_f64_dpp %0, -%0, %8" APM_BC(10)
        "v_fmac_f64_dpp %2, -%2, %8" APM_BC(10)
        "v_fmac_f64_dpp %4, -%4, %8" APM_BC(10)
        "v_fmac_f64_dpp %6, -%6, %8" APM_BC(10)
        "s_nop 1"
        : "+&v"(a0.x), "+&v"(a0.y), "+&v"(a1.x), "+&v"(a1.y), "+&v"(a2.x), "+&v"(a2.y), "+&v"(a3.x), "+&v"(a3.y)
        : "v"(w.x), "v"(w.y), "n"(P));
}

template <int P>
__device__ __forceinline__ void row_elim2(cd& a0, cd& a1, cd w)
{
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %1, %5" APM_BC(6)
        "v_fmac_f64_dpp %2, %3, %5" APM_BC(6)
        "v_fmac_f64_dpp %1, -%1, %4" APM_BC(6)
        "v_fmac_f64_dpp %3, -%3, %4" APM_BC(6)
        "v_fmac_f64_dpp %1, -%0, %5" APM_BC(6)
        "v_fmac_f64_dpp %3, -%2, %5" APM_BC(6)
        "v_fmac_f64_dpp %0, -%0, %4" APM_BC(6)
        "v_fmac_f64_dpp %2, -%2, %4" APM_BC(6)
        "s_nop 1"
        : "+&v"(a0.x), "+&v"(a0.y), "+&v"(a1.x), "+&v"(a1.y)
        : "v"(w.x), "v"(w.y), "n"(P));
}

// a[r] -= (lane P of s[r]) w, r = 0..1, with sources other than the results.
template <int P>
__device__ __forceinline__ void row_sub2(double& a0, double& a1, double s0, double s1, double w)
{
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, -%2, %4" APM_BC(5)
        "v_fmac_f64_dpp %1, -%3, %4" APM_BC(5)
        "s_nop 1"
        : "+&v"(a0), "+&v"(a1)
        : "v"(s0), "v"(s1), "v"(w), "n"(P));
}

template <int P>
__device__ __forceinline__ void row_sub2(cd& a0, cd& a1, cd s0, cd s1, cd w)
{
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %5, %9" APM_BC(10)
        "v_fmac_f64_dpp %2, %7, %9" APM_BC(10)
        "v_fmac_f64_dpp %1, -%5, %8" APM_BC(10)
        "v_fmac_f64_dpp %3, -%7, %8" APM_BC(10)
        "v_fmac_f64_dpp %0, -%4, %8" APM_BC(10)
        "v_fmac_f64_dpp %2, -%6, %8" APM_BC(10)
        "v_fmac_f64_dpp %1, -%4, %9" APM_BC(10)
        "v_fmac_f64_dpp %3, -%6, %9" APM_BC(10)
        "s_nop 1"
        : "+&v"(a0.x), "+&v"(a0.y), "+&v"(a1.x), "+&v"(a1.y)
        : "v"(s0.x), "v"(s0.y), "v"(s1.x), "v"(s1.y), "v"(w.x), "v"(w.y), "n"(P));
}

// a[r] -= (lane P + r of s) w, r = 0..3.
template <int P>
__device__ __forceinline__ void row_sub_lanes4(double& a0, double& a1, double& a2, double& a3, double s, double w)
{
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, -%4, %5" APM_BC(6)
        "v_fmac_f64_dpp %1, -%4, %5" APM_BC(7)
        "v_fmac_f64_dpp %2, -%4, %5" APM_BC(8)
        "v_fmac_f64_dpp %3, -%4, %5" APM_BC(9)
        "s_nop 1"
        : "+&v"(a0), "+&v"(a1), "+&v"(a2), "+&v"(a3)
        : "v"(s), "v"(w), "n"(P), "n"(P + 1), "n"(P + 2), "n"(P + 3));
}

template <int P>
__device__ __forceinline__ void row_sub_lanes4(cd& a0, cd& a1, cd& a2, cd& a3, cd s, cd w)
{
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %9, %11" APM_BC(12)
        "v_fmac_f64_dpp %2, %9, %11" APM_BC(13)
        "v_fmac_f64_dpp %4, %9, %11" APM_BC(14)
        "v_fmac_f64_dpp %6, %9, %11" APM_BC(15)
        "v_fmac_f64_dpp %1, -%9, %10" APM_BC(12)
        "v_fmac_f64_dpp %3, -%9, %10" APM_BC(13)
        "v_fmac_f64_dpp %5, -%9, %10" APM_BC(14)
        "v_fmac_f64_dpp %7, -%9, %10" APM_BC(15)
        "v_fmac_f64_dpp %0, -%8, %10" APM_BC(12)
        "v_fmac_f64_dpp %2, -%8, %10" APM_BC(13)
        "v_fmac_f64_dpp %4, -%8, %10" APM_BC(14)
        "v_fmac_f64_dpp %6, -%8, %10" APM_BC(15)
        "v_fmac_f64_dpp %1, -%8, %11" APM_BC(12)
        "v_fmac_f64_dpp %3, -%8, %11" APM_BC(13)
        "v_fmac_f64_dpp %5, -%8, %11" APM_BC(14)
        "v_fmac_f64_dpp %7, -%8, %11" APM_BC(15)
        "s_nop 1"
        : "+&v"(a0.x), "+&v"(a0.y), "+&v"(a1.x), "+&v"(a1.y), "+&v"(a2.x), "+&v"(a2.y), "+&v"(a3.x), "+&v"(a3.y)
        : "v"(s.x), "v"(s.y), "v"(w.x), "v"(w.y), "n"(P), "n"(P + 1), "n"(P + 2), "n"(P + 3));
}

#undef APM_BC

}  // namespace apm
