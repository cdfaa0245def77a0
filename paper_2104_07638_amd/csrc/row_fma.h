// row_fma.h -- multiply-adds whose one factor is a value of another lane of the row of 16
// lanes: v_fmac_f64_dpp with a row_newbcast operand, for Schur updates of matrices held one
// column per lane.  It issues at the rate of a plain fp64 multiply-add (5.0 against 4.7 to 5.0
// cycles per wavefront instruction), so the broadcast that row_bcast makes a move of its own is
// free.  The compiler has no form of it to choose, hence the assembly.
//
// Wait states: a DPP operand must not be written by a vector instruction among the two before
// its use.  The compiler does not look for that inside a block of assembly, so every block
// starts with two wait states or two other instructions, and inside a block no DPP operand is
// written less than three instructions ahead.  It does not look behind a block either: a value
// that a block has written may be read by DPP only through a block (row_bcast_after, or the
// functions here), never by row_bcast.  An s_nop 1 costs a lone wavefront 8 cycles, which is why
// the blocks hold several rows, and the copies of row_child.
// Dependent multiply-adds are 10 cycles apart: each block orders its instructions so that the
// two halves of a complex update are rows apart.
// The results are early-clobber: a block writes them before it has read all its operands.
//
// The rounding is that of F::upd, in its order: real a - c w; complex
// re: (a + c.y w.y) - c.x w.x, im: (a - c.y w.x) - c.x w.y.
#pragma once
#include "apm_device.h"

namespace apm {

#define APM_BC(P) " row_newbcast:%" #P " row_mask:0xf bank_mask:0xf\n\t"

// lane P of v, where an assembly block may have written v
template <int P>
__device__ __forceinline__ double row_bcast_after(double v)
{
    double r;
    asm("s_nop 1\n\t"
        "v_mov_b64_dpp %0, %1" APM_BC(2)
        : "=v"(r)
        : "v"(v), "n"(P));
    return r;
}

// lanes P and P + 1 of the last two rows of a node: its 2 x 2 pivot block
template <int P>
__device__ __forceinline__ void row_block_after(double r0, double r1, double& a00, double& a01, double& a10, double& a11)
{
    asm("s_nop 1\n\t"
        "v_mov_b64_dpp %0, %4" APM_BC(6)
        "v_mov_b64_dpp %1, %4" APM_BC(7)
        "v_mov_b64_dpp %2, %5" APM_BC(6)
        "v_mov_b64_dpp %3, %5" APM_BC(7)
        : "=&v"(a00), "=&v"(a01), "=&v"(a10), "=&v"(a11)
        : "v"(r0), "v"(r1), "n"(P), "n"(P + 1));
}

template <int P>
__device__ __forceinline__ void row_block_after(cd r0, cd r1, cd& a00, cd& a01, cd& a10, cd& a11)
{
    row_block_after<P>(r0.x, r1.x, a00.x, a01.x, a10.x, a11.x);
    row_block_after<P>(r0.y, r1.y, a00.y, a01.y, a10.y, a11.y);
}

// a[r] -= (lane P of a[r]) w, in place.  Complex: w must be zero in lane P, whose value the
// second half of the block reads again.
template <int P>
__device__ __forceinline__ void row_elim(double& a0, double& a1, double w)
{
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, -%0, %2" APM_BC(3)
        "v_fmac_f64_dpp %1, -%1, %2" APM_BC(3)
        : "+&v"(a0), "+&v"(a1)
        : "v"(w), "n"(P));
}

template <int P>
__device__ __forceinline__ void row_elim(double& a0, double& a1, double& a2, double& a3, double w)
{
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, -%0, %4" APM_BC(5)
        "v_fmac_f64_dpp %1, -%1, %4" APM_BC(5)
        "v_fmac_f64_dpp %2, -%2, %4" APM_BC(5)
        "v_fmac_f64_dpp %3, -%3, %4" APM_BC(5)
        : "+&v"(a0), "+&v"(a1), "+&v"(a2), "+&v"(a3)
        : "v"(w), "n"(P));
}

template <int P>
__device__ __forceinline__ void row_elim(double& a0, double& a1, double& a2, double& a3, double& a4, double& a5, double w)
{
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, -%0, %6" APM_BC(7)
        "v_fmac_f64_dpp %1, -%1, %6" APM_BC(7)
        "v_fmac_f64_dpp %2, -%2, %6" APM_BC(7)
        "v_fmac_f64_dpp %3, -%3, %6" APM_BC(7)
        "v_fmac_f64_dpp %4, -%4, %6" APM_BC(7)
        "v_fmac_f64_dpp %5, -%5, %6" APM_BC(7)
        : "+&v"(a0), "+&v"(a1), "+&v"(a2), "+&v"(a3), "+&v"(a4), "+&v"(a5)
        : "v"(w), "n"(P));
}

template <int P>
__device__ __forceinline__ void row_elim(double& a0, double& a1, double& a2, double& a3, double& a4, double& a5, double& a6, double& a7, double w)
{
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, -%0, %8" APM_BC(9)
        "v_fmac_f64_dpp %1, -%1, %8" APM_BC(9)
        "v_fmac_f64_dpp %2, -%2, %8" APM_BC(9)
        "v_fmac_f64_dpp %3, -%3, %8" APM_BC(9)
        "v_fmac_f64_dpp %4, -%4, %8" APM_BC(9)
        "v_fmac_f64_dpp %5, -%5, %8" APM_BC(9)
        "v_fmac_f64_dpp %6, -%6, %8" APM_BC(9)
        "v_fmac_f64_dpp %7, -%7, %8" APM_BC(9)
        : "+&v"(a0), "+&v"(a1), "+&v"(a2), "+&v"(a3), "+&v"(a4), "+&v"(a5), "+&v"(a6), "+&v"(a7)
        : "v"(w), "n"(P));
}

template <int P>
__device__ __forceinline__ void row_elim(cd& a0, cd& a1, cd w)
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
        : "+&v"(a0.x), "+&v"(a0.y), "+&v"(a1.x), "+&v"(a1.y)
        : "v"(w.x), "v"(w.y), "n"(P));
}

template <int P>
__device__ __forceinline__ void row_elim(cd& a0, cd& a1, cd& a2, cd& a3, cd w)
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
        : "+&v"(a0.x), "+&v"(a0.y), "+&v"(a1.x), "+&v"(a1.y), "+&v"(a2.x), "+&v"(a2.y), "+&v"(a3.x), "+&v"(a3.y)
        : "v"(w.x), "v"(w.y), "n"(P));
}

template <int P>
__device__ __forceinline__ void row_elim(cd& a0, cd& a1, cd& a2, cd& a3, cd& a4, cd& a5, cd w)
{
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %1, %13" APM_BC(14)
        "v_fmac_f64_dpp %2, %3, %13" APM_BC(14)
        "v_fmac_f64_dpp %4, %5, %13" APM_BC(14)
        "v_fmac_f64_dpp %6, %7, %13" APM_BC(14)
        "v_fmac_f64_dpp %8, %9, %13" APM_BC(14)
        "v_fmac_f64_dpp %10, %11, %13" APM_BC(14)
        "v_fmac_f64_dpp %1, -%1, %12" APM_BC(14)
        "v_fmac_f64_dpp %3, -%3, %12" APM_BC(14)
        "v_fmac_f64_dpp %5, -%5, %12" APM_BC(14)
        "v_fmac_f64_dpp %7, -%7, %12" APM_BC(14)
        "v_fmac_f64_dpp %9, -%9, %12" APM_BC(14)
        "v_fmac_f64_dpp %11, -%11, %12" APM_BC(14)
        "v_fmac_f64_dpp %1, -%0, %13" APM_BC(14)
        "v_fmac_f64_dpp %3, -%2, %13" APM_BC(14)
        "v_fmac_f64_dpp %5, -%4, %13" APM_BC(14)
        "v_fmac_f64_dpp %7, -%6, %13" APM_BC(14)
        "v_fmac_f64_dpp %9, -%8, %13" APM_BC(14)
        "v_fmac_f64_dpp %11, -%10, %13" APM_BC(14)
        "v_fmac_f64_dpp %0, -%0, %12" APM_BC(14)
        "v_fmac_f64_dpp %2, -%2, %12" APM_BC(14)
        "v_fmac_f64_dpp %4, -%4, %12" APM_BC(14)
        "v_fmac_f64_dpp %6, -%6, %12" APM_BC(14)
        "v_fmac_f64_dpp %8, -%8, %12" APM_BC(14)
        "v_fmac_f64_dpp %10, -%10, %12" APM_BC(14)
        : "+&v"(a0.x), "+&v"(a0.y), "+&v"(a1.x), "+&v"(a1.y), "+&v"(a2.x), "+&v"(a2.y), "+&v"(a3.x), "+&v"(a3.y), "+&v"(a4.x), "+&v"(a4.y), "+&v"(a5.x), "+&v"(a5.y)
        : "v"(w.x), "v"(w.y), "n"(P));
}

// The first two rows of a complex elimination: clears w in lane P (keep: 0 in that lane, 1 in
// the others) on the way, in place of the wait states.
template <int P>
__device__ __forceinline__ void row_elim_first(cd& a0, cd& a1, cd& w, double keep)
{
    asm("v_mul_f64 %4, %4, %6\n\t"
        "v_mul_f64 %5, %5, %6\n\t"
        "v_fmac_f64_dpp %0, %1, %5" APM_BC(7)
        "v_fmac_f64_dpp %2, %3, %5" APM_BC(7)
        "v_fmac_f64_dpp %1, -%1, %4" APM_BC(7)
        "v_fmac_f64_dpp %3, -%3, %4" APM_BC(7)
        "v_fmac_f64_dpp %1, -%0, %5" APM_BC(7)
        "v_fmac_f64_dpp %3, -%2, %5" APM_BC(7)
        "v_fmac_f64_dpp %0, -%0, %4" APM_BC(7)
        "v_fmac_f64_dpp %2, -%2, %4" APM_BC(7)
        : "+&v"(a0.x), "+&v"(a0.y), "+&v"(a1.x), "+&v"(a1.y), "+&v"(w.x), "+&v"(w.y)
        : "v"(keep), "n"(P));
}

// c[r] = a[r] - (lane P of a[r]) w
template <int P>
__device__ __forceinline__ void row_child(double& c0, double& c1, double a0, double a1, double w)
{
    asm("v_mov_b64_e32 %0, %2\n\t"
        "v_mov_b64_e32 %1, %3\n\t"
        "v_fmac_f64_dpp %0, -%2, %4" APM_BC(5)
        "v_fmac_f64_dpp %1, -%3, %4" APM_BC(5)
        : "=&v"(c0), "=&v"(c1)
        : "v"(a0), "v"(a1), "v"(w), "n"(P));
}

template <int P>
__device__ __forceinline__ void row_child(double& c0, double& c1, double& c2, double& c3, double a0, double a1, double a2, double a3, double w)
{
    asm("v_mov_b64_e32 %0, %4\n\t"
        "v_mov_b64_e32 %1, %5\n\t"
        "v_mov_b64_e32 %2, %6\n\t"
        "v_mov_b64_e32 %3, %7\n\t"
        "v_fmac_f64_dpp %0, -%4, %8" APM_BC(9)
        "v_fmac_f64_dpp %1, -%5, %8" APM_BC(9)
        "v_fmac_f64_dpp %2, -%6, %8" APM_BC(9)
        "v_fmac_f64_dpp %3, -%7, %8" APM_BC(9)
        : "=&v"(c0), "=&v"(c1), "=&v"(c2), "=&v"(c3)
        : "v"(a0), "v"(a1), "v"(a2), "v"(a3), "v"(w), "n"(P));
}

template <int P>
__device__ __forceinline__ void row_child(double& c0, double& c1, double& c2, double& c3, double& c4, double& c5, double a0, double a1, double a2, double a3, double a4, double a5, double w)
{
    asm("v_mov_b64_e32 %0, %6\n\t"
        "v_mov_b64_e32 %1, %7\n\t"
        "v_mov_b64_e32 %2, %8\n\t"
        "v_mov_b64_e32 %3, %9\n\t"
        "v_mov_b64_e32 %4, %10\n\t"
        "v_mov_b64_e32 %5, %11\n\t"
        "v_fmac_f64_dpp %0, -%6, %12" APM_BC(13)
        "v_fmac_f64_dpp %1, -%7, %12" APM_BC(13)
        "v_fmac_f64_dpp %2, -%8, %12" APM_BC(13)
        "v_fmac_f64_dpp %3, -%9, %12" APM_BC(13)
        "v_fmac_f64_dpp %4, -%10, %12" APM_BC(13)
        "v_fmac_f64_dpp %5, -%11, %12" APM_BC(13)
        : "=&v"(c0), "=&v"(c1), "=&v"(c2), "=&v"(c3), "=&v"(c4), "=&v"(c5)
        : "v"(a0), "v"(a1), "v"(a2), "v"(a3), "v"(a4), "v"(a5), "v"(w), "n"(P));
}

template <int P>
__device__ __forceinline__ void row_child(cd& c0, cd& c1, cd a0, cd a1, cd w)
{
    asm("v_mov_b64_e32 %0, %4\n\t"
        "v_mov_b64_e32 %1, %5\n\t"
        "v_mov_b64_e32 %2, %6\n\t"
        "v_mov_b64_e32 %3, %7\n\t"
        "v_fmac_f64_dpp %0, %5, %9" APM_BC(10)
        "v_fmac_f64_dpp %2, %7, %9" APM_BC(10)
        "v_fmac_f64_dpp %1, -%5, %8" APM_BC(10)
        "v_fmac_f64_dpp %3, -%7, %8" APM_BC(10)
        "v_fmac_f64_dpp %0, -%4, %8" APM_BC(10)
        "v_fmac_f64_dpp %2, -%6, %8" APM_BC(10)
        "v_fmac_f64_dpp %1, -%4, %9" APM_BC(10)
        "v_fmac_f64_dpp %3, -%6, %9" APM_BC(10)
        : "=&v"(c0.x), "=&v"(c0.y), "=&v"(c1.x), "=&v"(c1.y)
        : "v"(a0.x), "v"(a0.y), "v"(a1.x), "v"(a1.y), "v"(w.x), "v"(w.y), "n"(P));
}

template <int P>
__device__ __forceinline__ void row_child(cd& c0, cd& c1, cd& c2, cd& c3, cd a0, cd a1, cd a2, cd a3, cd w)
{
    asm("v_mov_b64_e32 %0, %8\n\t"
        "v_mov_b64_e32 %1, %9\n\t"
        "v_mov_b64_e32 %2, %10\n\t"
        "v_mov_b64_e32 %3, %11\n\t"
        "v_mov_b64_e32 %4, %12\n\t"
        "v_mov_b64_e32 %5, %13\n\t"
        "v_mov_b64_e32 %6, %14\n\t"
        "v_mov_b64_e32 %7, %15\n\t"
        "v_fmac_f64_dpp %0, %9, %17" APM_BC(18)
        "v_fmac_f64_dpp %2, %11, %17" APM_BC(18)
        "v_fmac_f64_dpp %4, %13, %17" APM_BC(18)
        "v_fmac_f64_dpp %6, %15, %17" APM_BC(18)
        "v_fmac_f64_dpp %1, -%9, %16" APM_BC(18)
        "v_fmac_f64_dpp %3, -%11, %16" APM_BC(18)
        "v_fmac_f64_dpp %5, -%13, %16" APM_BC(18)
        "v_fmac_f64_dpp %7, -%15, %16" APM_BC(18)
        "v_fmac_f64_dpp %0, -%8, %16" APM_BC(18)
        "v_fmac_f64_dpp %2, -%10, %16" APM_BC(18)
        "v_fmac_f64_dpp %4, -%12, %16" APM_BC(18)
        "v_fmac_f64_dpp %6, -%14, %16" APM_BC(18)
        "v_fmac_f64_dpp %1, -%8, %17" APM_BC(18)
        "v_fmac_f64_dpp %3, -%10, %17" APM_BC(18)
        "v_fmac_f64_dpp %5, -%12, %17" APM_BC(18)
        "v_fmac_f64_dpp %7, -%14, %17" APM_BC(18)
        : "=&v"(c0.x), "=&v"(c0.y), "=&v"(c1.x), "=&v"(c1.y), "=&v"(c2.x), "=&v"(c2.y), "=&v"(c3.x), "=&v"(c3.y)
        : "v"(a0.x), "v"(a0.y), "v"(a1.x), "v"(a1.y), "v"(a2.x), "v"(a2.y), "v"(a3.x), "v"(a3.y), "v"(w.x), "v"(w.y), "n"(P));
}

// a[r] -= (lane P of s[r]) w, with sources other than the results
template <int P>
__device__ __forceinline__ void row_sub(double& a0, double& a1, double& a2, double& a3, double s0, double s1, double s2, double s3, double w)
{
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, -%4, %8" APM_BC(9)
        "v_fmac_f64_dpp %1, -%5, %8" APM_BC(9)
        "v_fmac_f64_dpp %2, -%6, %8" APM_BC(9)
        "v_fmac_f64_dpp %3, -%7, %8" APM_BC(9)
        : "+&v"(a0), "+&v"(a1), "+&v"(a2), "+&v"(a3)
        : "v"(s0), "v"(s1), "v"(s2), "v"(s3), "v"(w), "n"(P));
}

template <int P>
__device__ __forceinline__ void row_sub(cd& a0, cd& a1, cd& a2, cd& a3, cd s0, cd s1, cd s2, cd s3, cd w)
{
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %9, %17" APM_BC(18)
        "v_fmac_f64_dpp %2, %11, %17" APM_BC(18)
        "v_fmac_f64_dpp %4, %13, %17" APM_BC(18)
        "v_fmac_f64_dpp %6, %15, %17" APM_BC(18)
        "v_fmac_f64_dpp %1, -%9, %16" APM_BC(18)
        "v_fmac_f64_dpp %3, -%11, %16" APM_BC(18)
        "v_fmac_f64_dpp %5, -%13, %16" APM_BC(18)
        "v_fmac_f64_dpp %7, -%15, %16" APM_BC(18)
        "v_fmac_f64_dpp %0, -%8, %16" APM_BC(18)
        "v_fmac_f64_dpp %2, -%10, %16" APM_BC(18)
        "v_fmac_f64_dpp %4, -%12, %16" APM_BC(18)
        "v_fmac_f64_dpp %6, -%14, %16" APM_BC(18)
        "v_fmac_f64_dpp %1, -%8, %17" APM_BC(18)
        "v_fmac_f64_dpp %3, -%10, %17" APM_BC(18)
        "v_fmac_f64_dpp %5, -%12, %17" APM_BC(18)
        "v_fmac_f64_dpp %7, -%14, %17" APM_BC(18)
        : "+&v"(a0.x), "+&v"(a0.y), "+&v"(a1.x), "+&v"(a1.y), "+&v"(a2.x), "+&v"(a2.y), "+&v"(a3.x), "+&v"(a3.y)
        : "v"(s0.x), "v"(s0.y), "v"(s1.x), "v"(s1.y), "v"(s2.x), "v"(s2.y), "v"(s3.x), "v"(s3.y), "v"(w.x), "v"(w.y), "n"(P));
}

// c[r] = a[r] - (lane P of a[r]) w0 - (lane P + 1 of a[r]) w1
template <int P>
__device__ __forceinline__ void row_child2(double& c0, double& c1, double a0, double a1, double w0, double w1)
{
    asm("v_mov_b64_e32 %0, %2\n\t"
        "v_mov_b64_e32 %1, %3\n\t"
        "v_fmac_f64_dpp %0, -%2, %4" APM_BC(6)
        "v_fmac_f64_dpp %1, -%3, %4" APM_BC(6)
        "v_fmac_f64_dpp %0, -%2, %5" APM_BC(7)
        "v_fmac_f64_dpp %1, -%3, %5" APM_BC(7)
        : "=&v"(c0), "=&v"(c1)
        : "v"(a0), "v"(a1), "v"(w0), "v"(w1), "n"(P), "n"(P + 1));
}

template <int P>
__device__ __forceinline__ void row_child2(double& c0, double& c1, double& c2, double& c3, double a0, double a1, double a2, double a3, double w0, double w1)
{
    asm("v_mov_b64_e32 %0, %4\n\t"
        "v_mov_b64_e32 %1, %5\n\t"
        "v_mov_b64_e32 %2, %6\n\t"
        "v_mov_b64_e32 %3, %7\n\t"
        "v_fmac_f64_dpp %0, -%4, %8" APM_BC(10)
        "v_fmac_f64_dpp %1, -%5, %8" APM_BC(10)
        "v_fmac_f64_dpp %2, -%6, %8" APM_BC(10)
        "v_fmac_f64_dpp %3, -%7, %8" APM_BC(10)
        "v_fmac_f64_dpp %0, -%4, %9" APM_BC(11)
        "v_fmac_f64_dpp %1, -%5, %9" APM_BC(11)
        "v_fmac_f64_dpp %2, -%6, %9" APM_BC(11)
        "v_fmac_f64_dpp %3, -%7, %9" APM_BC(11)
        : "=&v"(c0), "=&v"(c1), "=&v"(c2), "=&v"(c3)
        : "v"(a0), "v"(a1), "v"(a2), "v"(a3), "v"(w0), "v"(w1), "n"(P), "n"(P + 1));
}

template <int P>
__device__ __forceinline__ void row_child2(cd& c0, cd& c1, cd a0, cd a1, cd w0, cd w1)
{
    asm("v_mov_b64_e32 %0, %4\n\t"
        "v_mov_b64_e32 %1, %5\n\t"
        "v_mov_b64_e32 %2, %6\n\t"
        "v_mov_b64_e32 %3, %7\n\t"
        "v_fmac_f64_dpp %0, %5, %9" APM_BC(12)
        "v_fmac_f64_dpp %2, %7, %9" APM_BC(12)
        "v_fmac_f64_dpp %1, -%5, %8" APM_BC(12)
        "v_fmac_f64_dpp %3, -%7, %8" APM_BC(12)
        "v_fmac_f64_dpp %0, -%4, %8" APM_BC(12)
        "v_fmac_f64_dpp %2, -%6, %8" APM_BC(12)
        "v_fmac_f64_dpp %1, -%4, %9" APM_BC(12)
        "v_fmac_f64_dpp %3, -%6, %9" APM_BC(12)
        "v_fmac_f64_dpp %0, %5, %11" APM_BC(13)
        "v_fmac_f64_dpp %2, %7, %11" APM_BC(13)
        "v_fmac_f64_dpp %1, -%5, %10" APM_BC(13)
        "v_fmac_f64_dpp %3, -%7, %10" APM_BC(13)
        "v_fmac_f64_dpp %0, -%4, %10" APM_BC(13)
        "v_fmac_f64_dpp %2, -%6, %10" APM_BC(13)
        "v_fmac_f64_dpp %1, -%4, %11" APM_BC(13)
        "v_fmac_f64_dpp %3, -%6, %11" APM_BC(13)
        : "=&v"(c0.x), "=&v"(c0.y), "=&v"(c1.x), "=&v"(c1.y)
        : "v"(a0.x), "v"(a0.y), "v"(a1.x), "v"(a1.y), "v"(w0.x), "v"(w0.y), "v"(w1.x), "v"(w1.y), "n"(P),
          "n"(P + 1));
}

template <int P>
__device__ __forceinline__ void row_child2(cd& c0, cd& c1, cd& c2, cd& c3, cd a0, cd a1, cd a2, cd a3, cd w0, cd w1)
{
    asm("v_mov_b64_e32 %0, %8\n\t"
        "v_mov_b64_e32 %1, %9\n\t"
        "v_mov_b64_e32 %2, %10\n\t"
        "v_mov_b64_e32 %3, %11\n\t"
        "v_mov_b64_e32 %4, %12\n\t"
        "v_mov_b64_e32 %5, %13\n\t"
        "v_mov_b64_e32 %6, %14\n\t"
        "v_mov_b64_e32 %7, %15\n\t"
        "v_fmac_f64_dpp %0, %9, %17" APM_BC(20)
        "v_fmac_f64_dpp %2, %11, %17" APM_BC(20)
        "v_fmac_f64_dpp %4, %13, %17" APM_BC(20)
        "v_fmac_f64_dpp %6, %15, %17" APM_BC(20)
        "v_fmac_f64_dpp %1, -%9, %16" APM_BC(20)
        "v_fmac_f64_dpp %3, -%11, %16" APM_BC(20)
        "v_fmac_f64_dpp %5, -%13, %16" APM_BC(20)
        "v_fmac_f64_dpp %7, -%15, %16" APM_BC(20)
        "v_fmac_f64_dpp %0, -%8, %16" APM_BC(20)
        "v_fmac_f64_dpp %2, -%10, %16" APM_BC(20)
        "v_fmac_f64_dpp %4, -%12, %16" APM_BC(20)
        "v_fmac_f64_dpp %6, -%14, %16" APM_BC(20)
        "v_fmac_f64_dpp %1, -%8, %17" APM_BC(20)
        "v_fmac_f64_dpp %3, -%10, %17" APM_BC(20)
        "v_fmac_f64_dpp %5, -%12, %17" APM_BC(20)
        "v_fmac_f64_dpp %7, -%14, %17" APM_BC(20)
        "v_fmac_f64_dpp %0, %9, %19" APM_BC(21)
        "v_fmac_f64_dpp %2, %11, %19" APM_BC(21)
        "v_fmac_f64_dpp %4, %13, %19" APM_BC(21)
        "v_fmac_f64_dpp %6, %15, %19" APM_BC(21)
        "v_fmac_f64_dpp %1, -%9, %18" APM_BC(21)
        "v_fmac_f64_dpp %3, -%11, %18" APM_BC(21)
        "v_fmac_f64_dpp %5, -%13, %18" APM_BC(21)
        "v_fmac_f64_dpp %7, -%15, %18" APM_BC(21)
        "v_fmac_f64_dpp %0, -%8, %18" APM_BC(21)
        "v_fmac_f64_dpp %2, -%10, %18" APM_BC(21)
        "v_fmac_f64_dpp %4, -%12, %18" APM_BC(21)
        "v_fmac_f64_dpp %6, -%14, %18" APM_BC(21)
        "v_fmac_f64_dpp %1, -%8, %19" APM_BC(21)
        "v_fmac_f64_dpp %3, -%10, %19" APM_BC(21)
        "v_fmac_f64_dpp %5, -%12, %19" APM_BC(21)
        "v_fmac_f64_dpp %7, -%14, %19" APM_BC(21)
        : "=&v"(c0.x), "=&v"(c0.y), "=&v"(c1.x), "=&v"(c1.y), "=&v"(c2.x), "=&v"(c2.y), "=&v"(c3.x), "=&v"(c3.y)
        : "v"(a0.x), "v"(a0.y), "v"(a1.x), "v"(a1.y), "v"(a2.x), "v"(a2.y), "v"(a3.x), "v"(a3.y), "v"(w0.x), "v"(w0.y), "v"(w1.x), "v"(w1.y), "n"(P),
          "n"(P + 1));
}

// a[r] -= (lane P + r of s) w
template <int P>
__device__ __forceinline__ void row_sub_lanes(double& a0, double& a1, double& a2, double& a3, double& a4, double& a5, double& a6, double& a7, double s, double w)
{
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, -%8, %9" APM_BC(10)
        "v_fmac_f64_dpp %1, -%8, %9" APM_BC(11)
        "v_fmac_f64_dpp %2, -%8, %9" APM_BC(12)
        "v_fmac_f64_dpp %3, -%8, %9" APM_BC(13)
        "v_fmac_f64_dpp %4, -%8, %9" APM_BC(14)
        "v_fmac_f64_dpp %5, -%8, %9" APM_BC(15)
        "v_fmac_f64_dpp %6, -%8, %9" APM_BC(16)
        "v_fmac_f64_dpp %7, -%8, %9" APM_BC(17)
        : "+&v"(a0), "+&v"(a1), "+&v"(a2), "+&v"(a3), "+&v"(a4), "+&v"(a5), "+&v"(a6), "+&v"(a7)
        : "v"(s), "v"(w), "n"(P + 0), "n"(P + 1), "n"(P + 2), "n"(P + 3), "n"(P + 4), "n"(P + 5), "n"(P + 6), "n"(P + 7));
}

template <int P>
__device__ __forceinline__ void row_sub_lanes(cd& a0, cd& a1, cd& a2, cd& a3, cd s, cd w)
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
        : "+&v"(a0.x), "+&v"(a0.y), "+&v"(a1.x), "+&v"(a1.y), "+&v"(a2.x), "+&v"(a2.y), "+&v"(a3.x), "+&v"(a3.y)
        : "v"(s.x), "v"(s.y), "v"(w.x), "v"(w.y), "n"(P + 0), "n"(P + 1), "n"(P + 2), "n"(P + 3));
}

#undef APM_BC

}  // namespace apm
