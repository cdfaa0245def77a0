// xor_row.h -- block minors (Sec. III) with the node matrices in registers, on gfx950.
//
// The trees are those of xor.hip (XOR, XNOR; the last block is decided first, every Schur
// step in the same order of operations).  There a wavefront works through one matrix in
// small dependent passes over LDS and a workspace; here a node of order m <= 16 is held by
// one row of 16 lanes, lane j holding column j in registers, so that a Schur step needs no
// memory: the pivot column reaches the other lanes by DPP row broadcast, which costs no more
// than a move, and the scaled pivot row is already in its lanes.  A wavefront runs four such
// nodes ("units") side by side.  Three phases:
//   * top: a unit is a matrix and one choice for each of its T = max(0, N - 8) last blocks.
//     With the choices known, only their kept rows and columns are loaded (XOR: T of them,
//     XNOR: 2 T, those of a left-out block replaced by unit vectors) beside the 16 undecided
//     ones, and the kept ones are eliminated in the tree's order.  Nothing is shared between
//     units, so a matrix can be split over any number of wavefronts, and no workspace is
//     needed.  The kept columns sit in a second register of the lanes.
//   * rows: depth first from order 16 (2 N below 8 blocks) to order 8, fully unrolled.  The
//     order-8 nodes, 8 a unit at a time, go to LDS (16-byte columns, padded to an odd number
//     of elements).
//   * lanes: one order-6 child of them per lane (64 lanes, all busy from 7 blocks on), with
//     its three levels in the lane's registers.  Its minors are staged through LDS, so that
//     stores write whole lines.
// Bound by fp64 issue at one or two wavefronts per SIMD (a lone one issues every 4.8 cycles) and,
// for XOR, by the output.  Against one matrix per wavefront in LDS passes: 4096 complex XOR of 14
// blocks 2.83 -> 0.94 ms (2.3 TB/s), 3001 real XNOR of 11 blocks 149 -> 39 us, and small batches
// 5 to 100 times, a matrix being split over as many wavefronts as fill the chip.
// Why order 8: below it a row of 16 lanes is less than half used, while a lane cannot hold
// more than an order-6 complex node (144 registers) and its children.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "apm_device.h"
#include "apm_kernels.h"
#include "row_fma.h"

namespace apm {
namespace xrow {

constexpr int kXor = 0, kXnor = 1;
constexpr int kParents = 32;        // order-8 nodes in LDS at a time
constexpr int kPS = 65;             // their stride in elements
constexpr int kSlots = 16;

__host__ __device__ constexpr int top_levels(int N) { return N > 8 ? N - 8 : 0; }
// order-8 nodes of a unit per lane phase, and lane phases per unit
__host__ __device__ constexpr int parents(int N) { return N >= 7 ? 8 : 1 << (N - 4); }
__host__ __device__ constexpr int halves(int N) { return N >= 8 ? 2 : 1; }

template <class F>
struct Lds {
    typename F::E node[kParents * kPS];
    typename F::E mn[4 * kSlots];   // minors of the row phase, kSlots a unit (keep())
    typename F::E dump[64 + kSlots];
};

// v where m is all ones, zero where m is zero (no branch around the load of v)
__device__ __forceinline__ double keep_if(int m, double v)
{
    return __hiloint2double(__double2hiint(v) & m, __double2loint(v) & m);
}
__device__ __forceinline__ cd keep_if(int m, cd v) { return {keep_if(m, v.x), keep_if(m, v.y)}; }
__device__ __forceinline__ double unit_if(bool c) { return __hiloint2double(c ? 0x3FF00000 : 0, 0); }

// The lane number, new to the compiler at every call: addresses made from it are formed where
// they are used instead of being kept in registers across the whole loop over the units.
__device__ __forceinline__ int lane_here()
{
    int l = (int)threadIdx.x;
    asm volatile("" : "+v"(l));
    return l;
}

template <class F, int N, int MODE>
struct Unit {
    using E = typename F::E;
    static constexpr int T = top_levels(N);
    static constexpr int R0 = 2 * (N - T);
    static constexpr int NPR = parents(N);
    static constexpr int LV8 = N >= 7 ? 3 : N - 4;   // row-phase levels down to order 8
    static constexpr int kLast = LV8 ? (1 << LV8) - 2 : 0;   // slot of the first order-8 node's minor

    Lds<F>& sh;
    E* ob;            // this row's matrix's output
    int path;         // its choices of the top levels
    int l16;          // lane in the row
    bool valid;       // whether there is such a unit
    bool wr;          // the lane that writes the top levels' minors
    double chk = 0.0;

    __device__ Unit(Lds<F>& s) : sh(s) {}

    // ---------------------------------------------------------------- top phase
    // The depth-T node of the path: M[i] = row i of its lane's column; mk = its minor.
    __device__ __forceinline__ void top(const E* A0, E (&M)[R0], E& mk)
    {
        constexpr int w = 2 * N;
        if constexpr (T == 0) {
            const int c = l16 < w ? l16 : w - 1;
#pragma unroll
            for (int i = 0; i < R0; ++i) M[i] = A0[i * w + c];
        } else if constexpr (MODE == kXor) {
            // lane t's kept column: the chosen one of block N - 1 - t
            const int t = l16 < T ? l16 : T - 1;
            const int kc = 2 * (N - 1 - t) + ((path >> (T - 1 - t)) & 1);
            // every load first (one memory round trip; left alone, the compiler saves
            // registers by loading a row or two at a time): the kept rows, the kept columns
            // with a row per lane, the undecided rows
            E w0[T], w1[T], c[T];
#pragma unroll
            for (int k = 0; k < T; ++k) {
                const int row = 2 * (N - 1 - k) + ((path >> (T - 1 - k)) & 1);
                w0[k] = load_reg(&A0[row * w + l16]);
                w1[k] = load_reg(&A0[row * w + kc]);
            }
#pragma unroll
            for (int k = 0; k < T; ++k) c[k] = load_reg(&A0[l16 * w + 2 * (N - 1 - k) + ((path >> (T - 1 - k)) & 1)]);
#pragma unroll
            for (int i = 0; i < R0; ++i) M[i] = load_reg(&A0[i * w + l16]);
            __builtin_amdgcn_sched_barrier(0);
            top_xor_pivots<0>(w0, w1, mk);
            // the undecided rows' multipliers: the kept columns eliminated for all 16 rows at once
            multipliers<0, 1>(c, w1);
#pragma unroll
            for (int k = 0; k < T; ++k) sub_rows<0>(M, c[k], w0[k]);
        } else {
            // lane 2 t + r's kept column: column r of block N - 1 - t (zero if left out)
            const int t = l16 < 2 * T ? l16 >> 1 : T - 1;
            const int kc = 2 * (N - 1 - t) + (l16 & 1);
            const int lane_kept = -((path >> (T - 1 - t)) & 1);   // as a bit mask
            // the loads in two groups: the pivot blocks' rows and columns, then (their registers
            // free again) the undecided rows
            E wa0[T], wa1[T], wb0[T], wb1[T], ca[T], cb[T];
#pragma unroll
            for (int k = 0; k < T; ++k) {
                const E* p = A0 + 2 * (N - 1 - k) * w;
                wa0[k] = load_reg(&p[l16]);
                wa1[k] = load_reg(&p[kc]);
                wb0[k] = load_reg(&p[w + l16]);
                wb1[k] = load_reg(&p[w + kc]);
            }
#pragma unroll
            for (int k = 0; k < T; ++k) {
                const E* p = A0 + l16 * w + 2 * (N - 1 - k);
                ca[k] = load_reg(&p[0]);
                cb[k] = load_reg(&p[1]);
            }
            __builtin_amdgcn_sched_barrier(0);
            top_xnor_pivots<0>(lane_kept, wa0, wa1, wb0, wb1, mk);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < R0; ++i) M[i] = load_reg(&A0[i * w + l16]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < T; ++k) {
                const int in = -((path >> (T - 1 - k)) & 1);
                ca[k] = keep_if(in, ca[k]);
                cb[k] = keep_if(in, cb[k]);
            }
            multipliers2<0, 1>(ca, cb, wa1, wb1);
#pragma unroll
            for (int k = 0; k < T; ++k) {
                sub_rows<0>(M, ca[k], wa0[k]);
                sub_rows<0>(M, cb[k], wb0[k]);
            }
        }
    }

    // c[k2] -= c[K] (entry k2 of the scaled pivot row K), K < k2
    template <int K, int K2>
    __device__ __forceinline__ void multipliers(E (&c)[T], const E (&w1)[T])
    {
        if constexpr (K2 < T) {
            c[K2] = F::upd(c[K2], c[K], row_bcast<K2>(w1[K]));
            multipliers<K, K2 + 1>(c, w1);
        } else if constexpr (K + 2 < T) {
            multipliers<K + 1, K + 2>(c, w1);
        }
    }

    // the same for pivot blocks (two multipliers a block)
    template <int K, int K2>
    __device__ __forceinline__ void multipliers2(E (&ca)[T], E (&cb)[T], const E (&wa1)[T], const E (&wb1)[T])
    {
        if constexpr (K2 < T) {
            ca[K2] = F::upd(F::upd(ca[K2], ca[K], row_bcast<2 * K2>(wa1[K])), cb[K], row_bcast<2 * K2>(wb1[K]));
            cb[K2] = F::upd(F::upd(cb[K2], ca[K], row_bcast<2 * K2 + 1>(wa1[K])), cb[K],
                            row_bcast<2 * K2 + 1>(wb1[K]));
            multipliers2<K, K2 + 1>(ca, cb, wa1, wb1);
        } else if constexpr (K + 2 < T) {
            __builtin_amdgcn_sched_barrier(0);   // keep later broadcasts from being formed early (registers)
            multipliers2<K + 1, K + 2>(ca, cb, wa1, wb1);
        }
    }

    // M[i] -= (lane i of c) w
    template <int I>
    __device__ __forceinline__ void sub_rows(E (&M)[R0], E c, E w)
    {
        if constexpr (I < R0) {
            if constexpr (F::kComplex) {
                row_sub_lanes<I>(M[I], M[I + 1], M[I + 2], M[I + 3], c, w);
                sub_rows<I + 4>(M, c, w);
            } else {
                row_sub_lanes<I>(M[I], M[I + 1], M[I + 2], M[I + 3], M[I + 4], M[I + 5], M[I + 6], M[I + 7], c, w);
                sub_rows<I + 8>(M, c, w);
            }
        }
    }

    // subtract the contributions of the pivots J .. K-1 from a row (two registers)
    template <int J, int K>
    __device__ __forceinline__ void apply_xor(E& a0, E& a1, const E (&w0)[T], const E (&w1)[T])
    {
        if constexpr (J < K) {
            const E c = row_bcast<J>(a1);
            a0 = F::upd(a0, c, w0[J]);
            if constexpr (J + 1 < T) a1 = F::upd(a1, c, w1[J]);
            apply_xor<J + 1, K>(a0, a1, w0, w1);
        }
    }

    // kept row K (from the input) to its scaled pivot row, K upwards
    template <int K>
    __device__ __forceinline__ void top_xor_pivots(E (&w0)[T], E (&w1)[T], E& mk)
    {
        if constexpr (K < T) {
            constexpr int low = T - 1 - K;
            E a0 = w0[K], a1 = w1[K];
            apply_xor<0, K>(a0, a1, w0, w1);
            const E pv = row_bcast<K>(a1);
            mk = F::bmul(mk, pv, 0);
            // written by the first of the paths that share this node
            if (wr && (path & ((1 << low) - 1)) == 0) ob[(int64_t(2) << K) - 2 + (path >> low)] = mk;
            chk += F::fincheck(mk);
            const typename F::R r = F::recip(pv);
            w0[K] = F::rowscale(a0, r);
            w1[K] = F::rowscale(a1, r);
            top_xor_pivots<K + 1>(w0, w1, mk);
        }
    }

    // subtract the contributions of the pivot blocks J .. K-1 from a row (two registers)
    template <int J, int K>
    __device__ __forceinline__ void apply_xnor(E& a0, E& a1, const E (&wa0)[T], const E (&wa1)[T], const E (&wb0)[T],
                                               const E (&wb1)[T])
    {
        if constexpr (J < K) {
            const E c0 = row_bcast<2 * J>(a1), c1 = row_bcast<2 * J + 1>(a1);
            a0 = F::upd(F::upd(a0, c0, wa0[J]), c1, wb0[J]);
            if constexpr (J + 1 < T) a1 = F::upd(F::upd(a1, c0, wa1[J]), c1, wb1[J]);
            apply_xnor<J + 1, K>(a0, a1, wa0, wa1, wb0, wb1);
        }
    }

    // put 1 where c holds (and v is zero)
    static __device__ __forceinline__ void add_unit(double& v, bool c) { v += unit_if(c); }
    static __device__ __forceinline__ void add_unit(cd& v, bool c) { v.x += unit_if(c); }

    template <int K>
    __device__ __forceinline__ void top_xnor_pivots(int lane_kept, E (&wa0)[T], E (&wa1)[T],
                                                    E (&wb0)[T], E (&wb1)[T], E& mk)
    {
        if constexpr (K < T) {
            // a block left out: unit rows, so that its pivot block is the identity and changes nothing
            const int kept = -((path >> (T - 1 - K)) & 1);
            E a0 = keep_if(kept, wa0[K]), a1 = keep_if(kept & lane_kept, wa1[K]);
            E b0 = keep_if(kept, wb0[K]), b1 = keep_if(kept & lane_kept, wb1[K]);
            add_unit(a1, !kept && l16 == 2 * K);
            add_unit(b1, !kept && l16 == 2 * K + 1);
            apply_xnor<0, K>(a0, a1, wa0, wa1, wb0, wb1);
            apply_xnor<0, K>(b0, b1, wa0, wa1, wb0, wb1);
            const E a00 = row_bcast<2 * K>(a1), a01 = row_bcast<2 * K + 1>(a1);
            const E a10 = row_bcast<2 * K>(b1), a11 = row_bcast<2 * K + 1>(b1);
            const E det = F::det2(a00, a01, a10, a11);
            const typename F::R r = F::recip(det);
            wa0[K] = F::rowscale(F::upd(F::bmul(a0, a11, 0), a01, b0), r);
            wb0[K] = F::rowscale(F::upd(F::bmul(b0, a00, 0), a10, a0), r);
            wa1[K] = F::rowscale(F::upd(F::bmul(a1, a11, 0), a01, b1), r);
            wb1[K] = F::rowscale(F::upd(F::bmul(b1, a00, 0), a10, a1), r);
            if (kept) mk = F::bmul(mk, det, 0);
            chk += F::fincheck(mk);
            top_xnor_pivots<K + 1>(lane_kept, wa0, wa1, wb0, wb1, mk);
        }
    }

    // ---------------------------------------------------------------- row phase
    // XOR: the pivots of both children of an order-m node, their reciprocals and the
    // children's minors, in lanes m - 2 and m - 1 (one reciprocal for both).
    template <int m>
    __device__ __forceinline__ void pivots(const E (&M)[m], E mk, E& mkd, typename F::R& r)
    {
        const E d = l16 == m - 1 ? M[m - 1] : M[m - 2];
        mkd = F::bmul(mk, d, 0);
        r = F::recip(d);
    }

    // Keep the minors of the two children (lanes m - 2 and m - 1) in this unit's slots `at`,
    // `at` + 1; the other lanes write to a place of their own that nobody reads, which costs
    // less than masking them.
    template <int m>
    __device__ __forceinline__ void keep(int at, E mkd)
    {
        const bool own = l16 == m - 2 || l16 == m - 1;
        (own ? &sh.mn[kSlots * (int)(threadIdx.x >> 4) + l16 - (m - 2)] : &sh.dump[threadIdx.x])[at] = mkd;
    }

    // rows 0 .. n-1 of the child that keeps row P, in blocks of rows
    template <int P, int n, int m>
    __device__ __forceinline__ void child_rows(E (&M)[m], E (&C)[m - 2], E w)
    {
        if constexpr (n == 6 && !F::kComplex) {
            row_child<P>(C[0], C[1], C[2], C[3], C[4], C[5], M[0], M[1], M[2], M[3], M[4], M[5], w);
        } else if constexpr (n >= 4) {
            row_child<P>(C[n - 4], C[n - 3], C[n - 2], C[n - 1], M[n - 4], M[n - 3], M[n - 2], M[n - 1], w);
            child_rows<P, n - 4>(M, C, w);
        } else if constexpr (n > 0) {
            row_child<P>(C[n - 2], C[n - 1], M[n - 2], M[n - 1], w);
            child_rows<P, n - 2>(M, C, w);
        }
    }

    // the same in place
    template <int P, int n, int m>
    __device__ __forceinline__ void elim_rows(E (&M)[m], E w)
    {
        if constexpr (n == 8 && !F::kComplex) {
            row_elim<P>(M[0], M[1], M[2], M[3], M[4], M[5], M[6], M[7], w);
        } else if constexpr (n >= 6 && n != 8) {
            row_elim<P>(M[n - 6], M[n - 5], M[n - 4], M[n - 3], M[n - 2], M[n - 1], w);
            elim_rows<P, n - 6>(M, w);
        } else if constexpr (n >= 4) {
            row_elim<P>(M[n - 4], M[n - 3], M[n - 2], M[n - 1], w);
            elim_rows<P, n - 4>(M, w);
        } else if constexpr (n > 0) {
            row_elim<P>(M[n - 2], M[n - 1], w);
        }
    }

    // XOR: the child that keeps row m - 2 (rd: the reciprocals of pivots()).  Its last rows
    // come first and its own pivots right after them, so that their chain of dependent
    // operations runs beside the other rows' updates.
    template <int m>
    __device__ __forceinline__ void child_xor(E (&M)[m], E (&C)[m - 2], typename F::R rd, E mk, E& cmkd,
                                              typename F::R& crd)
    {
        constexpr int mc = m - 2, P = mc;
        const E w = F::rowscale(M[P], row_bcast<P>(rd));
        row_child<P>(C[mc - 2], C[mc - 1], M[mc - 2], M[mc - 1], w);
        if constexpr (mc > 8) pivots<mc>(C, mk, cmkd, crd);
        child_rows<P, mc - 2>(M, C, w);
    }

    // The child that keeps row m - 1, in place (the node is not needed any more).
    template <int m>
    __device__ __forceinline__ void last_child_xor(E (&M)[m], typename F::R rd, E mk, E& cmkd, typename F::R& crd)
    {
        constexpr int mc = m - 2, P = m - 1;
        E w = F::rowscale(M[P], row_bcast<P>(rd));
        if constexpr (F::kComplex)
            row_elim_first<P>(M[mc - 2], M[mc - 1], w, unit_if(l16 != P));
        else
            row_elim<P>(M[mc - 2], M[mc - 1], w);
        if constexpr (mc > 8) pivots<mc>(reinterpret_cast<E(&)[mc]>(M), mk, cmkd, crd);
        elim_rows<P, mc - 2>(M, w);
    }

    // XNOR: rows 0 .. n-1 of the child that keeps both rows
    template <int n, int m>
    __device__ __forceinline__ void child2_rows(const E (&M)[m], E (&C)[m - 2], E w0, E w1)
    {
        constexpr int P = m - 2;
        if constexpr (n >= 4) {
            row_child2<P>(C[n - 4], C[n - 3], C[n - 2], C[n - 1], M[n - 4], M[n - 3], M[n - 2], M[n - 1], w0, w1);
            child2_rows<n - 4>(M, C, w0, w1);
        } else if constexpr (n > 0) {
            row_child2<P>(C[n - 2], C[n - 1], M[n - 2], M[n - 1], w0, w1);
        }
    }

    // XNOR: the child that keeps both rows; its minor.
    template <int m>
    __device__ __forceinline__ E child_xnor(const E (&M)[m], E (&C)[m - 2], E mk)
    {
        constexpr int mc = m - 2;
        E a00, a01, a10, a11;
        row_block_after<mc>(M[mc], M[mc + 1], a00, a01, a10, a11);
        const E det = F::det2(a00, a01, a10, a11);
        const typename F::R r = F::recip(det);
        const E w0 = F::rowscale(F::upd(F::bmul(M[mc], a11, 0), a01, M[mc + 1]), r);
        const E w1 = F::rowscale(F::upd(F::bmul(M[mc + 1], a00, 0), a10, M[mc]), r);
        child2_rows<mc>(M, C, w0, w1);
        return F::bmul(mk, det, 0);
    }

    // The subtree of an order-m node (destroyed) down to order 8.  t: its place among the
    // phase's nodes of its depth; LV: levels below the phase's root; mkd, rd: its pivots()
    // (XOR above order 8).
    template <int m, int LV>
    __device__ __forceinline__ void node(E (&M)[m], E mk, E mkd, typename F::R rd, int t)
    {
        if constexpr (m == 8) {
            const int q = (int)(threadIdx.x >> 4) * NPR + t;
            if (l16 < 8) {
                E* d = &sh.node[q * kPS + l16];
#pragma unroll
                for (int i = 0; i < 8; ++i) d[i * 8] = M[i];
            }
            if constexpr (MODE == kXnor || LV == 0) {
                const bool own = l16 == 0;
                (own ? &sh.mn[kSlots * (int)(threadIdx.x >> 4) + kLast] : &sh.dump[threadIdx.x])[t] = mk;
                chk += F::fincheck(mk);
            }
        } else if constexpr (MODE == kXor) {
            keep<m>((2 << LV) - 2 + 2 * t, mkd);
            E cmkd = F::zero();
            typename F::R crd{};
            {
                E C[m - 2];
                const E mk0 = row_bcast<m - 2>(mkd);
                child_xor(M, C, rd, mk0, cmkd, crd);
                node<m - 2, LV + 1>(C, mk0, cmkd, crd, 2 * t);
            }
            const E mk1 = row_bcast<m - 1>(mkd);
            last_child_xor(M, rd, mk1, cmkd, crd);
            node<m - 2, LV + 1>(reinterpret_cast<E(&)[m - 2]>(M), mk1, cmkd, crd, 2 * t + 1);
        } else {
            {
                E C[m - 2];
                const E mc = child_xnor(M, C, mk);
                node<m - 2, LV + 1>(C, mc, mkd, rd, 2 * t + 1);
            }
            // the block left out: the leading part, minor unchanged
            node<m - 2, LV + 1>(reinterpret_cast<E(&)[m - 2]>(M), mk, mkd, rd, 2 * t);
        }
    }

    // ---------------------------------------------------------------- lane phase
    // k[j] = a[j] - c w[j] (F::upd), the dependent halves of the complex updates apart
    template <int n>
    static __device__ __forceinline__ void lane_row(double* k, const double* a, double c, const double* w)
    {
#pragma unroll
        for (int j = 0; j < n; ++j) k[j] = fma(-c, w[j], a[j]);
    }
    template <int n>
    static __device__ __forceinline__ void lane_row(cd* k, const cd* a, cd c, const cd* w)
    {
#pragma unroll
        for (int j = 0; j < n; ++j) {
            k[j].x = fma(c.y, w[j].y, a[j].x);
            k[j].y = fma(-c.y, w[j].x, a[j].y);
        }
#pragma unroll
        for (int j = 0; j < n; ++j) {
            k[j].x = fma(-c.x, w[j].x, k[j].x);
            k[j].y = fma(-c.x, w[j].y, k[j].y);
        }
    }

    // A lane's order-m node: its minors below, leaves (and, XOR, the depths above) in order.
    template <int m>
    __device__ __forceinline__ void leaf_levels(const E (&C)[m][m], E mk, E* lv8, E* lv4, E* lv2, int t)
    {
        constexpr int mc = m - 2;
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            E mk2, K[mc > 0 ? mc : 1][mc > 0 ? mc : 1];
            if constexpr (MODE == kXor) {
                const E pv = C[mc + a][mc + a];
                mk2 = F::bmul(mk, pv, 0);
                if constexpr (mc > 0) {
                    const typename F::R r = F::recip(pv);
                    E w[mc];
#pragma unroll
                    for (int j = 0; j < mc; ++j) w[j] = F::rowscale(C[mc + a][j], r);
#pragma unroll
                    for (int i = 0; i < mc; ++i) lane_row<mc>(K[i], C[i], C[i][mc + a], w);
                }
            } else if (a == 0) {
                mk2 = mk;
                if constexpr (mc > 0) {
#pragma unroll
                    for (int i = 0; i < mc; ++i)
#pragma unroll
                        for (int j = 0; j < mc; ++j) K[i][j] = C[i][j];
                }
            } else {
                const E a00 = C[mc][mc], a01 = C[mc][mc + 1], a10 = C[mc + 1][mc], a11 = C[mc + 1][mc + 1];
                const E det = F::det2(a00, a01, a10, a11);
                mk2 = F::bmul(mk, det, 0);
                if constexpr (mc > 0) {
                    const typename F::R r = F::recip(det);
                    E w0[mc], w1[mc];
#pragma unroll
                    for (int j = 0; j < mc; ++j) {
                        w0[j] = F::rowscale(F::upd(F::bmul(C[mc][j], a11, 0), a01, C[mc + 1][j]), r);
                        w1[j] = F::rowscale(F::upd(F::bmul(C[mc + 1][j], a00, 0), a10, C[mc][j]), r);
                    }
#pragma unroll
                    for (int i = 0; i < mc; ++i) {
                        lane_row<mc>(K[i], C[i], C[i][mc], w0);
                        lane_row<mc>(K[i], K[i], C[i][mc + 1], w1);
                    }
                }
            }
            if constexpr (MODE == kXor) chk_lane += F::fincheck(mk2);
            if constexpr (m == 6) {
                lv2[a] = mk2;
                leaf_levels<4>(K, mk2, lv8, lv4, lv2, a);
            } else if constexpr (m == 4) {
                lv4[2 * t + a] = mk2;
                leaf_levels<2>(K, mk2, lv8, lv4, lv2, 2 * t + a);
            } else {
                lv8[2 * t + a] = mk2;
                if constexpr (MODE == kXnor) chk_lane += F::fincheck(mk2);
            }
        }
    }

    // the leading 6 x 6 part of an order-8 node
    static __device__ __forceinline__ void load_leading(const E* P, E (&C)[6][6])
    {
#pragma unroll
        for (int i = 0; i < 6; ++i)
#pragma unroll
            for (int j = 0; j < 6; ++j) C[i][j] = load_reg(&P[i * 8 + j]);
        __builtin_amdgcn_sched_barrier(0);
    }

    double chk_lane = 0.0;   // of the minors formed in the lane phase (lanes grouped by parent)

    // The staged minors (W a lane, W + 1 apart) to a depth's place in the output, 64 at a time:
    // all reads, then all stores.
    template <int W, int IT = 0>
    __device__ __forceinline__ void flush(const E* st, E* out, int64_t u0, int64_t units, int h, int lane)
    {
        constexpr int seg = 2 * NPR * W;              // contiguous minors of a unit
        constexpr int64_t nout = MODE == kXor ? (int64_t(2) << N) - 2 : int64_t(1) << N;
        if constexpr (IT * 64 < 4 * seg) {
            const int e = IT * 64 + lane;
            const E v = load_reg(&st[IT * (64 / W) * (W + 1) + (lane / W) * (W + 1) + lane % W]);
            flush<W, IT + 1>(st, out, u0, units, h, lane);
            // with whole wavefronts in a unit the unit is known at compile time
            const int r = seg >= 64 ? IT * 64 / seg : e / seg;
            const int64_t u = u0 + r;
            if ((4 * seg >= 64 || e < 4 * seg) && (T >= 2 || u < units)) {
                E* o = out + ((u >> T) * nout + ((u & ((1 << T) - 1)) * halves(N) + h) * seg);
                o[e - r * seg] = v;
            }
        } else {
            __builtin_amdgcn_sched_barrier(0);
        }
    }

    // The order-8 nodes in LDS to their minors: lane 2 q + a takes child a of node q.  `u0`:
    // the unit of row 0, `units`: their number, `h`: which half of the units' nodes.
    __device__ __forceinline__ void lanes(E* out, int64_t u0, int64_t units, int h)
    {
        constexpr int per = 2 * NPR;               // lanes of a unit
        constexpr int64_t nout = MODE == kXor ? (int64_t(2) << N) - 2 : int64_t(1) << N;
        // (the addresses formed anew cost the real kernels, which have registers to spare, 6%)
        const int lane = F::kComplex ? lane_here() : (int)threadIdx.x, l16 = lane & 15;
        const int q = lane >> 1, a = lane & 1;
        E lv8[8], lv4[4], lv2[2], m6;
        const bool act = 4 * per == 64 || lane < 4 * per;
        wave_sync();
        if constexpr (MODE == kXor && LV8 > 0) {
            // the minors of the row phase: slot 2^j - 2 + t is place t of level j below the
            // phase's root, the last two slots (two phases a unit) the root's own level
            const int j = 31 - __clz(l16 + 2), t = l16 + 2 - (1 << j);
            const bool top2 = halves(N) == 2 && l16 >= kSlots - 2;
            const int d = top2 ? T + 1 : T + halves(N) - 1 + j;
            const int root = halves(N) == 2 ? 2 * path + h : path;
            const int p = top2 ? 2 * path + l16 - (kSlots - 2) : (root << j) + t;
            if (valid && (top2 ? h == 0 : l16 < (2 << LV8) - 2)) {
                const E v = sh.mn[lane];
                ob[(int64_t(1) << d) - 2 + p] = v;
                chk += F::fincheck(v);
            }
        }
        if (act) {
            const E* P = &sh.node[q * kPS];
            E C[6][6];
            // every read first: 49 to 63 in flight, one LDS round trip
            const E mq = load_reg(&sh.mn[kSlots * (q / NPR) + kLast + q % NPR]);
            if constexpr (MODE == kXor) {
                const E pv = load_reg(&P[(6 + a) * 8 + 6 + a]);
                E w[6], c[6];
#pragma unroll
                for (int j = 0; j < 6; ++j) w[j] = load_reg(&P[(6 + a) * 8 + j]);
#pragma unroll
                for (int i = 0; i < 6; ++i) c[i] = load_reg(&P[i * 8 + 6 + a]);
                load_leading(P, C);
                m6 = F::bmul(mq, pv, 0);
                const typename F::R r = F::recip(pv);
#pragma unroll
                for (int j = 0; j < 6; ++j) w[j] = F::rowscale(w[j], r);
#pragma unroll
                for (int i = 0; i < 6; ++i) lane_row<6>(C[i], C[i], c[i], w);
            } else {
                // both children in one instruction stream: the one that leaves the block out
                // subtracts zero times zero
                const E a00 = load_reg(&P[6 * 8 + 6]), a01 = load_reg(&P[6 * 8 + 7]), a10 = load_reg(&P[7 * 8 + 6]), a11 = load_reg(&P[7 * 8 + 7]);
                E p0[6], p1[6], c0[6], c1[6];
#pragma unroll
                for (int j = 0; j < 6; ++j) {
                    p0[j] = load_reg(&P[6 * 8 + j]);
                    p1[j] = load_reg(&P[7 * 8 + j]);
                }
                const E det = F::det2(a00, a01, a10, a11);
                m6 = a ? F::bmul(mq, det, 0) : mq;
                const typename F::R r = F::recip(det);
                load_leading(P, C);
#pragma unroll
                for (int i = 0; i < 6; ++i) {
                    c0[i] = load_reg(&P[i * 8 + 6]);
                    c1[i] = load_reg(&P[i * 8 + 7]);
                }
                const int in = -a;
#pragma unroll
                for (int j = 0; j < 6; ++j) {
                    const E t = p0[j];
                    p0[j] = keep_if(in, F::rowscale(F::upd(F::bmul(t, a11, 0), a01, p1[j]), r));
                    p1[j] = keep_if(in, F::rowscale(F::upd(F::bmul(p1[j], a00, 0), a10, t), r));
                }
#pragma unroll
                for (int i = 0; i < 6; ++i) {
                    lane_row<6>(C[i], C[i], keep_if(in, c0[i]), p0);
                    lane_row<6>(C[i], C[i], keep_if(in, c1[i]), p1);
                }
            }
            chk_lane += F::fincheck(m6);
            leaf_levels<6>(C, m6, lv8, lv4, lv2, 0);
        }
        wave_sync();                               // every lane has read its node
        E* st8 = sh.node;                          // 9 entries a lane
        E* st4 = sh.node + 64 * 9;                 // 5 entries a lane
        if (act) {
#pragma unroll
            for (int c = 0; c < 8; ++c) st8[lane * 9 + c] = lv8[c];
            if constexpr (MODE == kXor) {
#pragma unroll
                for (int c = 0; c < 4; ++c) st4[lane * 5 + c] = lv4[c];
                const int64_t u = u0 + lane / per;
                if (T >= 2 || u < units) {
                    const int64_t b = u >> T;
                    // this lane's node's path: the unit's, the half, its place
                    const int s = (((int)(u & ((1 << T) - 1)) * halves(N) + h) * per) + lane % per;
                    E* o = out + b * nout;
                    o[(int64_t(1) << (N - 3)) - 2 + s] = m6;
                    E* o2 = o + (int64_t(1) << (N - 2)) - 2 + 2 * s;
                    o2[0] = lv2[0];
                    o2[1] = lv2[1];
                }
            }
        }
        wave_sync();
        static_assert(64 * 14 <= kParents * kPS, "the staged minors fit the nodes' place");
        if constexpr (MODE == kXor) {
            flush<8>(st8, out + ((int64_t(1) << N) - 2), u0, units, h, lane);
            flush<4>(st4, out + ((int64_t(1) << (N - 1)) - 2), u0, units, h, lane);
        } else {
            flush<8>(st8, out, u0, units, h, lane);
        }
        wave_sync();                               // before the next nodes overwrite the stage
    }
};

// Wavefront blockIdx.x takes `per_wave` consecutive units (a multiple of 4 when T >= 2, else
// 4).  info: written directly if it holds all units of its matrices (shared == 0), else
// lowered with an atomic from the zero that xor_info_kernel wrote.
template <class F, int N, int MODE, int WAVES>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(WAVES))) void xor_row_kernel(
    const typename F::E* __restrict__ A, typename F::E* __restrict__ out, int32_t* __restrict__ info, int64_t units,
    int per_wave, int shared)
{
    using E = typename F::E;
    using U = Unit<F, N, MODE>;
    constexpr int T = U::T, w = 2 * N;
    constexpr int64_t nout = MODE == kXor ? (int64_t(2) << N) - 2 : int64_t(1) << N;
    constexpr int LPM = T >= 2 ? 64 : 16 << T;     // lanes that work on one matrix
    __shared__ Lds<F> sh;
    const int lane = threadIdx.x;
    const int64_t first = (int64_t)blockIdx.x * per_wave;
    U un(sh);
    un.l16 = lane & 15;
    bool finite = true;
    for (int64_t u0 = first; u0 < first + per_wave && u0 < units; u0 += 4) {
        const int64_t u = u0 + (lane >> 4);
        const bool valid = T >= 2 || u < units;   // T >= 2: whole groups of four
        const int64_t uc = valid ? u : units - 1;
        const int64_t b = uc >> T;
        const E* A0 = A + b * (w * w);
        un.path = (int)(uc & ((1 << T) - 1));
        un.ob = out + b * nout;
        un.valid = valid;
        un.wr = valid && un.l16 == 0;
        if (u0 == first || (u0 & ((1 << T) - 1)) == 0 || T < 2) {   // a matrix begins
            bool fin = true;
            for (int e = lane % LPM; e < w * w; e += LPM) fin = fin && F::in_finite(A0[e]);
            const uint64_t bad = ballot(!fin);
            finite = ((bad >> (lane / LPM * LPM)) & (LPM == 64 ? ~0ull : (1ull << (LPM & 63)) - 1)) == 0;
            un.chk = un.chk_lane = 0.0;
        }
        E M[U::R0], mk = F::one();
        // a non-finite input makes every minor NaN
        if (!finite) F::store_nan(&mk, nullptr, 0, false);
        un.top(A0, M, mk);
        if constexpr (MODE == kXnor) un.chk += F::fincheck(mk);
        if constexpr (halves(N) == 2) {
            E mkd = F::zero();
            typename F::R rd{};
            if constexpr (MODE == kXor) {
                un.template pivots<16>(M, mk, mkd, rd);
                un.template keep<16>(kSlots - 2, mkd);
            }
#pragma unroll 1
            for (int k = 0; k < 2; ++k) {
                // XNOR: the child that keeps the block first (the other one is formed in place)
                const int h = MODE == kXnor ? 1 - k : k;
                E cmkd = F::zero();
                typename F::R crd{};
                if (k == 0) {
                    E C[14];
                    if constexpr (MODE == kXor) {
                        const E mk0 = row_bcast<14>(mkd);
                        un.child_xor(M, C, rd, mk0, cmkd, crd);
                        un.template node<14, 0>(C, mk0, cmkd, crd, 0);
                    } else {
                        const E mc = un.child_xnor(M, C, mk);
                        un.template node<14, 0>(C, mc, cmkd, crd, 0);
                    }
                } else if constexpr (MODE == kXor) {
                    const E mk1 = row_bcast<15>(mkd);
                    un.last_child_xor(M, rd, mk1, cmkd, crd);
                    un.template node<14, 0>(reinterpret_cast<E(&)[14]>(M), mk1, cmkd, crd, 0);
                } else {
                    un.template node<14, 0>(reinterpret_cast<E(&)[14]>(M), mk, cmkd, crd, 0);
                }
                un.lanes(out, u0, units, h);
            }
        } else {
            E mkd = F::zero();
            typename F::R rd{};
            if constexpr (MODE == kXor && U::R0 > 8) un.template pivots<U::R0>(M, mk, mkd, rd);
            un.template node<U::R0, 0>(M, mk, mkd, rd, 0);
            un.lanes(out, u0, units, 0);
        }
        // the last units of a matrix here: its info
        const bool last = T < 2 || u0 + 4 >= first + per_wave || ((u0 + 4) & ((1 << T) - 1)) == 0;
        if (info && last) {
            const uint64_t rows = ballot(un.chk != 0.0 || un.chk != un.chk);
            const uint64_t lns = ballot(un.chk_lane != 0.0 || un.chk_lane != un.chk_lane);
            constexpr int per = 2 * U::NPR, lpm = T >= 2 ? 64 : per << T;   // lane phase's lanes of a matrix
            const int g = lane / LPM;
            const uint64_t mr = LPM == 64 ? ~0ull : ((1ull << (LPM & 63)) - 1) << (g * LPM & 63);
            const uint64_t ml = lpm == 64 ? ~0ull : ((1ull << (lpm & 63)) - 1) << (g * lpm & 63);
            const int code = !finite ? -2 : ((rows & mr) | (lns & ml)) ? -3 : 0;
            if (valid && lane % LPM == 0) {
                if (!shared)
                    info[b] = code;
                else if (code)
                    atomicMin(&info[b], code);
            }
        }
    }
}

}  // namespace xrow
}  // namespace apm
