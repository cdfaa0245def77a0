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
// Why order 8: below it a row of 16 lanes is less than half used, while a lane cannot hold
// more than an order-6 complex node (144 registers) and its children.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "apm_device.h"
#include "apm_kernels.h"

namespace apm {
namespace xrow {

constexpr int kXor = 0, kXnor = 1;
constexpr int kParents = 32;        // order-8 nodes in LDS at a time
constexpr int kPS = 65;             // their stride in elements

__host__ __device__ constexpr int top_levels(int N) { return N > 8 ? N - 8 : 0; }
// order-8 nodes of a unit per lane phase, and lane phases per unit
__host__ __device__ constexpr int parents(int N) { return N >= 7 ? 8 : 1 << (N - 4); }
__host__ __device__ constexpr int halves(int N) { return N >= 8 ? 2 : 1; }

template <class F>
struct Lds {
    typename F::E node[kParents * kPS];
    typename F::E mn[kParents];     // their minors
};

// c - col * w with col = lane P's value of column entries src
template <class F, int P>
__device__ __forceinline__ typename F::E row_upd(typename F::E a, typename F::E src, typename F::E w)
{
    return F::upd(a, row_bcast<P>(src), w);
}

template <class F, int N, int MODE>
struct Unit {
    using E = typename F::E;
    static constexpr int T = top_levels(N);
    static constexpr int R0 = 2 * (N - T);
    static constexpr int NPR = parents(N);
    static constexpr int D8 = N - 4;             // depth of the order-8 nodes

    Lds<F>& sh;
    E* ob;            // this row's matrix's output
    int path;         // its choices of the top levels
    int l16;          // lane in the row
    bool wr;          // the lane that writes the row's minors
    double chk = 0.0;

    __device__ Unit(Lds<F>& s) : sh(s) {}

    // a minor of depth d (path p below the root)
    __device__ __forceinline__ void record(int d, int p, E mk)
    {
        if constexpr (MODE == kXor) {
            if (wr) ob[(int64_t(1) << d) - 2 + p] = mk;
        }
        chk += F::fincheck(mk);
    }

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
            E w0[T], w1[T];
            top_xor_pivots<0>(A0, kc, w0, w1, mk);
#pragma unroll
            for (int i = 0; i < R0; ++i) {
                E a0 = A0[i * w + l16], a1 = A0[i * w + kc];
                apply_xor<0, T>(a0, a1, w0, w1);
                M[i] = a0;
            }
        } else {
            // lane 2 t + r's kept column: column r of block N - 1 - t (zero if left out)
            const int t = l16 < 2 * T ? l16 >> 1 : T - 1;
            const int kc = 2 * (N - 1 - t) + (l16 & 1);
            const bool kept = (path >> (T - 1 - t)) & 1;
            E wa0[T], wa1[T], wb0[T], wb1[T];
            top_xnor_pivots<0>(A0, kc, kept, wa0, wa1, wb0, wb1, mk);
#pragma unroll
            for (int i = 0; i < R0; ++i) {
                E a0 = A0[i * w + l16], a1 = A0[i * w + kc];
                if (!kept) a1 = F::zero();
                apply_xnor<0, T>(a0, a1, wa0, wa1, wb0, wb1);
                M[i] = a0;
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

    template <int K>
    __device__ __forceinline__ void top_xor_pivots(const E* A0, int kc, E (&w0)[T], E (&w1)[T], E& mk)
    {
        if constexpr (K < T) {
            constexpr int low = T - 1 - K;
            const int row = 2 * (N - 1 - K) + ((path >> low) & 1);
            E a0 = A0[row * (2 * N) + l16], a1 = A0[row * (2 * N) + kc];
            apply_xor<0, K>(a0, a1, w0, w1);
            const E pv = row_bcast<K>(a1);
            mk = F::bmul(mk, pv, 0);
            // written by the first of the paths that share this node
            if (wr && (path & ((1 << low) - 1)) == 0) ob[(int64_t(2) << K) - 2 + (path >> low)] = mk;
            chk += F::fincheck(mk);
            const typename F::R r = F::recip(pv);
            w0[K] = F::rowscale(a0, r);
            w1[K] = F::rowscale(a1, r);
            top_xor_pivots<K + 1>(A0, kc, w0, w1, mk);
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

    template <int K>
    __device__ __forceinline__ void top_xnor_pivots(const E* A0, int kc, bool lane_kept, E (&wa0)[T], E (&wa1)[T],
                                                    E (&wb0)[T], E (&wb1)[T], E& mk)
    {
        if constexpr (K < T) {
            constexpr int w = 2 * N, ra = 2 * (N - 1 - K);
            const bool kept = (path >> (T - 1 - K)) & 1;
            E a0 = A0[ra * w + l16], a1 = A0[ra * w + kc];
            E b0 = A0[(ra + 1) * w + l16], b1 = A0[(ra + 1) * w + kc];
            if (!lane_kept) a1 = b1 = F::zero();
            if (!kept) {   // unit rows: the pivot block is the identity and changes nothing
                a0 = a1 = b0 = b1 = F::zero();
                if (l16 == 2 * K) a1 = F::one();
                if (l16 == 2 * K + 1) b1 = F::one();
            }
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
            top_xnor_pivots<K + 1>(A0, kc, lane_kept, wa0, wa1, wb0, wb1, mk);
        }
    }

    // ---------------------------------------------------------------- row phase
    // The child of the order-m node M that keeps row m - 2 + A (XOR) or both (XNOR, A = 1).
    template <int m, int A>
    __device__ __forceinline__ void child(const E (&M)[m], E (&C)[m - 2], E mk, E& mc_out)
    {
        constexpr int mc = m - 2;
        if constexpr (MODE == kXor) {
            const E pv = row_bcast<mc + A>(M[mc + A]);
            mc_out = F::bmul(mk, pv, 0);
            const E w = F::rowscale(M[mc + A], F::recip(pv));
#pragma unroll
            for (int i = 0; i < mc; ++i) C[i] = row_upd<F, mc + A>(M[i], M[i], w);
        } else {
            const E a00 = row_bcast<mc>(M[mc]), a01 = row_bcast<mc + 1>(M[mc]);
            const E a10 = row_bcast<mc>(M[mc + 1]), a11 = row_bcast<mc + 1>(M[mc + 1]);
            const E det = F::det2(a00, a01, a10, a11);
            mc_out = F::bmul(mk, det, 0);
            const typename F::R r = F::recip(det);
            const E w0 = F::rowscale(F::upd(F::bmul(M[mc], a11, 0), a01, M[mc + 1]), r);
            const E w1 = F::rowscale(F::upd(F::bmul(M[mc + 1], a00, 0), a10, M[mc]), r);
#pragma unroll
            for (int i = 0; i < mc; ++i) C[i] = row_upd<F, mc + 1>(row_upd<F, mc>(M[i], M[i], w0), M[i], w1);
        }
    }

    // Node of order m at path p (from the root); its low bits are the place among the phase's
    // order-8 nodes.
    template <int m>
    __device__ __forceinline__ void node(const E (&M)[m], E mk, int p, int t)
    {
        if constexpr (m == 8) {
            const int q = (int)(threadIdx.x >> 4) * NPR + (t & (NPR - 1));
            if (l16 < 8) {
                E* d = &sh.node[q * kPS + l16];
#pragma unroll
                for (int i = 0; i < 8; ++i) d[i * 8] = M[i];
            }
            if (l16 == 0) sh.mn[q] = mk;
        } else {
            constexpr int d = N - m / 2 + 1;     // the children's depth
            branch<m, 0, d>(M, mk, p, t);
            branch<m, 1, d>(M, mk, p, t);
        }
    }

    template <int m, int A, int D>
    __device__ __forceinline__ void branch(const E (&M)[m], E mk, int p, int t)
    {
        E C[m - 2], mc;
        if constexpr (MODE == kXnor && A == 0) {
#pragma unroll
            for (int i = 0; i < m - 2; ++i) C[i] = M[i];   // the leading part, minor unchanged
            mc = mk;
        } else {
            child<m, A>(M, C, mk, mc);
            record(D, 2 * p + A, mc);
        }
        node<m - 2>(C, mc, 2 * p + A, 2 * t + A);
    }

    // ---------------------------------------------------------------- lane phase
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
#pragma unroll
                    for (int j = 0; j < mc; ++j) {
                        const E wj = F::rowscale(C[mc + a][j], r);
#pragma unroll
                        for (int i = 0; i < mc; ++i) K[i][j] = F::upd(C[i][j], C[i][mc + a], wj);
                    }
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
#pragma unroll
                    for (int j = 0; j < mc; ++j) {
                        const E w0 = F::rowscale(F::upd(F::bmul(C[mc][j], a11, 0), a01, C[mc + 1][j]), r);
                        const E w1 = F::rowscale(F::upd(F::bmul(C[mc + 1][j], a00, 0), a10, C[mc][j]), r);
#pragma unroll
                        for (int i = 0; i < mc; ++i) K[i][j] = F::upd(F::upd(C[i][j], C[i][mc], w0), C[i][mc + 1], w1);
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

    double chk_lane = 0.0;   // of the minors formed in the lane phase (lanes grouped by parent)

    // The order-8 nodes in LDS to their minors: lane 2 q + a takes child a of node q.  `u0`:
    // the unit of row 0, `units`: their number, `h`: which half of the units' nodes.
    __device__ __forceinline__ void lanes(E* out, int64_t u0, int64_t units, int h)
    {
        constexpr int per = 2 * NPR;               // lanes of a unit
        constexpr int64_t nout = MODE == kXor ? (int64_t(2) << N) - 2 : int64_t(1) << N;
        const int lane = threadIdx.x;
        const int q = lane >> 1, a = lane & 1;
        E lv8[8], lv4[4], lv2[2], m6;
        const bool act = lane < 4 * per;
        wave_sync();
        if (act) {
            const E* P = &sh.node[q * kPS];
            E C[6][6];
            if constexpr (MODE == kXor) {
                const E pv = P[(6 + a) * 8 + 6 + a];
                m6 = F::bmul(sh.mn[q], pv, 0);
                const typename F::R r = F::recip(pv);
                E w[6];
#pragma unroll
                for (int j = 0; j < 6; ++j) w[j] = F::rowscale(P[(6 + a) * 8 + j], r);
#pragma unroll
                for (int i = 0; i < 6; ++i) {
                    const E c = P[i * 8 + 6 + a];
#pragma unroll
                    for (int j = 0; j < 6; ++j) C[i][j] = F::upd(P[i * 8 + j], c, w[j]);
                }
            } else {
                // both children in one instruction stream: the one that leaves the block out
                // subtracts zero times zero
                const E a00 = P[6 * 8 + 6], a01 = P[6 * 8 + 7], a10 = P[7 * 8 + 6], a11 = P[7 * 8 + 7];
                const E det = F::det2(a00, a01, a10, a11);
                m6 = a ? F::bmul(sh.mn[q], det, 0) : sh.mn[q];
                const typename F::R r = F::recip(det);
                E w0[6], w1[6];
#pragma unroll
                for (int j = 0; j < 6; ++j) {
                    const E p0 = P[6 * 8 + j], p1 = P[7 * 8 + j];
                    w0[j] = a ? F::rowscale(F::upd(F::bmul(p0, a11, 0), a01, p1), r) : F::zero();
                    w1[j] = a ? F::rowscale(F::upd(F::bmul(p1, a00, 0), a10, p0), r) : F::zero();
                }
#pragma unroll
                for (int i = 0; i < 6; ++i) {
                    const E c0 = a ? P[i * 8 + 6] : F::zero(), c1 = a ? P[i * 8 + 7] : F::zero();
#pragma unroll
                    for (int j = 0; j < 6; ++j) C[i][j] = F::upd(F::upd(P[i * 8 + j], c0, w0[j]), c1, w1[j]);
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
                if (u < units) {
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
        auto flush = [&](const E* st, int64_t base, auto width) {
            constexpr int W = decltype(width)::value;     // minors a lane
            constexpr int seg = per * W;                  // contiguous minors of a unit
#pragma unroll
            for (int it = 0; it < (4 * seg + 63) / 64; ++it) {
                const int e = it * 64 + lane;
                // with whole wavefronts in a unit the unit is known at compile time
                const int r = seg >= 64 ? it * 64 / seg : e / seg;
                const int64_t u = u0 + r;
                if (e < 4 * seg && u < units) {
                    const int64_t b = u >> T;
                    E* o = out + (b * nout + base + ((u & ((1 << T) - 1)) * halves(N) + h) * seg);
                    o[e - r * seg] = st[(e / W) * (W + 1) + e % W];
                }
            }
        };
        if constexpr (MODE == kXor) {
            flush(st8, (int64_t(1) << N) - 2, std::integral_constant<int, 8>{});
            flush(st4, (int64_t(1) << (N - 1)) - 2, std::integral_constant<int, 4>{});
        } else {
            flush(st8, 0, std::integral_constant<int, 8>{});
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
        const bool valid = u < units;
        const int64_t uc = valid ? u : units - 1;
        const int64_t b = uc >> T;
        const E* A0 = A + b * (w * w);
        un.path = (int)(uc & ((1 << T) - 1));
        un.ob = out + b * nout;
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
#pragma unroll 1
            for (int h = 0; h < 2; ++h) {
                if (h == 0)
                    un.template branch<U::R0, 0, T + 1>(M, mk, un.path, 0);
                else
                    un.template branch<U::R0, 1, T + 1>(M, mk, un.path, 0);
                un.lanes(out, u0, units, h);
            }
        } else {
            un.template node<U::R0>(M, mk, un.path, 0);
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
