// nand_row.h -- NAND minors (Sec. III) with the node matrices in registers, on gfx950, without
// pivot shifts.
//
// The ternary tree of xor.hip, with the mapping of xor_row.h: a node of order m <= 16 in a row
// of 16 lanes (lane j: column j), four units side by side in a wavefront, the order-8 nodes
// through LDS to one order-6 child per lane.  Every kept row's pivot is put to the tree's shift
// test, on the same row and column entries.  A shifted pivot needs its subtree corrected
// afterwards, which this kernel does not do: it marks the parts below (nand_parts.h), which the
// launches behind this one form again.
//
//   * A unit is a matrix, a choice (left out, first row, second row) for each of its T =
//     max(0, N - 8) last blocks and, from 8 blocks on, the choice of the block below them: one
//     wavefront per four units and that choice, so that launches of a few matrices spread out.
//   * Top phase: the kept rows are eliminated as in xor_row.h; a left-out block has a zero
//     pivot row.  The rows that are dropped are followed in the kept columns alone: their
//     entries there take part in the tests.
//   * Row phase: for each choice of the next block (a part each), two levels to 9 order-8 nodes a
//     unit, 36 in all (37 KB complex, the LDS of one wavefront per SIMD).
//   * Lane phase: two passes of 54 lanes (18 nodes, 3 children each); a lane's 27 leaves are
//     staged 9 at a time in the place of the nodes that have been read.
// Bound by fp64 issue of one wavefront per SIMD.  1024 complex matrices of 10 blocks 1.81 ms with
// one wavefront per matrix in LDS, 0.30 here (no part marked); 512 with a zero diagonal
// (throughout marked) 2.61 -> 0.78 ms with the launches behind.  One shifted matrix among 1000
// of 7 blocks 91 -> 76 us, 16000 with a zero diagonal 0.80 -> 0.80 ms.
#pragma once
#include "nand_parts.h"
#include "xor_row.h"

namespace apm {
namespace nrow {

using xrow::keep_if;

__host__ __device__ constexpr int pow3(int k) { return k <= 0 ? 1 : 3 * pow3(k - 1); }
constexpr int kNodes = 36;
constexpr int kPS = 65;

template <class F>
struct Lds {
    typename F::E node[kNodes * kPS];
    typename F::E mn[kNodes];
    typename F::E dump[64 + 9];
};

// largest of a non-negative value over each row of 16 lanes, in every lane
__device__ __forceinline__ double row_max(double v)
{
    v = dpp_max_nonneg<0x128>(v);   // row_ror:8, 4, 2, 1
    v = dpp_max_nonneg<0x124>(v);
    v = dpp_max_nonneg<0x122>(v);
    return dpp_max_nonneg<0x121>(v);
}

template <class F, int N>
struct Unit {
    using E = typename F::E;
    using R = typename F::R;
    static constexpr int T = N > 8 ? N - 8 : 0;
    static constexpr int R0 = 2 * (N - T);
    static_assert(N >= 7, "order 14 at least");
    static constexpr int NPH = N >= 8 ? 9 : 3;   // order-12 nodes of a unit: parts (nand_parts.h)
    static constexpr int L = nand_levels(N);

    Lds<F>& sh;
    int l16;
    double tau2;
    bool finite = true;          // the row's matrix
    double chk_lane = 0.0;       // of the leaves a lane formed (row: lane_row())
    int first = L;               // the row's first level above its parts with a pivot to shift
    uint64_t bad_rows = 0;       // a part: lanes (by row) that saw a pivot to shift in the row phase
    uint32_t bad_units = 0;      // the same from the lane phase, a bit per row of lanes

    __device__ Unit(Lds<F>& s) : sh(s) {}

    // Whether the tree shifts pivot p with row / column maxima (or any of their entries) r, c.
    __device__ __forceinline__ bool small(double pm, double r, double c) const
    {
        return pm == 0.0 || pm * pm < tau2 * r * c;
    }

    // ---------------------------------------------------------------- top phase
    // digit of block N - 1 - k on the path
    static __device__ __forceinline__ int digit(int path, int k)
    {
        int w = 1;
        for (int i = 0; i < T - 1 - k; ++i) w *= 3;
        return (path / w) % 3;
    }

    // c[k2] -= c[K] (entry of the scaled pivot row K in block k2's kept column), K < k2; zero
    // where block K is left out (in[K]): its column may have overflowed, and its pivot row of
    // zeros would make that a NaN
    template <int K, int K2>
    __device__ __forceinline__ void multipliers(E (&c)[T > 0 ? T : 1], const E (&w1)[T > 0 ? T : 1], const int (&in)[T > 0 ? T : 1])
    {
        if constexpr (K2 == K + 1) c[K] = keep_if(in[K], c[K]);
        if constexpr (K2 < T) {
            c[K2] = F::upd(c[K2], c[K], row_bcast<2 * K2>(w1[K]));
            multipliers<K, K2 + 1>(c, w1, in);
        } else if constexpr (K + 1 < T) {
            multipliers<K + 1, K + 2>(c, w1, in);
        }
    }

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

    // pivots J .. K-1 off a decided block's row: the undecided columns a0 (if Both) and the
    // decided ones a1; cm[J]: largest entry met in pivot column J
    template <int J, int K, bool Both>
    __device__ __forceinline__ void apply(E& a0, E& a1, const E (&w0)[T > 0 ? T : 1], const E (&w1)[T > 0 ? T : 1],
                                          double (&cm)[T > 0 ? T : 1], const int (&in)[T > 0 ? T : 1])
    {
        if constexpr (J < K) {
            E c = row_bcast<2 * J>(a1);
            cm[J] = fmax(cm[J], F::mag(c));
            c = keep_if(in[J], c);
            if constexpr (Both) a0 = F::upd(a0, c, w0[J]);
            a1 = F::upd(a1, c, w1[J]);
            apply<J + 1, K, Both>(a0, a1, w0, w1, cm, in);
        }
    }

    // Decided block K (rows wk: the kept one, or zero; other: the other row, decided columns):
    // its scaled pivot row, and what its test needs of the row.
    template <int K>
    __device__ __forceinline__ void pivot_rows(E (&w0)[T > 0 ? T : 1], E (&w1)[T > 0 ? T : 1], E (&x1)[T > 0 ? T : 1],
                                               double (&cm)[T > 0 ? T : 1], double (&rm)[T > 0 ? T : 1],
                                               double (&pm)[T > 0 ? T : 1], const int (&in)[T > 0 ? T : 1], E& mk)
    {
        if constexpr (K < T) {
            E a0 = w0[K], a1 = w1[K], o1 = x1[K];
            apply<0, K, true>(a0, a1, w0, w1, cm, in);
            apply<0, K, false>(o1, o1, w1, w1, cm, in);
            const E pv = row_bcast<2 * K>(a1);
            const double m0 = F::mag(a0), m1 = F::mag(a1);
            rm[K] = row_max(l16 > 2 * K + 1 && l16 < 2 * T ? fmax(m0, m1) : m0);
            pm[K] = F::mag(pv);
            if (in[K]) mk = F::bmul(mk, pv, 0);
            const R r = F::recip(pv);
            w0[K] = keep_if(in[K], F::rowscale(a0, r));
            w1[K] = keep_if(in[K], F::rowscale(a1, r));
            pivot_rows<K + 1>(w0, w1, x1, cm, rm, pm, in, mk);
        }
    }

    // The depth-T node of the path: M[i] = row i of its lane's column; mk = its minor.
    __device__ __forceinline__ void top(const E* A0, int path, E (&M)[R0], E& mk)
    {
        constexpr int w = 2 * N;
        if constexpr (T == 0) {
            const int c = l16 < w ? l16 : w - 1;
#pragma unroll
            for (int i = 0; i < R0; ++i) M[i] = A0[i * w + c];
        } else {
            // lanes 2 k and 2 k + 1 of the decided columns: block N - 1 - k's kept (or first)
            // column and its other one
            const int t = l16 < 2 * T ? l16 >> 1 : T - 1;
            const int kc = 2 * (N - 1 - t) + ((l16 & 1) ^ (digit(path, t) == 2 ? 1 : 0));
            E w0[T], w1[T], x1[T], c[T];
#pragma unroll
            for (int k = 0; k < T; ++k) {
                const int second = digit(path, k) == 2 ? 1 : 0;
                const int row = 2 * (N - 1 - k) + second;
                w0[k] = load_reg(&A0[row * w + l16]);
                w1[k] = load_reg(&A0[row * w + kc]);
                x1[k] = load_reg(&A0[(row ^ 1) * w + kc]);
                c[k] = load_reg(&A0[l16 * w + row]);
            }
#pragma unroll
            for (int i = 0; i < R0; ++i) M[i] = load_reg(&A0[i * w + l16]);
            __builtin_amdgcn_sched_barrier(0);
            double cm[T], rm[T], pm[T];
            int in[T];                             // all ones where block k is kept
#pragma unroll
            for (int k = 0; k < T; ++k) {
                cm[k] = 0.0;
                in[k] = -(int)(digit(path, k) != 0);
            }
            pivot_rows<0>(w0, w1, x1, cm, rm, pm, in, mk);
            multipliers<0, 1>(c, w1, in);
            // the tests (a left-out block has none)
#pragma unroll
            for (int k = T - 1; k >= 0; --k) {
                const double cmax = fmax(cm[k], row_max(F::mag(c[k])));
                if (in[k] && small(pm[k], rm[k], cmax)) first = k;
            }
#pragma unroll
            for (int k = 0; k < T; ++k) sub_rows<0>(M, c[k], w0[k]);
        }
    }

    // ---------------------------------------------------------------- row phase
    template <int P, int n, int m>
    __device__ __forceinline__ void child_rows(const E (&M)[m], E (&C)[m - 2], E w)
    {
        if constexpr (n == 6 && !F::kComplex) {
            row_child<P>(C[0], C[1], C[2], C[3], C[4], C[5], M[0], M[1], M[2], M[3], M[4], M[5], w);
        } else if constexpr (n >= 4) {
            row_child<P>(C[n - 4], C[n - 3], C[n - 2], C[n - 1], M[n - 4], M[n - 3], M[n - 2], M[n - 1], w);
            child_rows<P, n - 4>(M, C, w);
        } else if constexpr (n > 0) {
            row_child<P>(C[n - 2], C[n - 1], M[n - 2], M[n - 1], w);
        }
    }

    // The pivots of both kept children of an order-m node, tested: their reciprocals and the
    // children's minors, in lanes m - 2 and m - 1; bad[A]: lanes (by row) that saw the pivot of
    // child A to be shifted.
    template <int m>
    __device__ __forceinline__ void pivots(const E (&M)[m], E mk, E& mkd, R& rd, uint64_t (&bad)[2])
    {
        constexpr int mc = m - 2;
        const E d = l16 == mc + 1 ? M[mc + 1] : M[mc];
        mkd = F::bmul(mk, d, 0);
        rd = F::recip(d);
        // lane mc + a: the largest entry of its column and the size of its pivot
        double cm = F::mag(M[0]);
#pragma unroll
        for (int i = 1; i < mc; ++i) cm = fmax(cm, F::mag(M[i]));
        const double pm = F::mag(d);
        const bool s0 = small(row_bcast<mc>(pm), F::mag(M[mc]), row_bcast<mc>(cm));
        const bool s1 = small(row_bcast<mc + 1>(pm), F::mag(M[mc + 1]), row_bcast<mc + 1>(cm));
        bad[0] = ballot(l16 < mc && s0);
        bad[1] = ballot(l16 < mc && s1);
    }

    // whether a lane of this lane's row is in the mask
    __device__ __forceinline__ bool row_in(uint64_t mask) const { return ((mask >> (threadIdx.x & 48)) & 0xFFFF) != 0; }

    // The child that keeps row m - 2 + A.
    template <int A, int m>
    __device__ __forceinline__ void child(const E (&M)[m], E (&C)[m - 2], R rd)
    {
        constexpr int mc = m - 2, P = mc + A;
        const E w = F::rowscale(M[P], row_bcast<P>(rd));
        child_rows<P, mc>(M, C, w);
    }

    // One choice (wavefront-uniform) below an order-m node with pivots() mkd, rd.
    template <int m>
    __device__ __forceinline__ E choose(int a, const E (&M)[m], E (&C)[m - 2], E mk, E mkd, R rd)
    {
        if (a == 1) {
            child<0>(M, C, rd);
            return row_bcast<m - 2>(mkd);
        }
        if (a == 2) {
            child<1>(M, C, rd);
            return row_bcast<m - 1>(mkd);
        }
#pragma unroll
        for (int i = 0; i < m - 2; ++i) C[i] = M[i];
        return mk;
    }

    // The subtree of an order-m node down to order 8; t: its place.
    template <int m>
    __device__ __forceinline__ void node(const E (&M)[m], E mk, int t)
    {
        if constexpr (m == 8) {
            const int lane = threadIdx.x;
            if (l16 < 8) {
                E* d = &sh.node[((lane >> 4) * 9 + t) * kPS + l16];
#pragma unroll
                for (int i = 0; i < 8; ++i) d[i * 8] = M[i];
            }
            (l16 == 0 ? &sh.mn[(lane >> 4) * 9] : &sh.dump[lane])[t] = mk;
        } else {
            E mkd;
            R rd;
            uint64_t bad[2];
            pivots(M, mk, mkd, rd, bad);
            bad_rows |= bad[0] | bad[1];
            {
                E C[m - 2];
                child<0>(M, C, rd);
                node<m - 2>(C, row_bcast<m - 2>(mkd), 3 * t + 1);
            }
            {
                E C[m - 2];
                child<1>(M, C, rd);
                node<m - 2>(C, row_bcast<m - 1>(mkd), 3 * t + 2);
            }
            node<m - 2>(reinterpret_cast<const E(&)[m - 2]>(M), mk, 3 * t);
        }
    }

    // ---------------------------------------------------------------- lane phase
    // size of row p's and column p's first mc entries of a lane's matrix
    template <int mc, int n>
    static __device__ __forceinline__ void extremes(const E (&C)[n][n], int p, double& r, double& c)
    {
        r = F::mag(C[p][0]);
        c = F::mag(C[0][p]);
#pragma unroll
        for (int j = 1; j < mc; ++j) {
            r = fmax(r, F::mag(C[p][j]));
            c = fmax(c, F::mag(C[j][p]));
        }
    }

    // A lane's order-4 node to its 9 leaves.
    __device__ __forceinline__ void leaves(const E (&C)[4][4], E mk, E (&lv)[9], bool& shift)
    {
#pragma unroll
        for (int g = 0; g < 3; ++g) {
            E D00 = C[0][0], D11 = C[1][1], m = mk;
            if (g) {
                const int p = 1 + g;
                double r, c;
                extremes<2>(C, p, r, c);
                shift = shift || small(F::mag(C[p][p]), r, c);
                m = F::bmul(mk, C[p][p], 0);
                const R rd = F::recip(C[p][p]);
                D00 = F::upd(D00, C[0][p], F::rowscale(C[p][0], rd));
                D11 = F::upd(D11, C[1][p], F::rowscale(C[p][1], rd));
            }
            lv[3 * g] = m;
            lv[3 * g + 1] = F::bmul(m, D00, 0);
            lv[3 * g + 2] = F::bmul(m, D11, 0);
        }
    }

    // Rows 2 H and 2 H + 1 of lanes (H: the pass): their 18 nodes' children, a lane each, to
    // the leaves at oa and ob (of the two rows; NULL if there is no such unit).
    template <int H>
    __device__ __forceinline__ void lanes(E* oa, E* ob)
    {
        const int lane = xrow::lane_here();
        const bool act = lane < 54;
        const int src = act ? lane : 53;           // idle lanes repeat the last one
        const int q = H * 18 + src / 3, c = src % 3, in = -(int)(c != 0), p = c == 2 ? 7 : 6;
        wave_sync();
        E C[6][6], pr[6], pc[6];
        const E* P = &sh.node[q * kPS];
        const E mq = load_reg(&sh.mn[q]), pv = load_reg(&P[p * 9]);
#pragma unroll
        for (int j = 0; j < 6; ++j) pr[j] = load_reg(&P[p * 8 + j]);
#pragma unroll
        for (int i = 0; i < 6; ++i) pc[i] = load_reg(&P[i * 8 + p]);
#pragma unroll
        for (int i = 0; i < 6; ++i)
#pragma unroll
            for (int j = 0; j < 6; ++j) C[i][j] = load_reg(&P[i * 8 + j]);
        __builtin_amdgcn_sched_barrier(0);
        double rm = F::mag(pr[0]), cm = F::mag(pc[0]);
#pragma unroll
        for (int j = 1; j < 6; ++j) {
            rm = fmax(rm, F::mag(pr[j]));
            cm = fmax(cm, F::mag(pc[j]));
        }
        bool shift = c != 0 && small(F::mag(pv), rm, cm);
        const E m6 = c ? F::bmul(mq, pv, 0) : mq;
        R r = F::recip(pv);
        // one instruction stream for the three children: the one that leaves the block out
        // subtracts zero times zero
#pragma unroll
        for (int j = 0; j < 6; ++j) pr[j] = keep_if(in, F::rowscale(pr[j], r));
#pragma unroll
        for (int i = 0; i < 6; ++i) lane_rows<6>(C[i], C[i], keep_if(in, pc[i]), pr);
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            double er, ec;
            extremes<4>(C, 4 + a, er, ec);
            shift = shift || small(F::mag(C[4 + a][4 + a]), er, ec);
        }
        E* st = &sh.node[H == 0 ? 0 : 18 * kPS];   // the place of this pass's nodes
        static_assert(64 * 9 <= 18 * kPS, "9 leaves a lane fit");
        wave_sync();                               // every lane has read its node
        // the staged leaves 63 at a time: lane 9 s + e is leaf e of source 7 it + s
        const int ls = lane / 9, le = lane - 9 * ls;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            E lv[9];
            if (k == 0) {
                E K[4][4];
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j) K[i][j] = C[i][j];
                leaves(K, m6, lv, shift);
            } else {
                const int pp = 3 + k;
                r = F::recip(C[pp][pp]);
                E w[4], K[4][4];
#pragma unroll
                for (int j = 0; j < 4; ++j) w[j] = F::rowscale(C[pp][j], r);
#pragma unroll
                for (int i = 0; i < 4; ++i) lane_rows<4>(K[i], C[i], C[i][pp], w);
                leaves(K, F::bmul(m6, C[pp][pp], 0), lv, shift);
            }
#pragma unroll
            for (int e = 0; e < 9; ++e) {
                st[lane * 9 + e] = lv[e];
                chk_lane += F::fincheck(lv[e]);
            }
            wave_sync();
            flush<0>(st + lane, oa + (ls * 27 + 9 * k + le), ob + (ls * 27 + 9 * k + le), oa != nullptr,
                     ob != nullptr, lane < 63, ls);
            wave_sync();
        }
        const uint64_t s = ballot(act && shift);
        if (s & 0x7FFFFFFull) bad_units |= 1u << (2 * H);
        if (s >> 27) bad_units |= 2u << (2 * H);
        // non-finite leaves, by row
        const uint64_t f = ballot(act && chk_lane != 0.0);
        if (f & 0x7FFFFFFull) nonfinite |= 1u << (2 * H);
        if (f >> 27) nonfinite |= 2u << (2 * H);
        chk_lane = 0.0;
    }

    uint32_t nonfinite = 0;      // units with a non-finite leaf, a bit per row of lanes

    template <int IT>
    __device__ __forceinline__ void flush(const E* st, E* oa, E* ob, bool va, bool vb, bool act, int ls)
    {
        if constexpr (IT < 8) {
            const E v = load_reg(&st[IT * 63]);
            flush<IT + 1>(st, oa, ob, va, vb, act, ls);
            // sources 7 IT + ls: the first 27 are the first row's
            const bool b = IT == 3 ? ls == 6 : IT > 3;
            if (act && (IT < 7 || ls < 5) && (b ? vb : va)) (b ? ob - 27 * 27 : oa)[IT * 7 * 27] = v;
        } else {
            __builtin_amdgcn_sched_barrier(0);
        }
    }

    template <int n>
    static __device__ __forceinline__ void lane_rows(double* k, const double* a, double c, const double* w)
    {
#pragma unroll
        for (int j = 0; j < n; ++j) k[j] = fma(-c, w[j], a[j]);
    }
    template <int n>
    static __device__ __forceinline__ void lane_rows(cd* k, const cd* a, cd c, const cd* w)
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
};

// Wavefront blockIdx.x: units 4 (blockIdx.x / C) .. + 3 (C = 3 choices of the block below the
// top ones from 8 blocks on, choice blockIdx.x % 3; else 1).  info gets 0 or -2 from the wavefront
// of a matrix's first part.
template <class F, int N, int WAVES>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(WAVES))) void nand_row_kernel(
    const typename F::E* __restrict__ A, typename F::E* __restrict__ out, int32_t* __restrict__ info,
    NandWs ws, int64_t units)
{
    using E = typename F::E;
    using U = Unit<F, N>;
    constexpr int T = U::T, w = 2 * N, C1 = N >= 8 ? 3 : 1;
    constexpr int64_t kUnits = pow3(T), nout = pow3(N);
    constexpr int kPhase = 9 * 81;                  // leaves of a phase
    __shared__ Lds<F> sh;
    const int lane = threadIdx.x;
    const int64_t u0 = (int64_t)(blockIdx.x / C1) * 4;
    const int c1 = (int)(blockIdx.x % C1);
    const int64_t u = u0 + (lane >> 4);
    const bool valid = u < units;
    const int64_t uc = valid ? u : units - 1;
    const int64_t b = uc / kUnits;
    const int path = (int)(uc - b * kUnits);
    const E* A0 = A + b * (w * w);
    U un(sh);
    un.l16 = lane & 15;
    un.tau2 = kDefaultPivTol * kDefaultPivTol;
    // (the loads of eight entries before their checks: a round trip for each took as long as a part)
    bool fin = true;
#pragma unroll
    for (int e0 = 0; e0 < w * w; e0 += 128) {
        E v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (e0 + 16 * k < w * w) v[k] = load_reg(&A0[min(e0 + 16 * k + un.l16, w * w - 1)]);
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (e0 + 16 * k < w * w) fin = fin & F::in_finite(v[k]);
    }
    un.finite = !un.row_in(ballot(!fin));
    E M[U::R0], mk = F::one();
    if (!un.finite) F::store_nan(&mk, nullptr, 0, false);   // makes every minor NaN
    if (info && valid && un.l16 == 0 && path == 0 && c1 == 0) info[b] = un.finite ? 0 : -2;
    un.top(A0, path, M, mk);

    // the rows' outputs of this wavefront's first phase
    E* o[4];
#pragma unroll
    for (int r = 0; r < 4; ++r)
        o[r] = u0 + r < units ? out + ((u0 + r) / kUnits) * nout +
                                    (((u0 + r) % kUnits) * U::NPH + (N >= 8 ? 3 * c1 : 0)) * kPhase
                              : nullptr;
    auto emit = [&](int ph) {
        un.template lanes<0>(o[0] ? o[0] + ph * kPhase : nullptr, o[1] ? o[1] + ph * kPhase : nullptr);
        un.template lanes<1>(o[2] ? o[2] + ph * kPhase : nullptr, o[3] ? o[3] + ph * kPhase : nullptr);
    };
    // The words of this wavefront's three parts per row, by its lanes 0 .. 2.  bad: the order-14
    // node's tests; deep, nonfinite: rows of lanes by part, four bits each.
    auto tell = [&](const uint64_t (&bad)[2], uint32_t deep, uint32_t nonfinite) {
        const int c = un.l16, at = 4 * c + (lane >> 4);
        int first = un.first;
        if (c && first == U::L && un.row_in(c == 1 ? bad[0] : bad[1])) first = U::L - 1;
        const bool redo = un.finite && (first < U::L || ((deep >> at) & 1));
        const bool bad_minor = un.finite && !redo && ((nonfinite >> at) & 1);
        const uint32_t part = (uint32_t)(u * U::NPH + (N >= 8 ? 3 * c1 : 0) + c);
        const bool own = valid && c < 3;
        if (own) ws.words[part] = (uint32_t)first | (redo ? kPartRedo : 0u) | (bad_minor ? kPartBad : 0u);
        const uint64_t again = ballot(own && redo);
        if (again) {
            int at0 = 0;
            const int sub = (int)blockIdx.x & (ws.subs - 1);
            if (lane == 0) at0 = atomicAdd(ws.head + sub * kHeadStride, __builtin_popcountll(again));
            at0 = __builtin_amdgcn_readfirstlane(at0) + sub * ws.cap;
            if (own && redo) ws.list[at0 + __builtin_popcountll(again & ((uint64_t(1) << lane) - 1))] = part;
        }
        if (ballot(own && bad_minor) && lane == 0) atomicAdd(ws.head + kHeadBad, 1);
    };
    // Whether every row has nothing to write: no such unit, or a pivot to shift (its parts are
    // formed again; those of a non-finite matrix are not, whatever its tests say)
    auto lost = [&](bool shift) { return ~ballot(!valid || (un.finite && (un.first < U::L || shift))) == 0; };
    auto below14 = [&](const E(&M14)[14], E mk14) {
        E mkd;
        typename F::R rd;
        uint64_t bad[2];
        un.pivots(M14, mk14, mkd, rd, bad);
        if (lost(un.row_in(bad[0]) && un.row_in(bad[1]))) return tell(bad, 0xFFFu, 0);
        uint32_t deep = 0, nonfinite = 0;
#pragma unroll 1
        for (int c2 = 0; c2 < 3; ++c2) {
            E C[12];
            un.bad_rows = 0;
            const E mc = un.choose(c2, M14, C, mk14, mkd, rd);
            un.template node<12>(C, mc, 0);
            un.bad_units = un.nonfinite = 0;
            emit(c2);
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if ((un.bad_rows >> (16 * r)) & 0xFFFF) un.bad_units |= 1u << r;
            deep |= un.bad_units << (4 * c2);
            nonfinite |= un.nonfinite << (4 * c2);
        }
        tell(bad, deep, nonfinite);
    };
    if constexpr (N >= 8) {
        E mkd, C[14];
        typename F::R rd;
        uint64_t bad[2];
        un.pivots(M, mk, mkd, rd, bad);
        if (c1 && un.row_in(c1 == 1 ? bad[0] : bad[1])) un.first = min(un.first, T);
        if (lost(false)) return tell(bad, 0xFFFu, 0);
        const E mc = un.choose(c1, M, C, mk, mkd, rd);
        below14(C, mc);
    } else {
        below14(M, mk);
    }
}

template <class F, int WAVES, int N>
hipError_t launch_n(const LaunchXor& L, hipStream_t st)
{
    if constexpr (N > 13) {
        return hipErrorInvalidValue;
    } else {
        if (L.n != N) return launch_n<F, WAVES, N + 1>(L, st);
        const int64_t units = (int64_t)L.batch * pow3(Unit<F, N>::T);
        const int64_t grid = nand_row_waves(N, L.batch);
        hipLaunchKernelGGL((nand_row_kernel<F, N, WAVES>), dim3((unsigned)grid), dim3(64), 0, st,
                           static_cast<const typename F::E*>(L.A), static_cast<typename F::E*>(L.out), L.info, L.nand,
                           units);
        return hipGetLastError();
    }
}

}  // namespace nrow
}  // namespace apm
