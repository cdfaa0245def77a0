// xor.hip -- XOR and XNOR principal minors of 2n x 2n block matrices (Sec. III) on gfx950.
//
// A 2n x 2n matrix is read as n x n blocks of 2 x 2.  Its XOR minors keep exactly one
// row/column of every block; with the Keldysh block matrix of Sec. V.C they are the
// determinants of all 2^n branch assignments.  The binary tree of the XOR case: a node at
// depth d holds the matrix of the blocks not yet decided, as the Schur complement over the
// rows kept so far.  Each of its two children keeps one row of the next block as pivot,
// drops the other, and is the Schur complement over that pivot; the child's minor is the
// node's minor times the pivot (the ratio rule of Sec. II with a 1 x 1 pivot).  No pivot
// shift is made: its correction would need minors this tree never forms (the paper notes
// the same), so a zero pivot leaves its subtree non-finite and info = -3.
//
// The NAND case (Sec. III) keeps at most one row of every block: a ternary tree whose
// children leave the block out (minor unchanged) or keep one of its rows (1 x 1 pivot).
// Its left-out children are the minors that the pivot correction needs, so a small or zero
// pivot is shifted (the test and C of the minors tree) and the kept child's subtree is
// corrected once it is complete (see nand_top_fix).
//
// The XNOR case (Sec. III) keeps both or neither row of every block.  Its tree has the
// same shape: one child drops the last undecided block (the node's leading part, minor
// unchanged), the other keeps it (the Schur complement over the 2 x 2 pivot block, minor
// times the block's determinant).  Only the 2^n leaves are minors of distinct subsets;
// they are written in block-mask order (bit i <-> block i kept).
//
// Which kernel: XOR and XNOR minors of 4 blocks and more run in xor_row.h, NAND minors of
// kNandRowMin blocks and more in nand_row.h (node matrices in registers).  Here are the XOR and
// XNOR minors of up to 3 blocks (a matrix is one LDS subtree), the NAND minors of up to 6, and
// the parts of larger ones whose pivots need shifts (nand_parts.h).
//
// Mapping (one wavefront per matrix of up to 6 blocks, or per such a node of a larger one; lanes
// exchange through LDS with wavefront syncs only, so the stores of the minors stay in flight):
//   * the last block is decided first, so a node's remaining blocks are the leading ones
//     and the pivot rows are the last two rows of its matrix; depth k of the output holds
//     the minors of the k trailing blocks, and every subtree's outputs are contiguous;
//   * top levels (NAND, d < T = n - Q <= 2): depth first over the 3^T depth-T nodes, the node
//     matrices in LDS, each row of the child split over as many lanes as the wavefront allows,
//     with the pivot row (scaled by 1/pivot) staged in LDS;
//   * the last Q = min(n, 4) levels (XOR, XNOR: all of at most 3) of each depth-T node: breadth
//     first in LDS, one row of a child per lane (split over column groups where the rows leave
//     lanes idle), so each level is one pass (at most 64 rows);
//   * the LDS arrays are sized for the one tree a kernel runs (binary or ternary), which
//     sets how many wavefronts a compute unit holds;
//   * every size is a compile-time constant (one kernel per number of blocks), so no index
//     arithmetic divides at run time.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

#include "apm_device.h"
#include "apm_kernels.h"
#include "nand_parts.h"

namespace apm {
namespace {

// XOR and XNOR: the register kernels (xor_row.h) take over at 4 blocks, the fewest they are
// built for.  They are not slower there (3000 complex matrices of 4 blocks: 9.8 us against
// 10.1, launch-bound) and gain from 6 blocks on (3000 complex XNOR of 6: 8.9 against 12.5).
constexpr int kRowMin = 4;
constexpr int kXQ = 3;       // levels expanded breadth first in LDS (XOR, XNOR)
constexpr int kXQ3 = 4;      // the same for the ternary NAND tree
// modes: the XOR, XNOR and NAND cases of Sec. III
constexpr int kXor = 0, kXnor = 1, kNand = 2;
__host__ __device__ constexpr int xq(int mode) { return mode == kNand ? kXQ3 : kXQ; }
__host__ __device__ constexpr int64_t pow3(int k) { return k <= 0 ? 1 : 3 * pow3(k - 1); }
#ifndef APM_XOR_PAD
#define APM_XOR_PAD 1
#endif
// Row stride of an order-m node matrix in LDS: one element of padding, so that lanes
// reading the same column of different rows fall on different banks.
__host__ __device__ constexpr int xs(int m) { return m + APM_XOR_PAD; }
// Subtree levels in LDS: level J (0: the root) is in place J & 1.  Entries of the largest level of
// a place (rows padded), and its number of nodes at most.
__host__ __device__ constexpr int xlevel_nodes(int mode, int J)
{
    int k = 1;
    for (int j = 0; j < J; ++j) k *= mode == kNand ? 3 : 2;
    return k;
}
__host__ __device__ constexpr int xbuf_need(int mode, int place)
{
    int need = 1;
    for (int J = place; J <= xq(mode); J += 2) {
        const int m = 2 * (xq(mode) - J), lvl = xlevel_nodes(mode, J) * m * xs(m);
        need = lvl > need ? lvl : need;
    }
    return need;
}
__host__ __device__ constexpr int xmn_need(int mode, int place)
{
    return xlevel_nodes(mode, (xq(mode) & 1) == place ? xq(mode) : xq(mode) - 1);
}
// The depth T-1 node (order 2(Q + 1)) is kept in LDS as well.
__host__ __device__ constexpr int xpre_need(int mode) { return 2 * (xq(mode) + 1) * xs(2 * (xq(mode) + 1)); }
// Lanes per row in a subtree pass of `rows` rows of mc entries: the largest divisor of mc
// that keeps rows x H within the wavefront (1 when the rows fill it).
__host__ __device__ constexpr int col_groups(int rows, int mc)
{
    int h = 1;
    for (int c = 2; c <= mc && rows * c <= 64; ++c)
        if (mc % c == 0) h = c;
    return h;
}
// Columns per lane in a top-level pass over a child of order mc (mc rows): as few as the
// wavefront allows, with the column groups as even as that count permits.
__host__ __device__ constexpr int top_cols(int mc)
{
    const int hmax = 64 / mc < mc ? 64 / mc : mc;
    return (mc + hmax - 1) / hmax;
}
// Zero pivot rows of the widest subtree level (two rows of order 2Q - 2).
__host__ __device__ constexpr int xzero_need(int mode) { return xq(mode) > 1 ? 4 * xq(mode) - 4 : 1; }

// NAND subtree levels that can shift (child order >= 1): J <= kXQ3 - 2.  Kept-row pairs of
// the widest such level, and the shift codes of all their children.
__host__ __device__ constexpr int xsub_pairs_max() { return 2 * (int)pow3(kXQ3 - 2); }
__host__ __device__ constexpr int xsub_codes() { return ((int)pow3(kXQ3) - 3) / 2; }
__host__ __device__ constexpr int xsub_code_base(int J) { return ((int)pow3(J + 1) - 3) / 2; }

template <class F, int MODE>
struct XorLds {
    typename F::E buf0[xbuf_need(MODE, 0)], buf1[xbuf_need(MODE, 1)];
    typename F::E mn0[xmn_need(MODE, 0)], mn1[xmn_need(MODE, 1)];   // the nodes' minors
    typename F::E wk[64];            // subtree levels: each child's pivot row times 1/pivot
    typename F::E wv[MODE == kNand ? 2 * xq(MODE) + 2 : 1];   // top levels: pivot row times 1/pivot
    typename F::E topm[3];           // minors along the top path
    typename F::E pre[MODE == kNand ? xpre_need(MODE) : 1];     // the depth T-1 node
    // zeros: the pivot column and rows of a child that leaves its block out, so that it
    // runs the keeping children's code
    typename F::E wz[xzero_need(MODE)];
    // NAND pivot shifts: the (possibly shifted) pivots of a subtree level's kept rows (levels
    // with a small pivot only), the shift codes of the subtree's nodes (level J + 1 children
    // from xsub_code_base(J) on; valid for the levels in XPiv::sub_mask)
    typename F::E pvs[MODE == kNand ? xsub_pairs_max() : 1];
    int8_t scode[MODE == kNand ? xsub_codes() : 1];
    // a shifted child's own entry (no deeper row kept), with the true pivot: subtree
    // children by code index, and the top-level child of the current path
    typename F::E sown[MODE == kNand ? xsub_codes() : 1];
    typename F::E topown;
    __device__ __forceinline__ typename F::E* buf(int place) { return place ? buf1 : buf0; }
    __device__ __forceinline__ typename F::E* mn(int place) { return place ? mn1 : mn0; }
};

// Biased binary exponent of max(|Re v|, |Im v|) (0 for zero and subnormals), from the high
// words: the fast pivot-shift test compares exponents with integer operations.  The exact
// test can fail only with an entry above |p| / tau >= 2^9 |p| (tau = 1e-3 <= 2^-9), whose
// exponent is then at least kFastExp above p's; so "p normal and no entry kFastExp or more
// above it" passes the exact test.
__device__ __forceinline__ int xexp(double v) { return (__double2hiint(v) & 0x7FFFFFFF) >> 20; }
__device__ __forceinline__ int xexp(cd v) { return xexp(v.x) > xexp(v.y) ? xexp(v.x) : xexp(v.y); }
constexpr int kFastExp = 9;
static_assert(kDefaultPivTol <= 0x1p-9, "an entry above |p| / tau has an exponent >= kFastExp above p's");

// Matrix-wide state of the NAND pivot shifts: tau^2, the exponent of the largest input
// magnitude, the shifts made, and whether the current subtree made any.
struct XPiv {
    double tau2;
    int es;
    int nsh;
    int sub_mask;    // subtree levels of the current subtree with a shifted pivot (bit J)
    bool top_own;    // the current path's last kept child was shifted (own entry in topown)
    uint32_t tc;     // shift codes of the path's children at the top levels: byte D
    __device__ int tcode(int D) const { return (int)(int8_t)(tc >> (8 * D)); }
    __device__ void set_tcode(int D, int code) { tc = (tc & ~(0xFFu << (8 * D))) | (uint32_t)(uint8_t)code << (8 * D); }
};

// Pivot of kept row p of an order-m subtree node P (rows of stride xs(m)), shifted if the
// test fails on the row and column entries that enter the child (the first mc = m - 2).
template <class F, int m>
__device__ __forceinline__ typename F::E nand_sub_pivot(const typename F::E* P, int p, const XPiv& xp, int8_t& code)
{
    constexpr int mc = m - 2;
    typename F::E pv = P[p * xs(m) + p];
    double rmax = 0.0, cmax = 0.0;
#pragma unroll
    for (int j = 0; j < mc; ++j) {
        rmax = fmax(rmax, F::mag(P[p * xs(m) + j]));
        cmax = fmax(cmax, F::mag(P[j * xs(m) + p]));
    }
    const double pm = F::mag(pv);
    code = kNoEv;
    if (pm == 0.0 || pm * pm < xp.tau2 * rmax * cmax) {
        code = shift_code(rmax, cmax, xp.es, F::re(pv) < 0.0);
        pv = F::shift(pv, shift_value(xp.es, code));
    }
    return pv;
}

// NAND top level D whose fast pivot test failed (rare, out of line): the test on the row and
// column maxima of kept row p of node P (row stride ps); if the pivot is shifted, the child C
// (row stride cs) is formed again with the shifted pivot, the node's minor times it goes to
// topm[D + 1] and the child's own entry (with the true pivot) to topown.  Returns the code.
template <class F, int N, int D>
__device__ __noinline__ int nand_top_slow(const typename F::E* P, typename F::E* C, int p, int ps, int cs,
                                          XorLds<F, kNand>& sh, double tau2, int es)
{
    using E = typename F::E;
    constexpr int m = 2 * (N - D), mc = m - 2;
    constexpr int cw = top_cols(mc), H = (mc + cw - 1) / cw;
    constexpr bool kEven = mc % cw == 0;
    const int lane = threadIdx.x;
    const int i = lane % mc, h = lane / mc, h0 = h * cw;
    const bool act = h < H;
    const E pv = P[p * ps + p];
    E pc = F::zero(), pr = F::zero();
    if (act) pc = P[i * ps + p];
    if (lane < mc) pr = P[p * ps + lane];
    const double rmax = wave_max_nonneg(lane < mc ? F::mag(pr) : 0.0);
    const double cmax = wave_max_nonneg(act ? F::mag(pc) : 0.0);
    const double pm = F::mag(pv);
    if (!(pm == 0.0 || pm * pm < tau2 * rmax * cmax)) return kNoEv;
    const int code = shift_code(rmax, cmax, es, F::re(pv) < 0.0);
    const E ps2 = F::shift(pv, shift_value(es, code));
    const typename F::R r2 = F::recip(ps2);
    wave_sync();   // every lane has read wv
    if (lane < mc) sh.wv[lane] = F::rowscale(pr, r2);
    if (lane == 0) {
        sh.topown = F::bmul(sh.topm[D], pv, 0);
        sh.topm[D + 1] = F::bmul(sh.topm[D], ps2, 0);
    }
    wave_sync();
    if (act) {
#pragma unroll
        for (int j = 0; j < cw; ++j)
            if (kEven || h0 + j < mc) C[i * cs + h0 + j] = F::upd(P[i * ps + h0 + j], pc, sh.wv[h0 + j]);
    }
    return code;
}

// Top level D of matrix order 2N (at most two levels): the child of the depth-D node on path s
// (a group of columns of a row of the child per lane), from the root P0 (row stride PS0; D = 0)
// or LDS to LDS, where rows have stride xs(order).
template <class F, int N, int T, int D, int PS0>
__device__ __forceinline__ void nand_top(int d0, int s, const typename F::E* P0, XorLds<F, kNand>& sh, double& chk,
                                         XPiv& xp)
{
    if constexpr (D < T) {
        using E = typename F::E;
        constexpr int m = 2 * (N - D), mc = m - 2;
        static_assert(T <= 2, "the child is the depth T-1 node (pre) or the depth-T node (buf)");
        if (D >= d0) {
            const int lane = threadIdx.x;
            constexpr int ps = D == 0 ? PS0 : xs(m), cs = xs(mc);
            static_assert(mc * xs(mc) <= (D == T - 1 ? xbuf_need(kNand, 0) : xpre_need(kNand)), "the node fits its buffer");
            const E* P = D == 0 ? P0 : sh.pre;
            E* C = D == T - 1 ? sh.buf(0) : sh.pre;
            // this level's choice: 0 leaves the block out, 1 and 2 keep its first or second row
            const int a = (int)((s / pow3(T - 1 - D)) % 3);
            // every load of the node first, then the arithmetic: one round trip per node.
            // Lane h mc + i takes columns [h cw, (h + 1) cw) of row i of the child.
            constexpr int cw = top_cols(mc), H = (mc + cw - 1) / cw;
            constexpr bool kEven = mc % cw == 0;
            const int i = lane % mc, h = lane / mc, h0 = h * cw;
            const bool act = h < H;
            E row[cw];
            if (act) {
#pragma unroll
                for (int j = 0; j < cw; ++j)
                    if (kEven || h0 + j < mc) row[j] = P[i * ps + h0 + j];
            }
            if (a != 0) {
                // child keeps row p of the last block: 1 x 1 pivot
                const int p = mc + a - 1;
                const E pv = P[p * ps + p];
                E pc = F::zero(), pr = F::zero();
                if (act) pc = P[i * ps + p];
                if (lane < mc) pr = P[p * ps + lane];
                const typename F::R r = F::recip(pv);
                if (lane < mc) sh.wv[lane] = F::rowscale(pr, r);
                if (lane == 0) {
                    const E mk = F::bmul(sh.topm[D], pv, 0);
                    sh.topm[D + 1] = mk;
                    chk += F::fincheck(mk);
                }
                wave_sync();
                if (act) {
#pragma unroll
                    for (int j = 0; j < cw; ++j)
                        if (kEven || h0 + j < mc) C[i * cs + h0 + j] = F::upd(row[j], pc, sh.wv[h0 + j]);
                }
                // pivot shift (Sec. II test on the kept row and column of the child's Schur
                // complement), checked once the child is written (its inputs are at hand by
                // then); a shifted child is formed again and corrected once its subtree is
                // complete.  No lane holding an entry kFastExp binary orders above p:
                // the test passes without the maxima.
                const int ep = xexp(pv);
                const int le = max(lane < mc ? xexp(pr) : 0, act ? xexp(pc) : 0);
                int code = kNoEv;
                if (ballot(ep == 0 || le >= ep + kFastExp)) {
                    code = nand_top_slow<F, N, D>(P, C, p, ps, cs, sh, xp.tau2, xp.es);
                }
                xp.set_tcode(D, code);
                xp.top_own = code != kNoEv;
            } else {
                // the block left out: the leading part of the node, minor unchanged
                if (lane == 0) sh.topm[D + 1] = sh.topm[D];
                xp.set_tcode(D, kNoEv);
                if (act) {
#pragma unroll
                    for (int j = 0; j < cw; ++j)
                        if (kEven || h0 + j < mc) C[i * cs + h0 + j] = row[j];
                }
            }
            wave_sync();   // the child is the next level's node (and wv is rewritten)
        }
        nand_top<F, N, T, D + 1, PS0>(d0, s, P0, sh, chk, xp);
    }
}

// Update pass of subtree level J: the children's matrices (orders 2(Q - J) - 2) from the
// nodes in buf[J & 1] and the scaled pivot rows in wk.  Lane (h, k, i) writes columns
// [h cw, (h + 1) cw) of row i of child k: where the rows do not fill the wavefront, each row
// is split over H lanes.
template <class F, int Q, int J, int MODE>
__device__ __forceinline__ void xor_sub_update(XorLds<F, MODE>& sh)
{
    using E = typename F::E;
    constexpr int cur = J & 1, nxt = cur ^ 1;
    constexpr int m = 2 * (Q - J), mc = m - 2;
    constexpr int kids = MODE == kNand ? (int)pow3(J + 1) : 2 << J;
    constexpr int rows = kids * mc, H = col_groups(rows, mc), cw = mc / H;
    const int lane = threadIdx.x;
    if (lane < rows * H) {
        const int r = lane % rows, h = lane / rows;
        const int k = r / mc, i = r - k * mc, j0 = h * cw;
        E* Cr = &sh.buf(nxt)[k * mc * xs(mc) + i * xs(mc)] + j0;
        // the node's entries from column j0 on (two children per node, three for NAND)
        const E* P = &sh.buf(cur)[(MODE == kNand ? k / 3 : k >> 1) * m * xs(m)] + j0;
        if constexpr (MODE == kNand) {
            const int c = k % 3;
            // one instruction stream for all three children (a copy branch beside the
            // update would issue both): the one that leaves the block out subtracts
            // zero times a zero row
            const E ci = c ? P[i * xs(m) + mc - j0 + c - 1] : F::zero();
            const E* wr = (c ? &sh.wk[(2 * (k / 3) + c - 1) * mc] : sh.wz) + j0;
#pragma unroll
            for (int j = 0; j < cw; ++j) Cr[j] = F::upd(P[i * xs(m) + j], ci, wr[j]);
        } else if constexpr (MODE == kXor) {
            const E ci = P[i * xs(m) + mc - j0 + (k & 1)];
            const E* wr = &sh.wk[k * mc] + j0;
#pragma unroll
            for (int j = 0; j < cw; ++j) Cr[j] = F::upd(P[i * xs(m) + j], ci, wr[j]);
        } else {
            // both children in one instruction stream: the one that drops the block
            // subtracts zero times zero rows
            const bool keep = k & 1;
            const E c0 = keep ? P[i * xs(m) + mc - j0] : F::zero();
            const E c1 = keep ? P[i * xs(m) + mc - j0 + 1] : F::zero();
            const E* w0 = (keep ? &sh.wk[(k >> 1) * 2 * mc] : sh.wz) + j0;
#pragma unroll
            for (int j = 0; j < cw; ++j) Cr[j] = F::upd(F::upd(P[i * xs(m) + j], c0, w0[j]), c1, w0[mc + j]);
        }
    }
    wave_sync();
}

// NAND subtree level J whose fast pivot test failed (rare, out of line): each kept row tested
// on its row and column maxima; if any is shifted, the level's kept children are formed again
// with the shifted pivots.  Returns the shifts made (codes and own entries in sh).
template <class F, int Q, int J>
__device__ __noinline__ int nand_sub_slow(XorLds<F, kNand>& sh, double tau2, int es)
{
    using E = typename F::E;
    constexpr int cur = J & 1, nxt = cur ^ 1;
    constexpr int m = 2 * (Q - J), mc = m - 2;
    constexpr int kids = (int)pow3(J + 1);
    const int lane = threadIdx.x;
    XPiv xp{tau2, es, 0, 0, false, 0};
    bool shifted = false;
    if (lane < 2 * (kids / 3)) {
        const int v = lane >> 1, p = mc + (lane & 1);
        const E* P = &sh.buf(cur)[v * m * xs(m)];
        int8_t code;
        const E pv = nand_sub_pivot<F, m>(P, p, xp, code);
        const int ci = xsub_code_base(J) + 3 * v + (lane & 1) + 1;
        if (code != kNoEv) {
            sh.sown[ci] = F::bmul(sh.mn(cur)[v], P[p * xs(m) + p], 0);
            shifted = true;
        }
        sh.scode[ci] = code;
        sh.pvs[lane] = pv;
    }
    const int ns = __builtin_popcountll(ballot(shifted));
    if (ns) {
        wave_sync();
        if (lane < kids) {
            const int v = lane / 3, c = lane - 3 * v;
            if (c) sh.mn(nxt)[lane] = F::bmul(sh.mn(cur)[v], sh.pvs[2 * v + c - 1], 0);
        }
        if (lane < 2 * (kids / 3) * mc) {
            const int v = lane / (2 * mc), rr = lane - v * 2 * mc, r = rr / mc, j = rr - r * mc;
            const E* P = &sh.buf(cur)[v * m * xs(m)];
            sh.wk[lane] = F::rowscale(P[(mc + r) * xs(m) + j], F::recip(sh.pvs[2 * v + r]));
        }
        wave_sync();
        xor_sub_update<F, Q, J, kNand>(sh);
    }
    return ns;
}

// Subtree level J of a Q-level subtree: the children of the 2^J nodes in buf[J & 1]
// (order 2(Q - J)) into buf[(J + 1) & 1], one row (or column group) of a child per lane.
// base is where the children's depth T+J+1 starts in the output (2^(T+J+1) - 2; XOR
// only: the XNOR minors are the 2^N leaves, written at the last level in block-mask order).
template <class F, int Q, int J, int MODE>
__device__ __forceinline__ void xor_sub(int64_t base, int s, typename F::E* ob, XorLds<F, MODE>& sh, double& chk,
                                        XPiv& xp)
{
    if constexpr (J < Q) {
        using E = typename F::E;
        constexpr int cur = J & 1, nxt = cur ^ 1;
        constexpr int m = 2 * (Q - J), mc = m - 2;
        constexpr int kids = MODE == kNand ? (int)pow3(J + 1) : 2 << J;
        static_assert(kids * mc <= 64 && (MODE == kNand || kids <= 64), "one pass per level");
        static_assert(kids * mc * xs(mc) <= xbuf_need(MODE, nxt) &&
                          m * xs(m) * (kids / (MODE == kNand ? 3 : 2)) <= xbuf_need(MODE, cur),
                      "a subtree level fits its LDS buffer");
        static_assert(2 * mc <= xzero_need(MODE), "zero pivot rows cover a level");
        static_assert(kids <= xmn_need(MODE, nxt), "a level's minors fit");
        const int lane = threadIdx.x;
        bool maybe = false;   // NAND: this lane's fast pivot-shift test failed
        if constexpr (MODE == kXor) {
            // child k of node k/2 keeps row mc + (k & 1) of the node's last block: its minor,
            // and the pivot row times 1/pivot (lane k mc + j holds entry j)
            if (lane < kids) {
                const int p = mc + (lane & 1);
                const E pv = sh.buf(cur)[(lane >> 1) * m * xs(m) + p * xs(m) + p];
                const E mk = F::bmul(sh.mn(cur)[lane >> 1], pv, 0);
                sh.mn(nxt)[lane] = mk;
                ob[base + ((int64_t)s << (J + 1)) + lane] = mk;
                chk += F::fincheck(mk);
            }
            if constexpr (mc > 0) {
                if (lane < kids * mc) {
                    const int k = lane / mc, j = lane - k * mc, p = mc + (k & 1);
                    const E* P = &sh.buf(cur)[(k >> 1) * m * xs(m)];
                    sh.wk[lane] = F::rowscale(P[p * xs(m) + j], F::recip(P[p * xs(m) + p]));
                }
            }
        } else if constexpr (MODE == kXnor) {
            // child 2v drops node v's last block (minor unchanged), child 2v+1 keeps it (minor
            // times the pivot block's determinant; the inverse times the two pivot rows go to
            // wk[v][0..1][...], lane 2 v mc + r mc + j holding entry j of row r)
            if (lane < kids) {
                const E* P = &sh.buf(cur)[(lane >> 1) * m * xs(m)];
                E mk = sh.mn(cur)[lane >> 1];
                if (lane & 1)
                    mk = F::bmul(mk, F::det2(P[mc * xs(m) + mc], P[mc * xs(m) + mc + 1], P[(mc + 1) * xs(m) + mc],
                                             P[(mc + 1) * xs(m) + mc + 1]), 0);
                sh.mn(nxt)[lane] = mk;
                if constexpr (J == Q - 1) ob[((int64_t)s << Q) + lane] = mk;
                chk += F::fincheck(mk);
            }
            if constexpr (mc > 0) {
                if (lane < kids * mc) {
                    const int v = lane / (2 * mc), rr = lane - v * 2 * mc, r = rr / mc, j = rr - r * mc;
                    const E* P = &sh.buf(cur)[v * m * xs(m)];
                    const E a00 = P[mc * xs(m) + mc], a01 = P[mc * xs(m) + mc + 1];
                    const E a10 = P[(mc + 1) * xs(m) + mc], a11 = P[(mc + 1) * xs(m) + mc + 1];
                    const typename F::R rd = F::recip(F::det2(a00, a01, a10, a11));
                    const E p0 = P[mc * xs(m) + j], p1 = P[(mc + 1) * xs(m) + j];
                    sh.wk[lane] = r == 0 ? F::rowscale(F::upd(F::bmul(p0, a11, 0), a01, p1), rd)
                                         : F::rowscale(F::upd(F::bmul(p1, a00, 0), a10, p0), rd);
                }
            }
        } else {
            // NAND: child 3v + c of node v leaves the last block out (c = 0, minor unchanged)
            // or keeps its row mc + c - 1; the kept rows' pivot rows times 1/pivot go to
            // wk[v][c - 1][...] (lane 2 v mc + r mc + j holds entry j of row mc + r)
            // (formed with the true pivots; the shift test comes after the update pass)
            for (int t = lane; t < kids; t += 64) {
                const int v = t / 3, c = t - 3 * v;
                E mk = sh.mn(cur)[v];
                if (c) {
                    const int p = mc + c - 1;
                    mk = F::bmul(mk, sh.buf(cur)[v * m * xs(m) + p * xs(m) + p], 0);
                }
                sh.mn(nxt)[t] = mk;
                if constexpr (J == Q - 1) {
                    // leaves: written here unless the subtree's corrections come first
                    if (!xp.sub_mask) {
                        ob[(int64_t)s * pow3(Q) + t] = mk;
                        chk += F::fincheck(mk);
                    }
                } else {
                    chk += F::fincheck(mk);
                }
            }
            if constexpr (mc > 0) {
                static_assert(2 * (kids / 3) <= xsub_pairs_max() && 2 * (kids / 3) * mc <= 64 && kids <= 64,
                              "one pass per level");
                if (lane < 2 * (kids / 3) * mc) {
                    const int v = lane / (2 * mc), rr = lane - v * 2 * mc, r = rr / mc, j = rr - r * mc;
                    const E* P = &sh.buf(cur)[v * m * xs(m)];
                    const int p = mc + r;
                    const E pv = P[p * xs(m) + p], pj = P[p * xs(m) + j];
                    sh.wk[lane] = F::rowscale(pj, F::recip(pv));
                    const int ep = xexp(pv);
                    maybe = ep == 0 || max(xexp(pj), xexp(P[j * xs(m) + p])) >= ep + kFastExp;
                }
            }
        }
        wave_sync();
        if constexpr (mc > 0) xor_sub_update<F, Q, J, MODE>(sh);
        if constexpr (MODE == kNand && mc > 0) {
            // the NAND pivot shift test (Sec. II), consumed after the children are formed (its
            // inputs are long loaded by then).  Fast test: each lane of the pivot-row pass
            // compared the exponents of one row and one column entry of its kept row with
            // p's; if no lane found one kFastExp above, no pivot of this level is shifted.  Otherwise each kept row
            // is tested on its row and column maxima, and if any is shifted the level's kept
            // children are formed again with the shifted pivots (pvs).
            if (ballot(maybe)) {
                const int ns = nand_sub_slow<F, Q, J>(sh, xp.tau2, xp.es);
                if (ns) {
                    xp.nsh += ns;
                    xp.sub_mask |= 1 << J;
                }
            }
        }
        xor_sub<F, Q, J + 1, MODE>(2 * base + 2, s, ob, sh, chk, xp);   // XOR depth T+J+2 starts at 2^(T+J+2) - 2
    }
}

// NAND pivot corrections (Sec. II, pivot correction; Sec. III, NAND case: applied once the
// subtree below the shifted node is complete, deepest node first).  A kept row l whose pivot
// was shifted by C makes every minor of the child's subtree det A~[S]; the true minor is
// det A~[S] - C det A[S \ {l}], and S \ {l} is the entry with the same choices except block
// l left out: digit 0 instead of the child's digit c, i.e. c spans earlier in the ternary
// order.  The child's own entry (no deeper row kept) is not corrected: it is the parent's
// minor times the true pivot, kept aside when the shift is made (as the minors tree records
// a node's own minor with the true pivot).

// Subtree levels, on the 3^Q leaves in LDS: child x of level J + 1 (digits of the leaf
// index above the span 3^(Q - 1 - J)).
template <class F, int Q, int MODE>
__device__ __noinline__ void nand_sub_fix(XorLds<F, MODE>& sh, int es, int mask)
{
    using E = typename F::E;
    constexpr int nl = (int)pow3(Q);
    E* mn = sh.mn(Q & 1);
    const int lane = threadIdx.x;
    for (int J = Q - 2; J >= 0; --J) {
        if (!((mask >> J) & 1)) continue;
        int span = 1;
        for (int k = 0; k < Q - 1 - J; ++k) span *= 3;
        for (int t = lane; t < nl; t += 64) {
            const int x = t / span, c = x % 3;
            if (c) {
                const int code = sh.scode[xsub_code_base(J) + x];
                if (code != kNoEv) {
                    // the child's own entry (t = x span) takes its minor with the true pivot
                    mn[t] = t == x * span ? sh.sown[xsub_code_base(J) + x]
                                          : F::sub_scaled(mn[t], shift_value(es, code), mn[t - c * span]);
                }
            }
        }
        wave_sync();
    }
}

// Top levels: the children chosen by path sp at depths T-1 .. dlo, whose subtrees end with
// path sp, on the outputs in global memory (this wavefront's own stores).
template <class F, int N, int T, int Q>
__device__ __noinline__ double nand_top_fix(int dlo, int sp, typename F::E* ob, uint32_t tc, int es)
{
    const XPiv xp{0.0, es, 0, 0, false, tc};
    double chk = 0.0;
    using E = typename F::E;
    const int lane = threadIdx.x;
    constexpr int64_t q3 = pow3(Q);
    int64_t w = 1;                                  // top paths below a depth-D child: 3^(T-1-D)
    for (int D = T - 1; D >= dlo; --D, w *= 3) {
        const int code = xp.tcode(D);
        if (code == kNoEv) continue;
        wave_mem_fence();                           // the subtree's stores, and deeper corrections
        const int a = (int)((sp / w) % 3);
        const int64_t span = w * q3, base = (int64_t)(sp - sp % w) * q3;
        const double C = shift_value(xp.es, code);
        constexpr int kU = 2;
        for (int64_t i0 = base; i0 < base + span; i0 += 64 * kU) {
            E va[kU], vb[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int64_t i = i0 + lane + 64 * u;
                if (i < base + span && i != base) {
                    va[u] = ob[i];
                    vb[u] = ob[i - a * span];
                }
            }
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int64_t i = i0 + lane + 64 * u;
                if (i < base + span && i != base) {
                    const E r = F::sub_scaled(va[u], C, vb[u]);
                    ob[i] = r;
                    chk += F::fincheck(r);
                }
            }
        }
    }
    return chk;
}


// The tree of N <= 6 blocks below the node P0 (order 2N, row stride PS0) whose minor is
// sh.topm[0], by one wavefront: its minors to ob.  NAND: xp.top_own and sh.topown say whether
// the node itself was shifted.  Returns the check of the minors for non-finite ones.
template <class F, int N, int MODE, int PS0>
__device__ __forceinline__ double xor_tree(const typename F::E* P0, typename F::E* ob, XorLds<F, MODE>& sh, XPiv& xp)
{
    using E = typename F::E;
    constexpr int Q = N < xq(MODE) ? N : xq(MODE);
    constexpr int T = N - Q;
    static_assert(MODE == kNand || T == 0, "XOR and XNOR: no top levels");
    constexpr int w = 2 * N;
    const int lane = threadIdx.x;
    double chk = 0.0;
    xp.tc = 0;
    for (int e = lane; e < xzero_need(MODE); e += 64) sh.wz[e] = F::zero();
    constexpr int ntop = (int)pow3(T);
    for (int s = 0; s < ntop; ++s) {
        if constexpr (T > 0) {
            // top levels: redo the path below the first choice that changed from s - 1 (the
            // number of trailing zero digits of s)
            int d0 = 0;
            if (s) {
                int tz = 0;
                for (int t = s; t % 3 == 0; t /= 3) ++tz;
                d0 = T - 1 - tz;
                if (xp.tc) chk += nand_top_fix<F, N, T, Q>(d0, s - 1, ob, xp.tc, xp.es);
            }
            nand_top<F, N, T, 0, PS0>(d0, s, P0, sh, chk, xp);
        }
        // the subtree of depth-T node s, breadth first in LDS
        if constexpr (T == 0) {
            for (int e = lane; e < w * w; e += 64) sh.buf(0)[(e / w) * xs(w) + e % w] = P0[(e / w) * PS0 + e % w];
        }
        if (lane == 0) sh.mn(0)[0] = sh.topm[T];
        wave_sync();
        xp.sub_mask = 0;
        xor_sub<F, Q, 0, MODE>((int64_t(2) << T) - 2, s, ob, sh, chk, xp);
        if constexpr (MODE == kNand) {
            if (xp.sub_mask) {
                nand_sub_fix<F, Q, MODE>(sh, xp.es, xp.sub_mask);
                for (int t = lane; t < (int)pow3(Q); t += 64) {
                    const E v = sh.mn(Q & 1)[t];
                    ob[(int64_t)s * pow3(Q) + t] = v;
                    chk += F::fincheck(v);
                }
            }
            // a child shifted on this path: its own entry (leaf 0 of this subtree, written by
            // lane 0 above) with the true pivot
            if (xp.top_own) {
                xp.nsh += 1;
                if (lane == 0) {
                    ob[(int64_t)s * pow3(Q)] = sh.topown;
                    chk += F::fincheck(sh.topown);
                }
            }
            xp.top_own = false;
        }
    }
    if constexpr (MODE == kNand && T > 0) {
        if (xp.tc) chk += nand_top_fix<F, N, T, Q>(0, ntop - 1, ob, xp.tc, xp.es);
    }
    return chk;
}

// The block minors of matrix blockIdx.x (one wavefront).
template <class F, int N, int MODE>
__device__ __forceinline__ void xor_matrix(const typename F::E* __restrict__ A, typename F::E* __restrict__ out,
                                           int32_t* __restrict__ info, int32_t batch)
{
    using E = typename F::E;
    constexpr int w = 2 * N;
    __shared__ XorLds<F, MODE> sh;
    const int b = blockIdx.x;
    if (b >= batch) return;
    const int lane = threadIdx.x;
    const E* A0 = A + (int64_t)b * w * w;
    constexpr int64_t nout = MODE == kNand ? pow3(N) : MODE == kXnor ? (int64_t(1) << N) : (int64_t(2) << N) - 2;
    E* ob = out + (int64_t)b * nout;

    bool fin = true;
    double amax = 0.0;
    for (int e = lane; e < w * w; e += 64) {
        fin = fin && F::in_finite(A0[e]);
        amax = fmax(amax, F::mag(A0[e]));
    }
    if (!__all(fin ? 1 : 0)) {
        for (int64_t i = lane; i < nout; i += 64) F::store_nan(ob, nullptr, i, false);
        if (info && lane == 0) info[b] = -2;
        return;
    }
    XPiv xp{kDefaultPivTol * kDefaultPivTol, 0, 0, 0, false, 0};
    if constexpr (MODE == kNand) (void)frexp(wave_max(amax), &xp.es);
    if (lane == 0) sh.topm[0] = F::one();
    const double chk = xor_tree<F, N, MODE, w>(A0, ob, sh, xp);
    const bool bad = __any(chk == 0.0 ? 0 : 1);
    if (info && lane == 0) info[b] = bad ? -3 : xp.nsh;
}

template <class F, int N, int MODE>
__global__ __launch_bounds__(64) void xor_kernel(const typename F::E* __restrict__ A, typename F::E* __restrict__ out,
                                                 int32_t* __restrict__ info, int32_t batch)
{
    xor_matrix<F, N, MODE>(A, out, info, batch);
}

// fp64: registers capped for four wavefronts per SIMD (the compiler's choice holds three); a
// few spilled registers cost less than the residency gains.
template <int N, int MODE>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4))) void xor_kernel_r64(
    const double* __restrict__ A, double* __restrict__ out, int32_t* __restrict__ info, int32_t batch)
{
    xor_matrix<FR64, N, MODE>(A, out, info, batch);
}

template <class F, int N, int MODE>
constexpr auto xor_kernel_for()
{
    if constexpr (F::kId == FR64::kId)
        return xor_kernel_r64<N, MODE>;
    else
        return xor_kernel<F, N, MODE>;
}

// ------------------------------------------------------------ NAND parts (nand_parts.h)
// The levels above a part run in one buffer, a node in the place of its parent; the part's node
// (order 12) then is the root of a tree of six blocks, whose buffers take the same place.
template <class F, int N>
struct PartLds {
    static constexpr int kOrder = 2 * N - 2;
    struct Up {
        typename F::E path[kOrder * xs(kOrder)];
        typename F::E wv[kOrder];    // the pivot row times 1/pivot
    };
    union {
        XorLds<F, kNand> tree;
        Up up;
    };
    typename F::E root[12 * xs(12)];
};

// What a path's levels leave: the minor of its last node, the codes of its shifts, and whether
// the last kept block's pivot was shifted (own: the minor with the true pivot).
template <class F>
struct PartPath {
    typename F::E mk, own;
    uint64_t codes;
    bool top_own;
};

// Level D of the path to part q: level `first` is shifted, those above are not, those behind it
// are tested.
template <class F, int N, int D>
__device__ __forceinline__ void part_path(int q, int first, double tau2, int es, const typename F::E* A0, PartLds<F, N>& sh,
                                          PartPath<F>& pp)
{
    constexpr int L = nand_levels(N);
    if constexpr (D < L) {
        using E = typename F::E;
        constexpr int m = 2 * (N - D), mc = m - 2;
        constexpr int ps = D == 0 ? 2 * N : xs(2 * N - 2), cs = D == L - 1 ? xs(12) : xs(2 * N - 2);
        const E* P = D == 0 ? A0 : sh.up.path;
        E* C = D == L - 1 ? sh.root : sh.up.path;
        const int lane = threadIdx.x;
        const int a = (int)((q / pow3(L - 1 - D)) % 3);
        // lane h mc + i: columns [h cw, (h + 1) cw) of row i of the child; every load of the node
        // comes before the first store of the child, which takes its place
        constexpr int cw = top_cols(mc), H = (mc + cw - 1) / cw;
        constexpr bool kEven = mc % cw == 0;
        const int i = lane % mc, h = lane / mc, h0 = h * cw;
        const bool act = h < H;
        if (a != 0 || D == 0 || D == L - 1) {
            E row[cw];
            if (act) {
#pragma unroll
                for (int j = 0; j < cw; ++j)
                    if (kEven || h0 + j < mc) row[j] = P[i * ps + h0 + j];
            }
            if (a != 0) {
                const int p = mc + a - 1;
                E pv = P[p * ps + p], pc = F::zero(), pr = F::zero();
                if (act) pc = P[i * ps + p];
                if (lane < mc) pr = P[p * ps + lane];
                int code = kNoEv;
                if (D >= first) {
                    const double rmax = wave_max_nonneg(lane < mc ? F::mag(pr) : 0.0);
                    const double cmax = wave_max_nonneg(act ? F::mag(pc) : 0.0);
                    const double pm = F::mag(pv);
                    if (D == first || pm == 0.0 || pm * pm < tau2 * rmax * cmax) {
                        code = shift_code(rmax, cmax, es, F::re(pv) < 0.0);
                        pp.own = F::bmul(pp.mk, pv, 0);
                        pv = F::shift(pv, shift_value(es, code));
                    }
                }
                pp.codes |= (uint64_t)(uint8_t)code << (8 * D);
                pp.top_own = code != kNoEv;
                pp.mk = F::bmul(pp.mk, pv, 0);
                const typename F::R r = F::recip(pv);
                if (lane < mc) sh.up.wv[lane] = F::rowscale(pr, r);
                wave_sync();
                if (act) {
#pragma unroll
                    for (int j = 0; j < cw; ++j)
                        if (kEven || h0 + j < mc) row[j] = F::upd(row[j], pc, sh.up.wv[h0 + j]);
                }
            }
            wave_sync();
            if (act) {
#pragma unroll
                for (int j = 0; j < cw; ++j)
                    if (kEven || h0 + j < mc) C[i * cs + h0 + j] = row[j];
            }
            wave_sync();
        }
        part_path<F, N, D + 1>(q, first, tau2, es, A0, sh, pp);
    }
}

// Part q of a matrix (es: exponent of its largest magnitude), formed with shifts; returns the
// word, and the codes.
template <class F, int N>
__device__ __forceinline__ uint32_t nand_part(const typename F::E* __restrict__ A0, typename F::E* __restrict__ ob, int q,
                                              uint32_t word, int es, PartLds<F, N>& sh, uint64_t& codes)
{
    XPiv xp{kDefaultPivTol * kDefaultPivTol, es, 0, 0, false, 0};
    PartPath<F> pp{F::one(), F::zero(), 0, false};
    part_path<F, N, 0>(q, (int)(word & kPartFirst), xp.tau2, es, A0, sh, pp);
    if (threadIdx.x == 0) {
        sh.tree.topm[0] = pp.mk;
        sh.tree.topown = pp.own;
    }
    xp.top_own = pp.top_own;
    const double chk = xor_tree<F, 6, kNand, xs(12)>(sh.root, ob, sh.tree, xp);
    codes = pp.codes;
    const bool bad = __any(chk == 0.0 ? 0 : 1);
    return (word & (kPartFirst | kPartRedo)) | (bad ? kPartBad : 0u) | (uint32_t)xp.nsh << kPartShifts |
           (uint32_t)(es + kPartScaleBias) << kPartScale;
}

// Correction of a level whose nodes have sp parts each, on the nq parts of one wavefront: the
// minors of every part below a shifted node minus C times those of the part with that block
// left out.  sh: the place of the level's shift codes in those of the parts.
template <class F>
__device__ __noinline__ double part_group_fix(typename F::E* ob, int nq, int sp, int es, const uint64_t* codes, int sh)
{
    using E = typename F::E;
    constexpr int kU = 4;
    const int lane = threadIdx.x;
    double chk = 0.0;
    wave_mem_fence();                               // the parts' stores, and deeper corrections
    for (int q = 0; q < nq; ++q) {
        const int a = (q / sp) % 3, base = q - q % sp;
        const int cd = a ? (int)(int8_t)(codes[base] >> sh) : (int)kNoEv;
        if (cd == kNoEv) continue;
        const double C = shift_value(es, cd);
        E* x = ob + q * 729;
        const E* y = x - a * sp * 729;
        for (int i0 = 0; i0 < 729; i0 += 64 * kU) {
            E va[kU], vb[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int i = i0 + lane + 64 * u;
                if (i < 729) {
                    va[u] = x[i];
                    vb[u] = y[i];
                }
            }
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int i = i0 + lane + 64 * u;
                if (i < 729 && !(q == base && i == 0)) {   // (the node's own entry)
                    const E r = F::sub_scaled(va[u], C, vb[u]);
                    x[i] = r;
                    chk += F::fincheck(r);
                }
            }
        }
    }
    return chk;
}

// The marked parts.  Few: from the list, a part a wavefront.  If at least half of all parts are
// marked, groups of 3^group consecutive parts, taken in strides of the grid: the wavefront
// then applies the corrections of the levels inside the group as well, whose minors it has just
// stored (in a launch of their own they are bound by HBM, 220 us for 16000 complex zero-diagonal
// matrices of 7 blocks; here this launch takes its 790 us with and without them).
template <class F, int N>
__device__ __forceinline__ void nand_part_batch(const typename F::E* __restrict__ A, typename F::E* __restrict__ out,
                                                const NandWs& ws, int64_t parts, int group)
{
    constexpr int L = nand_levels(N), kParts = (int)pow3(L);
    __shared__ PartLds<F, N> sh;
    __shared__ uint64_t codes_s[9];
    const int lane = threadIdx.x;
    const int sub = (int)blockIdx.x & (ws.subs - 1);
    int marked = lane < ws.subs ? ws.head[lane * kHeadStride] : 0;
    const int in_sub = __builtin_amdgcn_readlane(marked, sub);
    marked = wave_sum(marked);
    if (2 * (int64_t)marked < parts) group = 0;
    if (blockIdx.x == 0 && lane == 0) {
        ws.head[kHeadRedo2] = marked;
        ws.head[kHeadBad2] = ws.head[kHeadBad];
        ws.head[kHeadGroup] = group;
    }
    const int in = group == 2 ? 9 : group == 1 ? 3 : 1;
    // (the grid is a multiple of the lists: wavefront i has list i mod subs, and with groups all)
    const int64_t items = group ? parts / in : in_sub, stride = group ? gridDim.x : gridDim.x / (unsigned)ws.subs;
    const uint32_t* list = ws.list + (int64_t)sub * ws.cap;
    for (int64_t i0 = group ? blockIdx.x : blockIdx.x / (unsigned)ws.subs; i0 < items; i0 += 64 * stride) {
        const int64_t it = i0 + lane * stride;
        int64_t mine = it * in;                     // the lane's first part
        bool due = it < items;
        if (due && group == 0) mine = list[it];
        if (due && group) {
            uint32_t any = 0;
            for (int k = 0; k < in; ++k) any |= ws.words[mine + k];
            due = (any & kPartRedo) != 0;
        }
        uint64_t todo = ballot(due);
        while (todo) {
            const int l = __builtin_ctzll(todo);
            todo &= todo - 1;
            const int64_t p0 = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)mine, l), b = p0 / kParts;
            const int q0 = (int)(p0 - b * kParts);
            const typename F::E* A0 = A + b * (4 * N * N);
            typename F::E* ob = out + b * pow3(N) + (int64_t)q0 * 729;
            double amax = 0.0;
            for (int e = lane; e < 4 * N * N; e += 64) amax = fmax(amax, F::mag(A0[e]));
            int es;
            (void)frexp(wave_max(amax), &es);
#pragma unroll 1
            for (int k = 0; k < in; ++k) {
                const uint32_t word = (uint32_t)__builtin_amdgcn_readfirstlane((int)ws.words[p0 + k]);
                uint64_t cd = 0;
                if (word & kPartRedo) {
                    const uint32_t w = nand_part<F, N>(A0, ob + k * 729, q0 + k, word, es, sh, cd);
                    if (lane == 0) {
                        ws.words[p0 + k] = w;
                        ws.codes[p0 + k] = cd;
                    }
                }
                if (group && lane == 0) codes_s[k] = cd;
                wave_sync();   // before the next part takes the place
            }
            double chk = 0.0;
            for (int g = 0; g < group; ++g)
                chk += part_group_fix<F>(ob, in, g ? 3 : 1, es, codes_s, 8 * (L - 1 - g));
            if (group && __any(chk == 0.0 ? 0 : 1) && lane == 0) ws.words[p0] |= kPartBad;
        }
    }
}

template <class F, int N>
__global__ __launch_bounds__(64) void nand_part_kernel(const typename F::E* __restrict__ A, typename F::E* __restrict__ out,
                                                       NandWs ws, int64_t parts, int group)
{
    nand_part_batch<F, N>(A, out, ws, parts, group);
}

// (as xor_kernel_r64)
template <int N>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4))) void nand_part_kernel_r64(
    const double* __restrict__ A, double* __restrict__ out, NandWs ws, int64_t parts, int group)
{
    nand_part_batch<FR64, N>(A, out, ws, parts, group);
}

// Corrections of the K levels D0 .. D0 + K - 1 at once, with 3^K minors in registers (the same
// place of the parts that differ in these levels' choices), on pieces y, y + ys, ... of 64 places
// of one matrix.  A thread reads and writes no other thread's minors of the piece, but those of
// other passes.
constexpr int kFixThreads = 512, kFixWaves = kFixThreads / 64;
constexpr int kFixPieces = (729 + 63) / 64;

template <class F, int L, int D0, int K>
__device__ __forceinline__ double fix_levels(typename F::E* ob, const uint32_t* wd, const uint64_t* cd, int es, int y, int ys,
                                             int pieces, int wave, int lane)
{
    using E = typename F::E;
    constexpr int V = (int)pow3(K), sp = (int)pow3(L - D0 - K), kUpper = (int)pow3(D0);
    double chk = 0.0;
    for (int t = wave; t < kUpper * sp * pieces; t += kFixWaves) {
        const int piece = t % pieces, ur = t / pieces, r = ur % sp, q0 = ur / sp * (V * sp) + r;
        const int i = (y + ys * piece) * 64 + lane;
        uint64_t code[V];
#pragma unroll
        for (int v = 1; v < V; ++v) {
            const int base = q0 - r + v * sp;
            code[v] = (wd[base] & kPartRedo) ? cd[base] >> (8 * D0) : 0;
        }
        E x[V];
        E* p = ob + (int64_t)q0 * 729 + i;
        if (i < 729) {
#pragma unroll
            for (int v = 0; v < V; ++v) x[v] = p[(int64_t)v * sp * 729];
        }
        uint32_t changed = 0;
#pragma unroll
        for (int k = K - 1; k >= 0; --k) {
            const int w = (int)pow3(K - 1 - k);
#pragma unroll
            for (int v = 1; v < V; ++v) {
                const int a = v / w % 3, first = v - v % w;     // first value below the node
                if (a == 0) continue;
                const int c = (int)(int8_t)(code[first] >> (8 * k));
                if (c == kNoEv || (v == first && r == 0 && i == 0)) continue;   // (the node's own entry)
                x[v] = F::sub_scaled(x[v], shift_value(es, c), x[v - a * w]);
                changed |= 1u << v;
            }
        }
        if (i < 729) {
#pragma unroll
            for (int v = 1; v < V; ++v)
                if ((changed >> v) & 1) {
                    p[(int64_t)v * sp * 729] = x[v];
                    chk += F::fincheck(x[v]);
                }
        }
    }
    return chk;
}

// Levels 0 .. M - 1, deepest first, two at a time.
template <class F, int L, int M>
__device__ __forceinline__ double fix_passes(typename F::E* ob, const uint32_t* wd, const uint64_t* cd, int es, int y, int ys,
                                             int pieces, int wave, int lane)
{
    if constexpr (M <= 0) {
        return 0.0;
    } else {
        constexpr int K = M >= 2 ? 2 : 1;
        const double chk = fix_levels<F, L, M - K, K>(ob, wd, cd, es, y, ys, pieces, wave, lane);
        __syncthreads();                               // the next pass reads these
        return chk + fix_passes<F, L, M - K>(ob, wd, cd, es, y, ys, pieces, wave, lane);
    }
}

// Corrections of the levels above the groups of nand_part_batch, and info.  A wavefront looks
// through the words of a matrix; the workgroup then corrects the matrices that need it, one after
// the other.  blockIdx.y: see fix_levels.
template <class F, int N>
__global__ __launch_bounds__(kFixThreads) void nand_fix_kernel(typename F::E* __restrict__ out, int32_t* __restrict__ info,
                                                               NandWs ws, int32_t batch)
{
    using E = typename F::E;
    constexpr int L = nand_levels(N), kParts = (int)pow3(L);
    __shared__ int levels_s[kFixWaves];        // whether a matrix has a shift in these levels
    __shared__ int scale_s[kFixWaves];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    if (blockIdx.x == 0 && blockIdx.y == 0) {
        if (threadIdx.x < kSubLists) ws.head[threadIdx.x * kHeadStride] = 0;
        if (threadIdx.x == 0) ws.head[kHeadBad] = 0;
    }
    if ((ws.head[kHeadRedo2] | ws.head[kHeadBad2]) == 0) return;
    const int levels = L - ws.head[kHeadGroup];
    const uint64_t mask = levels > 0 ? ~0ull >> (64 - 8 * levels) : 0;
    const int y = blockIdx.y, ys = gridDim.y, pieces = (kFixPieces - y + ys - 1) / ys;
    for (int64_t b0 = (int64_t)blockIdx.x * kFixWaves; b0 < batch; b0 += (int64_t)gridDim.x * kFixWaves) {
        const int64_t bw = b0 + wave;
        uint32_t bad = 0;
        int shifts = 0, scale = 0;
        uint64_t codes = 0;
        for (int q = lane; bw < batch && q < kParts; q += 64) {
            const uint32_t w = ws.words[bw * kParts + q];
            bad |= w & kPartBad;
            if (w & kPartRedo) {
                shifts += (int)(w >> kPartShifts & 0xFFFu);
                scale = (int)(w >> kPartScale);
                codes |= ws.codes[bw * kParts + q] & mask;
            }
        }
        const bool any_bad = ballot(bad != 0) != 0, redo = ballot(scale != 0) != 0;
        if (any_bad || redo) {
            for (int o = 32; o > 0; o >>= 1) {
                shifts += __shfl_xor(shifts, o);
                scale = max(scale, __shfl_xor(scale, o));
            }
            // info is 0 here, or -3 from another piece
            if (info && lane == 0 && y == 0) {
                if (any_bad)
                    atomicMin(&info[bw], -3);
                else
                    atomicCAS(&info[bw], 0, shifts);
            }
        }
        const bool shifted = ballot(codes != 0) != 0;
        if (lane == 0) {
            levels_s[wave] = shifted;
            scale_s[wave] = scale - kPartScaleBias;
        }
        __syncthreads();
        for (int v = 0; v < kFixWaves; ++v) {
            if (levels_s[v] == 0) continue;
            const int64_t b = b0 + v;
            E* ob = out + b * pow3(N);
            const uint32_t* wd = ws.words + b * kParts;
            const uint64_t* cd = ws.codes + b * kParts;
            const double chk = levels == L       ? fix_passes<F, L, L>(ob, wd, cd, scale_s[v], y, ys, pieces, wave, lane)
                               : levels == L - 1 ? fix_passes<F, L, L - 1>(ob, wd, cd, scale_s[v], y, ys, pieces, wave, lane)
                                                 : fix_passes<F, L, L - 2>(ob, wd, cd, scale_s[v], y, ys, pieces, wave, lane);
            if (info && ballot(chk != 0.0 || chk != chk) && lane == 0) atomicMin(&info[b], -3);
        }
        __syncthreads();                               // before levels_s is written again
    }
}

template <class F, int N>
constexpr auto nand_part_kernel_for()
{
    if constexpr (F::kId == FR64::kId)
        return nand_part_kernel_r64<N>;
    else
        return nand_part_kernel<F, N>;
}

// The launches behind the register kernel.  Groups (if most parts are marked): the largest that
// take about as long as single parts would, in rounds of wavefronts times parts, within a tenth.
template <class F, int N>
hipError_t nand_parts_launch(const LaunchXor& L, hipStream_t st)
{
    if constexpr (N > 13) {
        return hipErrorInvalidValue;
    } else {
        if (L.n != N) return nand_parts_launch<F, N + 1>(L, st);
        constexpr int kLevels = nand_levels(N);
        // per CU: four wavefronts per SIMD (fp64); 11 by LDS, from 11 blocks on two per SIMD by registers
        constexpr int64_t kWaves = kCus * (F::kComplex ? (N >= 11 ? 8 : 11) : 16);
        const int64_t parts = (int64_t)L.batch * pow3(kLevels);
        auto rounds = [&](int g) { return (parts / pow3(g) + kWaves - 1) / kWaves * pow3(g); };
        const int most = kLevels < 2 ? kLevels : 2;
        int64_t least = rounds(0);
        for (int g = 1; g <= most; ++g) least = rounds(g) < least ? rounds(g) : least;
        int group = most;
        while (group > 0 && 10 * rounds(group) > 11 * least) --group;
        static_assert(kWaves % kSubLists == 0, "the same number of wavefronts for every list");
        const int64_t waves = parts < kWaves ? (parts + L.nand.subs - 1) / L.nand.subs * L.nand.subs : kWaves;
        hipLaunchKernelGGL((nand_part_kernel_for<F, N>()), dim3((unsigned)waves), dim3(64), 0, st,
                           static_cast<const typename F::E*>(L.A), static_cast<typename F::E*>(L.out), L.nand, parts, group);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        // wavefronts that look through the words; more pieces where the matrices are few
        constexpr int64_t kGroups = 512;
        const int64_t need = ((int64_t)L.batch + kFixWaves - 1) / kFixWaves, gx = need < kGroups ? need : kGroups;
        const int64_t gy = kGroups / gx < kFixPieces ? kGroups / gx : kFixPieces;
        hipLaunchKernelGGL((nand_fix_kernel<F, N>), dim3((unsigned)gx, (unsigned)gy), dim3(kFixThreads), 0, st,
                           static_cast<typename F::E*>(L.out), L.info, L.nand, L.batch);
        return hipGetLastError();
    }
}

template <class F, int N>
hipError_t xor_launch_n(const LaunchXor& L, hipStream_t st)
{
    if constexpr (N >= kNandRowMin) {
        return hipErrorInvalidValue;
    } else {
        if (L.n != N) return xor_launch_n<F, N + 1>(L, st);
        auto go = [&](auto kern) {
            hipLaunchKernelGGL(kern, dim3((unsigned)L.batch), dim3(64), 0, st, static_cast<const typename F::E*>(L.A),
                               static_cast<typename F::E*>(L.out), L.info, L.batch);
        };
        if (L.mode == kNand) {
            go(xor_kernel_for<F, N, kNand>());
        } else if constexpr (N < kRowMin) {
            if (L.mode == kXnor)
                go(xor_kernel_for<F, N, kXnor>());
            else
                go(xor_kernel_for<F, N, kXor>());
        } else {
            return hipErrorInvalidValue;
        }
        return hipGetLastError();
    }
}

}  // namespace

size_t nand_ws_bytes(int n, int64_t batch)
{
    if (n < kNandRowMin) return 0;
    return kNandHeadBytes + (size_t)(pow3(nand_levels(n)) * batch) * 12 +
           (size_t)((nand_row_waves(n, batch) + kSubLists) * kRowParts) * 4;
}

NandWs nand_ws_carve(void* ws, int n, int64_t batch)
{
    const int64_t parts = pow3(nand_levels(n)) * batch;
    NandWs w;
    w.head = static_cast<int32_t*>(ws);
    w.codes = reinterpret_cast<uint64_t*>(static_cast<char*>(ws) + kNandHeadBytes);
    w.words = reinterpret_cast<uint32_t*>(w.codes + parts);
    w.list = w.words + parts;
    // (a list for 32 wavefronts or more)
    const int64_t waves = nand_row_waves(n, batch);
    w.subs = 1;
    while (w.subs < kSubLists && waves >= 64 * (int64_t)w.subs) w.subs *= 2;
    w.cap = (int32_t)((waves + w.subs - 1) / w.subs * kRowParts);
    return w;
}

hipError_t xor_launch(const LaunchXor& L, hipStream_t st)
{
    if (L.dtype != 0 && L.dtype != 2) return hipErrorInvalidValue;
    if (L.mode != kNand && L.n >= kRowMin) {
        if (L.mode == kXor) return L.dtype == 0 ? xor_row_launch_r64(L, st) : xor_row_launch_c128(L, st);
        return L.dtype == 0 ? xnor_row_launch_r64(L, st) : xnor_row_launch_c128(L, st);
    }
    if (L.mode == kNand && L.n >= kNandRowMin) {
        const hipError_t e = L.dtype == 0 ? nand_row_launch_r64(L, st) : nand_row_launch_c128(L, st);
        if (e != hipSuccess) return e;
        return L.dtype == 0 ? nand_parts_launch<FR64, kNandRowMin>(L, st) : nand_parts_launch<FC128, kNandRowMin>(L, st);
    }
    return L.dtype == 0 ? xor_launch_n<FR64, 1>(L, st) : xor_launch_n<FC128, 1>(L, st);
}

}  // namespace apm
