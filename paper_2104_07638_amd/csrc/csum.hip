// csum.hip -- CDet connected sums (Sec. V.A, Eq. (recursion)) on gfx950.
//
//   c[S] = a[S] - sum_{T subsetneq S, j in T} c[T] a[S \ T],   a[S] = m_up[S] m_dn[S].
//
// For a distinguished vertex j write S = {j} + X and T = {j} + Y with X, Y subsets of the
// vertices above j (m = n-1-j bits).  Then, with c'[X] = c[{j}+X], a0[X] = a[{j}+X] and
// b[U] = a[U] (U above j, nonempty),
//
//   c'[X] = a0[X] - sum_{Y subsetneq X} c'[Y] b[X \ Y]                          (*)
//
// a triangular subset convolution of 3^m multiply-adds.  Rooted mode solves (*) for j = 0;
// "all" mode solves it for every j (independent problems, one workgroup each).
//
// Blocking:
//   * problems of at most 10 bits: one wavefront, b and the right-hand side in LDS, the result
//     in place of the right-hand side.  X = (Xh, Xl) with Xl the low LB bits held in registers
//     (LB = 4, or 3 up to 9 bits): one (Xh, Yh) pair is an LB-bit subset convolution of two rows
//     of 2^LB values (27 FMAs for 16 loaded values, 81 for 32).  The pairs of a row are split
//     over G lanes and summed with DPP row shifts, rank by rank (|Xh|).
//   * larger problems: blocks of 2^11 values, csum_blocks.h (csum_walk.h for Monte Carlo).
//   * rows in LDS are padded (see the layouts below), so that lanes reading different rows at
//     the same column spread over the LDS banks.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "apm_device.h"
#include "apm_kernels.h"

namespace apm {
namespace {

// c[x] = r[x] - sum_{y subsetneq x} c[y] g0[x \ y], x in increasing order (in place on r).
template <int LB>
__device__ __forceinline__ void tri_tile(double (&r)[1 << LB], const double (&g0)[1 << LB])
{
    constexpr int W = 1 << LB;
#pragma unroll
    for (int x = 1; x < W; ++x)
#pragma unroll
        for (int y = 0; y < W; ++y)
            if ((y & ~x) == 0 && y != x) r[x] = fma(-r[y], g0[x ^ y], r[x]);
}

template <int HB>
__device__ __forceinline__ void conv_half(const double (&f)[1 << HB], const double (&g)[1 << HB], double* acc)
{
    constexpr int W = 1 << HB;
#pragma unroll
    for (int x = 0; x < W; ++x)
#pragma unroll
        for (int y = 0; y < W; ++y)
            if ((y & ~x) == 0) acc[x] = fma(-f[y], g[x ^ y], acc[x]);
}

template <int W>
__device__ __forceinline__ void ld_row_at(const double* buf, uint32_t off, double (&v)[W])
{
#pragma unroll
    for (int p = 0; p < W / 2; ++p) {
        const double2 t = *reinterpret_cast<const double2*>(reinterpret_cast<const char*>(buf) + off + 16 * p);
        v[2 * p] = t.x;
        v[2 * p + 1] = t.y;
    }
}

// v += v of the lane DELTA below (0 if outside the row of 16 / the group), for doubles.
template <int CTRL, int ROWMASK = 0xF>
__device__ __forceinline__ double dpp_add(double v)
{
    const int lo = __double2loint(v), hi = __double2hiint(v);
    const int slo = __builtin_amdgcn_update_dpp(0, lo, CTRL, ROWMASK, 0xF, true);
    const int shi = __builtin_amdgcn_update_dpp(0, hi, CTRL, ROWMASK, 0xF, true);
    return v + __hiloint2double(shi, slo);
}

// Sum over aligned groups of G consecutive lanes; the total lands in the LAST lane of
// each group.  row_shr:k (0x110 + k) shifts within rows of 16 lanes; row_bcast:15 (0x142)
// and row_bcast:31 (0x143) carry row ends across rows.
template <int W>
__device__ __forceinline__ void group_sum(double (&acc)[W], int G)
{
    if (G >= 2) {
#pragma unroll
        for (int i = 0; i < W; ++i) acc[i] = dpp_add<0x111>(acc[i]);
    }
    if (G >= 4) {
#pragma unroll
        for (int i = 0; i < W; ++i) acc[i] = dpp_add<0x112>(acc[i]);
    }
    if (G >= 8) {
#pragma unroll
        for (int i = 0; i < W; ++i) acc[i] = dpp_add<0x114>(acc[i]);
    }
    if (G >= 16) {
#pragma unroll
        for (int i = 0; i < W; ++i) acc[i] = dpp_add<0x118>(acc[i]);
    }
    if (G >= 32) {
#pragma unroll
        for (int i = 0; i < W; ++i) acc[i] = dpp_add<0x142, 0xA>(acc[i]);
    }
    if (G >= 64) {
#pragma unroll
        for (int i = 0; i < W; ++i) acc[i] = dpp_add<0x143, 0xC>(acc[i]);
    }
}

struct CsArgs {
    const double* up;
    const double* dn;
    double* c;
    int weights;       // m_up already holds a[]
    double* summ;      // rooted problems of at most 11 bits: (c[V], d[V]) per matrix instead of c[]
};

// a[S] from the inputs
__device__ __forceinline__ double weight(const CsArgs& g, int64_t base, int64_t S)
{
    const double u = g.up[base + S];
    if (g.weights) return u;
    return u * (g.dn ? g.dn[base + S] : u);
}

// Problems of at most 10 bits: rows of 2^LB values in registers, H row bits.
template <int M>
struct CsPlan {
    static constexpr int LBW = M <= 9 ? 3 : 4;
    static constexpr int LB = M < LBW ? M : LBW;
    static constexpr int H = M - LB;
    static constexpr int ROWS = 1 << H;
    // Rows in LDS are 16 bytes apart beyond their length, so that lanes reading different rows at
    // one column spread over the banks.
    static constexpr int ROW = 8 * ((1 << LB) + (LB > 0 ? 2 : 0));           // bytes from a row to the next
    static constexpr int LEN = ROWS * ROW / 8;                               // values of a block
    // value x1 of a block
    __device__ static __forceinline__ int at(int x1) { return (x1 >> LB) * (ROW / 8) + (x1 & ((1 << LB) - 1)); }
};

// The fixed schedule of a problem: for every rank r >= 1 its rows, G lanes a row (G the largest
// power of two with rows G <= 32 that the pairs of a row fill), and each lane's pairs step by
// step.  The LDS offsets of a pair's two rows are one table entry per step and lane (c' row in
// the low half, b row in the high half), loaded once at the start of the problem, so a step is
// its LDS reads and multiply-adds; computing Yh and the offsets from the lane number took twice
// the instructions of the multiply-adds.  A lane without a pair in a step is masked:
// reading a row of zeros instead kept the banks busier, and the blocks of 9 bits with such rows took
// 10.6 KB, 14 wavefronts per CU instead of 16 (8192 problems 35.3 -> 32.7 us).
// The order of the rows over the lanes is free within a rank: for 64 rows it was searched for the
// fewest reads of one bank by the 16 lanes that a 16-byte read serves at a time (121 cycles a
// problem for the reads of all ranks, 152 in order of the row numbers).
struct RowOrder {
    uint8_t row[64];
};
constexpr RowOrder kRowOrder9 = {
    {0, 16, 1, 4, 8, 2, 32, 33, 5, 20, 9, 10, 12, 34, 36, 17, 24, 3, 6, 48, 40, 18,
     21, 11, 41, 37, 42, 13, 22, 19, 35, 38, 26, 25, 28, 14, 44, 49, 50, 52, 7, 56, 57, 30,
     27, 54, 23, 58, 60, 29, 46, 39, 15, 53, 51, 45, 43, 62, 61, 59, 55, 31, 47, 63}};
constexpr RowOrder kRowOrder10 = {
    {0, 4, 1, 8, 16, 2, 32, 33, 40, 10, 6, 18, 24, 48, 5, 20, 17, 9, 36, 34, 12, 3,
     13, 28, 42, 49, 38, 14, 26, 21, 44, 37, 19, 22, 11, 25, 41, 50, 52, 56, 35, 7, 29, 60,
     53, 27, 58, 30, 23, 57, 46, 15, 51, 45, 39, 43, 54, 55, 59, 61, 62, 31, 47, 63}};

template <int M>
struct OneWave {
    using CP = CsPlan<M>;
    static constexpr int H = CP::H, W = 1 << CP::LB;
    static constexpr int rows(int r)
    {
        int c = 1;
        for (int i = 0; i < r; ++i) c = c * (H - i) / (i + 1);
        return c;
    }
    static constexpr int items(int r) { return (1 << r) - 1; }
    static constexpr int lanes(int r)
    {
        int g = 1;
        while (g * 2 <= kWave && rows(r) * g * 2 <= kWave && g * 2 <= (items(r) > 0 ? items(r) : 1)) g *= 2;
        return g;
    }
    static constexpr int steps(int r) { return (items(r) + lanes(r) - 1) / lanes(r); }
    static constexpr int first(int r)
    {
        int s = 0;
        for (int i = 1; i < r; ++i) s += steps(i);
        return s;
    }
    static constexpr int total = first(H + 1);
    static constexpr uint32_t kNone = 0xFFFFFFFFu;
    // every lane has a pair in step k of rank r
    static constexpr bool full(int r, int k) { return rows(r) * lanes(r) == kWave && lanes(r) * (k + 1) <= items(r); }
    struct Table {
        uint32_t pair[total > 0 ? total : 1][kWave];
        uint16_t row[H + 1][kWave];      // offset of the lane's row, 0xFFFF: none
    };
    static constexpr int bits(int x)
    {
        int c = 0;
        for (; x; x &= x - 1) ++c;
        return c;
    }
    static constexpr Table make()
    {
        Table t{};
        for (int r = 0; r <= H; ++r) {
            int o = 0;
            const int g = lanes(r);
            for (int l = 0; l < kWave; ++l) {
                t.row[r][l] = 0xFFFF;
                for (int k = 0; r > 0 && k < steps(r); ++k)
                    t.pair[first(r) + k][l] = kNone;
            }
            for (int i = 0; i < CP::ROWS; ++i) {
                const int x = H < 6 ? i : (M == 9 ? kRowOrder9.row[i] : kRowOrder10.row[i]);
                if (bits(x) != r) continue;
                // the lowest log2(g) bits of x take the bits of the lane in the group
                int low[8] = {}, hi = x, nl = 0;
                for (int q = 1; q < g; q <<= 1) {
                    low[nl++] = hi & -hi;
                    hi &= hi - 1;
                }
                for (int s = 0; s < g; ++s) {
                    int ys = 0;
                    for (int q = 0; q < nl; ++q)
                        if ((s >> q) & 1) ys |= low[q];
                    t.row[r][o * g + s] = (uint16_t)(x * CP::ROW);
                    int z = 0;
                    for (int k = 0; r > 0 && k < steps(r); ++k, z = (z - hi) & hi) {
                        if (s + g * k >= items(r)) continue;
                        const int y = ys | z;
                        t.pair[first(r) + k][o * g + s] = (uint32_t)(y * CP::ROW) | ((uint32_t)((x ^ y) * CP::ROW) << 16);
                    }
                }
                ++o;
            }
        }
        return t;
    }
};

template <int M>
__constant__ typename OneWave<M>::Table kOneWave = OneWave<M>::make();

// Ranks R .. H of the triangular solve in place on the c' block.
template <int M, int R, int TOT>
__device__ __forceinline__ void one_wave_ranks(const uint32_t (&pair)[TOT], const uint32_t (&row)[OneWave<M>::H + 1],
                                               double* cb, const double* bb)
{
    using OW = OneWave<M>;
    constexpr int LB = CsPlan<M>::LB, W = OW::W;
    if constexpr (R <= OW::H) {
        double acc[W];
#pragma unroll
        for (int i = 0; i < W; ++i) acc[i] = 0.0;
        if constexpr (R > 0) {
#pragma unroll
            for (int k = 0; k < OW::steps(R); ++k) {
                const uint32_t e = pair[OW::first(R) + k];
                if (!OW::full(R, k) && e == OW::kNone) continue;
                double f[W], g[W];
                ld_row_at<W>(cb, e & 0xFFFFu, f);
                ld_row_at<W>(bb, e >> 16, g);
                conv_half<LB - 1>(reinterpret_cast<const double(&)[W / 2]>(f), reinterpret_cast<const double(&)[W / 2]>(g), acc);
                conv_half<LB - 1>(reinterpret_cast<const double(&)[W / 2]>(f),
                                  reinterpret_cast<const double(&)[W / 2]>(g[W / 2]), acc + W / 2);
                conv_half<LB - 1>(reinterpret_cast<const double(&)[W / 2]>(f[W / 2]),
                                  reinterpret_cast<const double(&)[W / 2]>(g), acc + W / 2);
            }
            group_sum<W>(acc, OW::lanes(R));
        }
        constexpr int G = OW::lanes(R);
        if (row[R] != 0xFFFFu && ((int)threadIdx.x & (G - 1)) == G - 1) {
            double rr[W], g0[W];
            ld_row_at<W>(cb, row[R], rr);
            ld_row_at<W>(bb, 0, g0);
#pragma unroll
            for (int i = 0; i < W; ++i) rr[i] += acc[i];
            tri_tile<LB>(rr, g0);
#pragma unroll
            for (int p = 0; p < W / 2; ++p)
                *reinterpret_cast<double2*>(reinterpret_cast<char*>(cb) + row[R] + 16 * p) =
                    make_double2(rr[2 * p], rr[2 * p + 1]);
        }
        __syncthreads();
        one_wave_ranks<M, R + 1>(pair, row, cb, bb);
    }
}

// Problem (matrix at base, root j): solve (*) for the M = n-1-j vertices above j.
template <int M>
__device__ void cs_problem(const CsArgs& g, int64_t base, int j, bool zero_even, double* lds_c, double* lds_b)
{
    using CP = CsPlan<M>;
    using OW = OneWave<M>;
    constexpr int N = 1 << M, IT = (N + kWave - 1) / kWave, full = N - 1;
    const int tid = (int)threadIdx.x;
    const int jsh = j + 1;                          // X -> S = (1 << j) | (X << (j+1))
    double* c = g.c;
    if constexpr (M == 0) {
        // one vertex: c'[empty] = a[{j}]
        if (tid == 0) {
            const double a = weight(g, base, int64_t(1) << j);
            if (g.summ) {
                g.summ[0] = a;
                g.summ[1] = fabs(a);
                return;
            }
            c[base + (int64_t(1) << j)] = a;
            if (j == 0) c[base] = 0.0;   // c[empty] = 0
        }
        return;
    } else {
        uint32_t pair[OW::total > 0 ? OW::total : 1], row[OW::H + 1];
#pragma unroll
        for (int k = 0; k < OW::total; ++k) pair[k] = kOneWave<M>.pair[k][tid];
#pragma unroll
        for (int r = 0; r <= OW::H; ++r) row[r] = kOneWave<M>.row[r][tid];
        if (j == 0 && !(base & 1)) {
            // rooted problem: a0[x] = a[2x + 1] and b[x] = a[2x] are neighbours, so one 16-byte load
            // per x stages both; the loads of CH entries are issued before their stores (one
            // memory round trip per CH entries instead of per entry)
            constexpr int CH = IT < 4 ? IT : 4;
            const bool two = !g.weights && g.dn;
#pragma unroll
            for (int i0 = 0; i0 < IT; i0 += CH) {
                double2 u[CH], d[CH];
#pragma unroll
                for (int i = 0; i < CH; ++i) {
                    const int x1 = tid + (i0 + i) * kWave;
                    if (x1 < N) {
                        u[i] = *reinterpret_cast<const double2*>(g.up + base + 2 * x1);
                        if (two) d[i] = *reinterpret_cast<const double2*>(g.dn + base + 2 * x1);
                    }
                }
#pragma unroll
                for (int i = 0; i < CH; ++i) {
                    const int x1 = tid + (i0 + i) * kWave;
                    if (x1 < N) {
                        double w0, w1;
                        if (g.weights) {
                            w0 = u[i].x;
                            w1 = u[i].y;
                        } else if (two) {
                            w0 = u[i].x * d[i].x;
                            w1 = u[i].y * d[i].y;
                        } else {
                            w0 = u[i].x * u[i].x;
                            w1 = u[i].y * u[i].y;
                        }
                        lds_b[CP::at(x1)] = x1 ? w0 : 0.0;
                        lds_c[CP::at(x1)] = w1;
                    }
                }
            }
        } else {
            for (int x1 = tid; x1 < N; x1 += kWave) {
                lds_c[CP::at(x1)] = weight(g, base, (int64_t(1) << j) | ((int64_t)x1 << jsh));
                lds_b[CP::at(x1)] = x1 ? weight(g, base, (int64_t)x1 << jsh) : 0.0;
            }
        }
        __syncthreads();
        // a[V] for the summary (the in-place solve overwrites it)
        const double a_full = g.summ ? lds_c[CP::at(full)] : 0.0;
        one_wave_ranks<M, 0>(pair, row, lds_c, lds_b);
        if (g.summ) {
            // only the full-set value and the recursion's rounding scale at it:
            // d[V] = |a[V]| + sum_{X full-exclusive} |c'[X]| |b[full \ X]|, with a[V] = a0[full]
            double part = 0.0;
            for (int x1 = tid; x1 < full; x1 += kWave) part += fabs(lds_c[CP::at(x1)]) * fabs(lds_b[CP::at(full ^ x1)]);
            for (int o = kWave / 2; o > 0; o >>= 1) part += __shfl_xor(part, o);
            if (tid == 0) {
                g.summ[0] = lds_c[CP::at(full)];
                g.summ[1] = fabs(a_full) + part;
            }
            return;
        }
        if (zero_even && !(base & 1)) {
            // rooted problem: write (c[2x] = 0, c[2x+1] = c'[x]) as one 16-byte store
            for (int x1 = tid; x1 < N; x1 += kWave)
                *reinterpret_cast<double2*>(c + base + 2 * x1) = make_double2(0.0, lds_c[CP::at(x1)]);
        } else {
            for (int x1 = tid; x1 < N; x1 += kWave) {
                c[base + (int64_t(1) << j) + ((int64_t)x1 << jsh)] = lds_c[CP::at(x1)];
                if (zero_even) c[base + 2 * x1] = 0.0;
            }
        }
        if (j == 0 && tid == 0) c[base] = 0.0;   // c[empty] = 0
    }
}

// The problems of a launch: matrix b (through the size-sorted queue order when given) with the
// roots j0 .. j0 + roots - 1.
struct CsMap {
    int32_t batch;
    int n_uniform;
    const int32_t* nv;
    const int64_t* off;
    const int32_t* order;   // mixed-order rooted batches: matrix indices by decreasing order, else NULL
    int j0, roots;
    bool rooted;            // rooted mode: also c[S] = 0 for the sets without vertex 0
};

#include "csum_blocks.h"
#include "csum_walk.h"

// One problem per workgroup of one wavefront: those of LO to HI bits (the workgroups of others
// end).  One order: a kernel for each number of bits.  Several: a launch that few problems of it
// fill costs 4.7 us, so 0 to 7 bits, 8 and 9 (twice the registers, four times the LDS) and 10
// share one each.
template <int LO, int HI>
constexpr int cs_len()
{
    if constexpr (LO > HI) {
        return 0;
    } else {
        return CsPlan<LO>::LEN > cs_len<LO + 1, HI>() ? CsPlan<LO>::LEN : cs_len<LO + 1, HI>();
    }
}

template <int M, int HI>
__device__ __forceinline__ void cs_dispatch(int m, const CsArgs& g, int64_t base, int j, bool rooted, double* lds_c, double* lds_b)
{
    if constexpr (M <= HI) {
        if (m == M) return cs_problem<M>(g, base, j, rooted, lds_c, lds_b);
        cs_dispatch<M + 1, HI>(m, g, base, j, rooted, lds_c, lds_b);
    }
}

template <int LO, int HI>
__global__ __launch_bounds__(kWave) void cs_kernel(CsArgs g, CsMap mp)
{
    __shared__ __align__(16) double lds_c[cs_len<LO, HI>()];
    __shared__ __align__(16) double lds_b[cs_len<LO, HI>()];
    int b = (int)(blockIdx.x / (unsigned)mp.roots);
    const int j = mp.j0 + (int)(blockIdx.x - (unsigned)b * (unsigned)mp.roots);
    if (mp.order) b = mp.order[b];
    const int n = mp.n_uniform > 0 ? mp.n_uniform : mp.nv[b];
    const int m = n - 1 - j;
    if (m < LO || m > HI) return;
    const int64_t base = mp.off ? mp.off[b] : ((int64_t)b << n);
    CsArgs gb = g;
    if (gb.summ) gb.summ += 2 * (int64_t)b;
    cs_dispatch<LO, HI>(m, gb, base, j, mp.rooted, lds_c, lds_b);
}

// Every problem of 11 bits or more in one launch, largest first, so that the shorter problems
// fill the end of the launch: the queue order for mixed-order rooted batches, root by root
// otherwise.
template <BlockWeights K>
__global__ __launch_bounds__(kBlockThreads) __attribute__((amdgpu_waves_per_eu(5))) void cs_block_kernel(CsArgs g, CsMap mp)
{
    __shared__ __align__(16) double lds_c[kBlockLen];
    __shared__ __align__(16) double lds_b[kBlockLen];
    const int j = (int)(blockIdx.x / (unsigned)mp.batch);
    int b = (int)(blockIdx.x - (unsigned)j * (unsigned)mp.batch);
    if (mp.order) b = mp.order[b];
    const int n = mp.n_uniform > 0 ? mp.n_uniform : mp.nv[b];
    const int m = n - 1 - j;
    if (m < kBlockBits) return;
    const int64_t base = mp.off ? mp.off[b] : ((int64_t)b << n);
    block_problem<K>(g, base, j, m, mp.rooted, lds_c, lds_b);
}

template <BlockWeights K>
hipError_t launch_blocks(int64_t problems, const CsArgs& g, const CsMap& mp, hipStream_t st)
{
    hipLaunchKernelGGL(cs_block_kernel<K>, dim3((unsigned)problems), dim3(kBlockThreads), 0, st, g, mp);
    return hipGetLastError();
}

// The problems of LO to HI bits of a launch; all modes, orders up to nmax.
template <int LO, int HI>
hipError_t launch_range(const CsArgs& g, CsMap mp, int nmax, hipStream_t st)
{
    if (!mp.rooted) {
        mp.j0 = mp.n_uniform > 0 && nmax - 1 > HI ? nmax - 1 - HI : 0;
        mp.roots = nmax - LO - mp.j0;
        if (mp.roots <= 0) return hipSuccess;
    }
    hipLaunchKernelGGL((cs_kernel<LO, HI>), dim3((unsigned)((int64_t)mp.batch * mp.roots)), dim3(kWave), 0, st, g, mp);
    return hipGetLastError();
}

template <int M>
hipError_t launch_one(int m, const CsArgs& g, const CsMap& mp, hipStream_t st)
{
    if constexpr (M < kBlockBits) {
        if (m == M) return launch_range<M, M>(g, mp, M + 1, st);
        return launch_one<M + 1>(m, g, mp, st);
    }
    return hipSuccess;
}

}  // namespace

hipError_t cs_launch(const LaunchCS& L, hipStream_t st)
{
    CsArgs g{L.m_up, L.m_dn, L.c, (L.mode & 2u) ? 1 : 0, L.summ};
    const bool all = (L.mode & 1u) != 0;
    const int nmax = L.n_uniform > 0 ? L.n_uniform : L.n_max;
    const bool mixed = L.n_uniform <= 0;
    CsMap mp{L.batch, L.n_uniform, L.n, L.off, !all && mixed ? L.order : nullptr, 0, 1, !all};
    if (L.walkers && nmax > kBlockBits) {
        auto k = nmax - 1 == kBlockBits ? cs_walk_kernel<true> : cs_walk_kernel<false>;
        hipLaunchKernelGGL(k, dim3((unsigned)L.batch), dim3(kWalkThreads), 0, st, g, nmax);
        return hipGetLastError();
    }
    if (nmax > kBlockBits) {
        const int64_t problems = (int64_t)mp.batch * (all ? nmax - kBlockBits : 1);
        const hipError_t e = g.weights ? launch_blocks<kGiven>(problems, g, mp, st)
                             : g.dn    ? launch_blocks<kProduct>(problems, g, mp, st)
                                       : launch_blocks<kSquare>(problems, g, mp, st);
        if (e != hipSuccess || (!all && !mixed)) return e;
    }
    if (!all && !mixed) return launch_one<0>(nmax - 1, g, mp, st);
    hipError_t e = hipSuccess;
    if (nmax > 10) e = launch_range<10, 10>(g, mp, nmax, st);
    if (e == hipSuccess && nmax > 8) e = launch_range<8, 9>(g, mp, nmax, st);
    if (e == hipSuccess) e = launch_range<0, 7>(g, mp, nmax, st);
    return e;
}

}  // namespace apm
