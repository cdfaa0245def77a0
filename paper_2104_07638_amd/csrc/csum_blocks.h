// csum_blocks.h -- connected sums of 11 bits and more: blocks of 2^11 values staged in LDS, one
// workgroup of five wavefronts per problem.
//
// Block X2 of c' needs every block Y2 subsetneq X2 (a full subset convolution of the c' block Y2
// with the b block X2 \ Y2), then the triangular solve of the block with the b block 0.  A
// block is 128 rows (Xh, 7 bits) of 16 values; a pair (Xh, Yh) is a subset convolution of two
// rows, 81 multiply-adds for 32 values read from LDS.
//
// Row Xh has 2^|Xh| pairs.  It is shared by G = max(1, 2^(|Xh| - 3)) lanes: lane s of them takes
// the pairs whose Yh has the bits of s in the lowest log2(G) bits of Xh, so every lane of a row
// of three bits or more has exactly eight pairs (the subsets of the row's other three bits), and
// the 128 rows take 290 of the 320 lanes: 40 wavefront steps for the 34.2 that 3^7 pairs fill.
// A lane keeps its part of its row in registers through all the blocks Y2 and on into the
// triangular solve, where the pairs with |Yh| = r follow the solve of the rows of rank r: the
// parts are summed once per block, not once per pair of blocks, and no right-hand side is held
// in LDS.  Offsets of rows are additive in the bits of the row number, so stepping through a
// lane's pairs is one addition and one subtraction a pair.
//
// Four workgroups (20 wavefronts) share a CU: 96 registers, 38.7 KB.  Fewer in flight were slower
// (2.76 ms with three for 2.42 of 8192 matrices of 10 to 16 vertices); with all of this the same
// takes 2.1 ms, and 3.25 with four wavefronts a problem, parts summed for every pair of blocks
// and a right-hand side in LDS.  16 vertices, 64 matrices: 765 -> 435 us.  What bounds it: the
// pairs (56% of the cycles issue vector instructions, 49% read LDS), then the loads of blocks
// (0.4 ms of the 2.1) and the eight ranks of the triangular solve (0.5 ms).
#pragma once

constexpr int kBlockBits = 11;
constexpr int kBlockLb = 4, kBlockW = 1 << kBlockLb;         // bits and values of a row
constexpr int kBlockH = kBlockBits - kBlockLb;
constexpr int kBlockRows = 1 << kBlockH;
constexpr int kBlockThreads = 320;
constexpr int kBlockIo = 256;                                // threads that move blocks
constexpr int kBlockIter = (1 << kBlockBits) / kBlockIo;

// Byte offset of a row in LDS: rows of 128 bytes with gaps.  A 16-byte read serves 16 lanes a
// cycle, the 32 lanes of half a wavefront as {0-3, 12-15, 20-27} and the rest (measured), from
// 16 columns of 16 bytes.  The gaps are a sum over the bits of the row, so that offsets stay
// additive, and they and the order of the rows over the lanes (kBlockOrder, free within a rank)
// were searched for the fewest reads of one column by one group: a conv step takes 3.9 cycles a
// read with them and 6.5 with rows 144 bytes apart in order of their numbers.
constexpr int kBlockGap[kBlockH] = {0, 4, 5, 10, 25, 44, 98};
__host__ __device__ constexpr uint32_t block_row(uint32_t row)
{
    uint32_t a = row * (8u * kBlockW);
    for (int i = 0; i < kBlockH; ++i)
        if (row >> i & 1u) a += 16u * (uint32_t)kBlockGap[i];
    return a;
}
constexpr int kBlockLen = (int)(block_row(kBlockRows - 1) / 8u) + kBlockW;
constexpr bool block_gaps_ok()
{
    for (int i = 0, sum = 0; i < kBlockH; sum += kBlockGap[i], ++i)
        if (kBlockGap[i] < sum) return false;     // rows would overlap
    return true;
}
static_assert(block_gaps_ok(), "rows in order");

// The rows by falling rank: the lanes are dealt to them in this order.
struct BlockOrder {
    uint8_t row[kBlockRows];
};
constexpr BlockOrder kBlockOrder = {{
    127, 119, 123, 95, 126, 125, 111, 63, 61, 59, 62, 87, 93, 91, 103, 47, 79, 94, 31, 107,
    110, 55, 121, 109, 124, 122, 117, 118, 115, 116, 71, 46, 86, 89, 58, 53, 54, 102, 99, 57,
    60, 83, 75, 78, 77, 85, 51, 113, 101, 43, 39, 29, 30, 92, 108, 15, 45, 105, 106, 90,
    120, 27, 23, 114, 112, 84, 41, 74, 13, 35, 19, 25, 70, 22, 98, 49, 67, 81, 76, 42,
    38, 14, 82, 88, 97, 52, 104, 7, 50, 73, 37, 69, 21, 26, 56, 28, 44, 100, 11, 40,
    10, 72, 65, 96, 6, 80, 48, 3, 18, 9, 17, 5, 24, 12, 20, 33, 68, 66, 34, 36,
    16, 8, 2, 32, 1, 4, 64, 0}};
__constant__ BlockOrder kBlockOrderDev = kBlockOrder;

// What a lane does: part s of row x.  Byte offsets of rows; |x| = -1: nothing.
struct BlockLane {
    uint32_t x, y;         // the row, and the bits of Yh that s fixes
    uint32_t u[3];         // the row's other bits, lowest first (0: none)
    int rank;              // |x|
    int pairs;             // 8, or 2^|x| in rows of fewer bits
    bool last;             // the lane that holds the sum of the row
};

__device__ __forceinline__ BlockLane block_lane(int tid)
{
    BlockLane q{};
    q.rank = -1;
    int o = 0, s = 0, sh = 0, first = 0, before = 0, rows = 1;
    // the rows of rank 7, 6, ..., 0: C(7, r) 2^max(0, r - 3) lanes each
    for (int k = kBlockH; k >= 0; --k) {
        const int h = k > 3 ? k - 3 : 0, t = tid - first;
        if (t >= 0 && t < rows << h) {
            q.rank = k;
            sh = h;
            o = before + (t >> h);
            s = t & ((1 << h) - 1);
        }
        first += rows << h;
        before += rows;
        rows = rows * k / (kBlockH + 1 - k);
    }
    if (q.rank < 0) return q;
    uint32_t x = kBlockOrderDev.row[o];
    q.x = block_row(x);
    q.last = s == (1 << sh) - 1;
    for (int i = 0; i < sh; ++i) {
        const uint32_t low = x & (0u - x);
        if ((s >> i) & 1) q.y += block_row(low);
        x ^= low;
    }
    q.pairs = 1 << (q.rank < 3 ? q.rank : 3);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const uint32_t low = x & (0u - x);
        q.u[i] = block_row(low);
        x ^= low;
    }
    return q;
}

// acc -= (row y of cb) * (row d of bb)
__device__ __forceinline__ void block_pair(const double* cb, uint32_t y, const double* bb, uint32_t d, double (&acc)[kBlockW])
{
    constexpr int HW = kBlockW / 2;
    double f[HW], g0[HW], g1[HW];
    ld_row_at<HW>(cb, y, f);
    ld_row_at<HW>(bb, d, g0);
    ld_row_at<HW>(bb, d + 8 * HW, g1);
    conv_half<kBlockLb - 1>(f, g0, acc);
    conv_half<kBlockLb - 1>(f, g1, acc + HW);
    ld_row_at<HW>(cb, y + 8 * HW, f);
    conv_half<kBlockLb - 1>(f, g0, acc + HW);
}

__device__ __forceinline__ void block_conv(const BlockLane& q, const double* cb, const double* bb, double (&acc)[kBlockW])
{
    // (opaque: sixteen offsets formed ahead and kept through the loop over blocks would spill)
    uint32_t y0 = q.y, x = q.x;
    asm volatile("" : "+v"(y0), "+v"(x));
#pragma unroll 1
    for (int h = 0; h < 8; h += 4, y0 += q.u[2]) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t y = y0 + (k & 1 ? q.u[0] : 0u) + (k & 2 ? q.u[1] : 0u);
            if (h + k < q.pairs) block_pair(cb, y, bb, x - y, acc);
        }
    }
}

// Pairs of the triangular solve: after the rows of rank r are solved, wavefront w takes
// steps(w, r) of its list, one pair a lane and step.  The lists are earliest-deadline-first: a
// row's pairs in order of |Yh|, as many in a step as the row has lanes, a pair of |Yh| = r no
// earlier than after rank r and all of them before the row's own rank.  The counts below are the
// fewest steps on the critical path (14 over the ranks, 12 being what the rows next to be solved
// need), then the fewest in total (44); taking every pair as soon as its row is solved needs 19
// and 65.
struct BlockTri {
    static constexpr int kSlots = 10;
    static constexpr int kNone = 0xFFFF;
    static constexpr uint32_t kSteps[kBlockThreads / kWave] = {0x1132200, 0x0132300, 0x0022420, 0x0002421, 0x0000421};
    static constexpr int steps(int w, int r) { return (int)(kSteps[w] >> (4 * r) & 15u); }
    uint32_t entry[kSlots / 2][kBlockThreads];       // two byte offsets of rows Yh each, in order
    bool complete;
    static constexpr int bits(int x)
    {
        int c = 0;
        for (; x; x &= x - 1) ++c;
        return c;
    }
    static constexpr BlockTri make()
    {
        BlockTri t{};
        t.complete = true;
        for (auto& e : t.entry)
            for (auto& v : e) v = 0xFFFFFFFFu;
        int first = 0;
        for (int o = 0; o < kBlockRows; ++o) {
            const int x = kBlockOrder.row[o], r = bits(x), g = r > 3 ? 1 << (r - 3) : 1;
            const int w = first / kWave;
            int slot = 0, level = 0, y = 0, left = (1 << r) - 1;   // next pair: the first y of this level
            for (int st = 0; st < r; ++st) {
                for (int k = 0; k < steps(w, st); ++k, ++slot) {
                    for (int l = 0; l < g && level <= st;) {
                        if (y == kBlockRows) {
                            ++level;
                            y = 0;
                        } else {
                            if ((y & ~x) == 0 && bits(y) == level) {
                                const int sh = 16 * (slot & 1);
                                uint32_t& e = t.entry[slot / 2][first + l];
                                e = (e & ~(0xFFFFu << sh)) | block_row((uint32_t)y) << sh;
                                ++l;
                                --left;
                            }
                            ++y;
                        }
                    }
                }
            }
            if (left != 0) t.complete = false;
            first += g;
        }
        return t;
    }
};

__constant__ BlockTri kBlockTri = BlockTri::make();
static_assert(BlockTri::make().complete, "every pair has its step");

struct BlockList {
    uint32_t e[BlockTri::kSlots / 2];
};

__device__ __forceinline__ void block_stage(const BlockLane& q, int n, BlockList& list, const double* cb, const double* bb,
                                            double (&acc)[kBlockW])
{
#pragma unroll 1
    for (; n > 0; --n) {
        const uint32_t y = list.e[0] & 0xFFFFu;
#pragma unroll
        for (int i = 0; i < BlockTri::kSlots / 2; ++i)
            list.e[i] = __builtin_amdgcn_alignbit(i + 1 < BlockTri::kSlots / 2 ? list.e[i + 1] : 0u, list.e[i], 16);
        if (y != BlockTri::kNone) block_pair(cb, y, bb, q.x - y, acc);
    }
}

// Rows of rank r: sum of the parts, then c'[X] within the row, into the c' block.
__device__ __forceinline__ void block_solve(const BlockLane& q, int r, double* cb, const double* bb, double (&acc)[kBlockW])
{
    if (q.rank != r) return;
    if (r > 3) group_sum<kBlockW>(acc, 1 << (r - 3));
    if (q.last) {
        double g0[kBlockW];
        ld_row_at<kBlockW>(bb, 0, g0);
        tri_tile<kBlockLb>(acc, g0);
#pragma unroll
        for (int p = 0; p < kBlockW / 2; ++p)
            *reinterpret_cast<double2*>(reinterpret_cast<char*>(cb) + q.x + 16 * p) = make_double2(acc[2 * p], acc[2 * p + 1]);
    }
}

// Block moves: thread t of the first 256 has the values x1 = t + 256 i, whose rows are those of t
// plus multiples of 16 (constant offsets).  The thread number is opaque here, so that addresses
// are formed where they are used and not kept in registers through the whole problem.
__device__ __forceinline__ uint32_t block_thread()
{
    uint32_t t = threadIdx.x & (kBlockIo - 1);
    asm volatile("" : "+v"(t));
    return t;
}

// v[i] = src[x1 << sh]: one 32-bit offset a thread, scalar steps
__device__ __forceinline__ double block_load(const double* src, int sh, uint32_t off, int i)
{
    return *reinterpret_cast<const double*>(reinterpret_cast<const char*>(src + ((int64_t)(i * kBlockIo) << sh)) + off);
}

__device__ __forceinline__ void block_get(const double* src, int sh, double (&v)[kBlockIter])
{
    const uint32_t off = block_thread() << (sh + 3);
#pragma unroll
    for (int i = 0; i < kBlockIter; ++i) v[i] = block_load(src, sh, off, i);
}

// The same of the weights a[s0 + (x1 << sh)]: given, squares of up or products of up and dn (a
// template argument: with branches around the loads the values would spill).
enum BlockWeights { kGiven, kSquare, kProduct };

template <BlockWeights K>
__device__ __forceinline__ void block_weights(const CsArgs& g, int64_t s0, int sh, double (&v)[kBlockIter])
{
    block_get(g.up + s0, sh, v);
    if constexpr (K == kSquare) {
#pragma unroll
        for (int i = 0; i < kBlockIter; ++i) v[i] *= v[i];
    } else if constexpr (K == kProduct) {
        const uint32_t off = block_thread() << (sh + 3);
        constexpr int HI = kBlockIter / 4;
#pragma unroll
        for (int h = 0; h < kBlockIter; h += HI) {
            double d[HI];
#pragma unroll
            for (int i = 0; i < HI; ++i) d[i] = block_load(g.dn + s0, sh, off, h + i);
#pragma unroll
            for (int i = 0; i < HI; ++i) v[h + i] *= d[i];
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// Address in LDS of the thread's value i.
__device__ __forceinline__ uint32_t block_at(uint32_t t) { return block_row((t >> kBlockLb) & 15u) + (t & 15u) * 8u; }
__device__ __forceinline__ double& block_value(double* buf, uint32_t at, int i)
{
    return *reinterpret_cast<double*>(reinterpret_cast<char*>(buf) + at + block_row((uint32_t)i * (kBlockIo / kBlockW)));
}

__device__ __forceinline__ void block_put(double* buf, const double (&v)[kBlockIter])
{
    const uint32_t at = block_at(block_thread());
#pragma unroll
    for (int i = 0; i < kBlockIter; ++i) block_value(buf, at, i) = v[i];
}

// Problem (matrix at base, root j) of m >= 11 bits.
template <BlockWeights K>
__device__ __forceinline__ void block_problem(const CsArgs& g, int64_t base, int j, int m, bool zero_even, double* lds_c,
                                              double* lds_b)
{
    const int tid = (int)threadIdx.x;
    const BlockLane q = block_lane(tid);
    const int sh = j + 1;                            // X -> S = (1 << j) | (X << (j + 1))
    const int64_t sroot = base + (int64_t(1) << j);  // element index of S = {j}
    double* c = g.c;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    uint32_t wave_steps = BlockTri::kSteps[0];
#pragma unroll
    for (int w = 1; w < kBlockThreads / kWave; ++w)
        if (wave == w) wave_steps = BlockTri::kSteps[w];
#pragma unroll 1
    for (uint32_t x2 = 0; x2 < (1u << (m - kBlockBits)); ++x2) {
        double acc[kBlockW];
#pragma unroll
        for (int i = 0; i < kBlockW; ++i) acc[i] = 0.0;
        // the blocks below
        for (uint32_t y2 = 0; y2 != x2; y2 = (y2 - x2) & x2) {
            const uint32_t d2 = x2 ^ y2;
            double v[kBlockIter], w[kBlockIter];
            const int64_t cy = sroot + ((int64_t)y2 << (kBlockBits + sh));
            block_get(c + cy, sh, w);
            block_weights<K>(g, base + ((int64_t)d2 << (kBlockBits + sh)), sh, v);
            __syncthreads();
            block_put(lds_c, w);
            block_put(lds_b, v);
            __syncthreads();
            block_conv(q, lds_c, lds_b, acc);
        }
        // the block's own solve: the right-hand side a0 goes through the c' block, of which row
        // x is read only by the lane that later writes c'[X] there, until it is written
        double v[kBlockIter], w[kBlockIter];
        block_weights<K>(g, base, sh, v);
        block_weights<K>(g, sroot + ((int64_t)x2 << (kBlockBits + sh)), sh, w);
        BlockList list;
#pragma unroll
        for (int i = 0; i < BlockTri::kSlots / 2; ++i) list.e[i] = kBlockTri.entry[i][tid];
        uint32_t steps = wave_steps;
        __syncthreads();
        if ((tid & (kBlockIo - 1)) == 0) v[0] = 0.0;
        block_put(lds_b, v);
        block_put(lds_c, w);
        __syncthreads();
        if (q.rank >= 0 && q.last) {
            double a0[kBlockW];
            ld_row_at<kBlockW>(lds_c, q.x, a0);
#pragma unroll
            for (int i = 0; i < kBlockW; ++i) acc[i] += a0[i];
        }
#pragma unroll 1
        for (int r = 0; r <= kBlockH; ++r) {
            block_solve(q, r, lds_c, lds_b, acc);
            __syncthreads();
            block_stage(q, (int)(steps & 15u), list, lds_c, lds_b, acc);
            steps >>= 4;
        }
        const uint32_t t = block_thread(), at = block_at(t);
        if (tid < kBlockIo) {
            const int64_t x = ((int64_t)x2 << kBlockBits) + t;
            if (zero_even && !(base & 1)) {
                // rooted problem: write (c[2x] = 0, c[2x+1] = c'[x]) as one 16-byte store
#pragma unroll
                for (int i = 0; i < kBlockIter; ++i)
                    *reinterpret_cast<double2*>(c + base + 2 * (x + i * kBlockIo)) = make_double2(0.0, block_value(lds_c, at, i));
            } else {
#pragma unroll
                for (int i = 0; i < kBlockIter; ++i) {
                    c[sroot + ((x + i * kBlockIo) << sh)] = block_value(lds_c, at, i);
                    if (zero_even) c[base + 2 * (x + i * kBlockIo)] = 0.0;
                }
            }
        }
        __syncthreads();     // the next block reads these values of c
    }
    if (j == 0 && tid == 0) c[base] = 0.0;   // c[empty] = 0
}
