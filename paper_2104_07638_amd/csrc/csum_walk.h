// csum_walk.h -- connected sums of Monte Carlo walkers of 12 vertices and more.
//
// c[V] of a walker is what remains of sums that nearly cancel: another order of the same sums
// moves log|c[V]| by up to 1e-7 at 12 and 13 vertices, and with it the recorded weights of a
// walk.  Here the order of every sum is fixed, apart from that of csum_blocks.h (which is the
// faster one, 62 us for 70 at 2000 problems of 11 bits): blocks of 2^11 values on four
// wavefronts, the pairs of a row dealt round robin to G lanes and summed once per pair of
// blocks.  Rows of 16 values are 144 bytes apart.
#pragma once

constexpr int kWalkThreads = 4 * kWave;
constexpr uint32_t kWalkRow = 144;
constexpr int kWalkLen = kBlockRows * (int)kWalkRow / 8;

// Rows by rank: row[] lists the masks of popcount 0, 1, ..., off[r] is where rank r starts.
struct WalkRanks {
    uint8_t row[kBlockRows];
    int off[kBlockH + 2];
};
constexpr WalkRanks walk_ranks()
{
    WalkRanks t{};
    int pos = 0;
    for (int r = 0; r <= kBlockH; ++r) {
        t.off[r] = pos;
        for (int x = 0; x < kBlockRows; ++x)
            if (BlockTri::bits(x) == r) t.row[pos++] = (uint8_t)x;
    }
    t.off[kBlockH + 1] = pos;
    return t;
}
__constant__ WalkRanks kWalkRanks = walk_ranks();

// Lane s of the G lanes of row xh takes the pairs s, s + G, ... of the row (Yh subsetneq Xh for
// TRI, Yh subset of Xh otherwise); the last lane adds the sum to the right-hand side in rb (TRI:
// then solves the row and writes it to cb_out).  Every lane of the wavefront has the same G.
template <bool TRI>
__device__ __forceinline__ void walk_row(bool valid, uint32_t xh, int items, int G, int s, const double* cb,
                                         const double* bb, double* rb, double* cb_out)
{
    double acc[kBlockW];
#pragma unroll
    for (int i = 0; i < kBlockW; ++i) acc[i] = 0.0;
    if (valid) {
        // pair k = s + G t has Yh = pdep(s) | pdep(t) over the bits of Xh above its lowest
        // log2(G) ones: the second part steps through the subsets of those bits in order
        uint32_t ys = 0, xhi = xh, z = 0;
        for (int gg = 1; gg < G; gg <<= 1) {
            const uint32_t low = xhi & (0u - xhi);
            if (s & gg) ys |= low;
            xhi ^= low;
        }
#pragma unroll 1
        for (int k = s; k < items; k += G, z = (z - xhi) & xhi) {
            const uint32_t y = ys | z;
            block_pair(cb, y * kWalkRow, bb, (xh ^ y) * kWalkRow, acc);
        }
    }
    group_sum<kBlockW>(acc, G);
    if (valid && s == G - 1) {
        double rr[kBlockW];
        ld_row_at<kBlockW>(rb, xh * kWalkRow, rr);
#pragma unroll
        for (int i = 0; i < kBlockW; ++i) rr[i] += acc[i];
        if constexpr (TRI) {
            double g0[kBlockW];
            ld_row_at<kBlockW>(bb, 0, g0);
            tri_tile<kBlockLb>(rr, g0);
        }
        char* out = reinterpret_cast<char*>(TRI ? cb_out : rb) + xh * kWalkRow;
#pragma unroll
        for (int p = 0; p < kBlockW / 2; ++p)
            *reinterpret_cast<double2*>(out + 16 * p) = make_double2(rr[2 * p], rr[2 * p + 1]);
    }
}

// k1 rows of rank r1 and k2 rows of rank r2, G lanes a row, on one wavefront.
__device__ __forceinline__ void walk_task(int lane, int G, int r1, int k1, int r2, int k2, const uint8_t* row, const double* cb,
                                          const double* bb, double* rb)
{
    const int q = lane / G;
    const bool in1 = q < k1, valid = q < k1 + k2;
    const int r = in1 ? r1 : r2;
    const uint32_t xh = valid ? row[kWalkRanks.off[r] + (in1 ? q : q - k1)] : 0u;
    walk_row<false>(valid, xh, 1 << r, G, lane % G, cb, bb, rb, nullptr);
}

// Index in LDS of value x1 of a block.
__device__ __forceinline__ int walk_at(int x1) { return (x1 >> kBlockLb) * (int)(kWalkRow / 8) + (x1 & (kBlockW - 1)); }

// Walker b: c[] (or its summary) of m = n - 1 >= 11 bits rooted at vertex 0, with the squares of
// up[] as weights.  ONE: m = 11, solved in place of the right-hand side.
template <bool ONE>
__global__ __launch_bounds__(kWalkThreads) __attribute__((amdgpu_waves_per_eu(ONE ? 4 : 2))) void cs_walk_kernel(CsArgs g, int n)
{
    __shared__ __align__(16) double lds_c[kWalkLen];
    __shared__ __align__(16) double lds_b[kWalkLen];
    __shared__ __align__(16) double lds_r[ONE ? 2 : kWalkLen];
    __shared__ uint8_t rk[kBlockRows];
    constexpr int N = 1 << kBlockBits, full = N - 1;
    const int tid = (int)threadIdx.x, lane = tid % kWave, wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const double* up = g.up + ((int64_t)blockIdx.x << n);
    double* c = g.c + ((int64_t)blockIdx.x << n);
    double* rhs = ONE ? lds_c : lds_r;
    if (tid < kBlockRows) rk[tid] = kWalkRanks.row[tid];
    const uint32_t blocks = ONE ? 1u : 1u << (n - 1 - kBlockBits);
    for (uint32_t x2 = 0; x2 < blocks; ++x2) {
        // (one block: b and the right-hand side are neighbours)
#pragma unroll 4
        for (int x1 = tid; x1 < N; x1 += kWalkThreads) {
            const double2 u = *reinterpret_cast<const double2*>(up + 2 * (((int64_t)x2 << kBlockBits) | x1));
            rhs[walk_at(x1)] = u.y * u.y;
            if (ONE) lds_b[walk_at(x1)] = x1 ? u.x * u.x : 0.0;
        }
        for (uint32_t y2 = 0; !ONE && y2 != x2; y2 = (y2 - x2) & x2) {
            __syncthreads();
#pragma unroll 4
            for (int x1 = tid; x1 < N; x1 += kWalkThreads) {
                const double u = up[2 * (((int64_t)(x2 ^ y2) << kBlockBits) | x1)];
                lds_c[walk_at(x1)] = c[2 * (((int64_t)y2 << kBlockBits) | x1) + 1];
                lds_b[walk_at(x1)] = u * u;
            }
            __syncthreads();
            // the rows are independent: a fixed share of the ranks for each wavefront
            if (wave == 0) {
                walk_task(lane, 2, 5, 21, 0, 0, rk, lds_c, lds_b, rhs);
            } else if (wave == 1) {
                walk_task(lane, 1, 4, 35, 0, 0, rk, lds_c, lds_b, rhs);
            } else if (wave == 2) {
                walk_task(lane, 8, 6, 7, 0, 0, rk, lds_c, lds_b, rhs);
                walk_task(lane, 1, 2, 21, 0, 1, rk, lds_c, lds_b, rhs);
            } else {
                walk_task(lane, 1, 3, 35, 1, 7, rk, lds_c, lds_b, rhs);
                walk_task(lane, 64, 7, 1, 0, 0, rk, lds_c, lds_b, rhs);
            }
        }
        __syncthreads();
        if (!ONE) {
#pragma unroll 4
            for (int x1 = tid; x1 < N; x1 += kWalkThreads) {
                const double u = up[2 * (int64_t)x1];
                lds_b[walk_at(x1)] = x1 ? u * u : 0.0;
            }
            __syncthreads();
        }
        const double a_full = g.summ ? rhs[walk_at(full)] : 0.0;
#pragma unroll 1
        for (int r = 0; r <= kBlockH; ++r) {
            const int first = kWalkRanks.off[r], rows = kWalkRanks.off[r + 1] - first, items = (1 << r) - 1;
            int lg = 0;   // G = 2^lg lanes a row
            while (lg < 6 && rows << lg <= kWalkThreads / 2 && 2 << lg <= (items > 0 ? items : 1)) ++lg;
#pragma unroll 1
            for (int ob = 0; ob < rows; ob += kWalkThreads >> lg) {
                const int o = ob + (tid >> lg);
                const bool valid = o < rows;
                walk_row<true>(valid, valid ? rk[first + o] : 0u, items, 1 << lg, tid & ((1 << lg) - 1), lds_c,
                               lds_b, rhs, lds_c);
            }
            __syncthreads();
        }
        if (ONE && g.summ) {
            double part = 0.0;
#pragma unroll 4
            for (int x1 = tid; x1 < full; x1 += kWalkThreads) part += fabs(lds_c[walk_at(x1)]) * fabs(lds_b[walk_at(full ^ x1)]);
            for (int o = kWave / 2; o > 0; o >>= 1) part += __shfl_xor(part, o);
            __syncthreads();
            if (lane == 0) lds_b[wave] = part;   // b block no longer needed
            __syncthreads();
            if (tid == 0) {
                part = 0.0;
                for (int w = 0; w < kWalkThreads / kWave; ++w) part += lds_b[w];
                g.summ[2 * (int64_t)blockIdx.x] = lds_c[walk_at(full)];
                g.summ[2 * (int64_t)blockIdx.x + 1] = fabs(a_full) + part;
            }
            return;
        }
#pragma unroll 4
        for (int x1 = tid; x1 < N; x1 += kWalkThreads)
            *reinterpret_cast<double2*>(c + 2 * (((int64_t)x2 << kBlockBits) | x1)) = make_double2(0.0, lds_c[walk_at(x1)]);
    }
}
