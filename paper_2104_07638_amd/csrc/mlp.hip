// mlp.hip -- the proposal network on the gfx950 matrix cores: BF16 operands, fp32 sums.
//
// Network: h1 = tanh(W1 x + b1), h2 = tanh(W2 h1 + b2), out = W3 h2 + b3, hidden width
// 128.  Every product is computed transposed, Z^T = W H^T, with v_mfma_f32_16x16x16_bf16:
//   A operand (16 x 16, M x K): lane l holds A[l % 16][4 (l / 16) + 0..3]
//   B operand (16 x 16, K x N): lane l holds B[4 (l / 16) + 0..3][l % 16]
//   D result  (16 x 16, M x N): lane l holds D[4 (l / 16) + 0..3][l % 16]
// With the weights as A and the activations (features x batch) as B, the D tile of 16
// output features is exactly the B operand of the next layer's k-step over those
// features.  The forward pass runs one workgroup per 32 batch rows (two N tiles sharing
// every weight load); its wavefronts split each layer's output features and pass the
// activations on through LDS.
//
// The forward pass reads its BF16 weights (net.w) in that A-operand order: for a layer of
// M x K weights, tile (mt, ks) (rows 16 mt.., columns 16 ks..) is 64 lanes x 4 values stored
// contiguously from ((mt (K / 16) + ks) 64 + lane) 4, so that one load instruction of a
// wavefront reads 512 consecutive bytes (from row-major rows it would touch 16 cache lines).
//
// Backward: the hidden gradients are chained the same way through the transposed
// weights (W^T kept as a second BF16 copy); the weight gradients dW = dZ^T H sum over
// the batch as the K dimension, from BF16 copies of dZ and H in the operand order of
// those products (store_t).  The Monte Carlo training step passes its output gradient in picked form
// (two entries a row, MlpPick), computed in the backward kernel itself.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <type_traits>

#include "apm_kernels.h"

namespace apm {
namespace {

constexpr int H = 128;

typedef short v4s __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint16_t f2bf(float f)
{
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);   // round to nearest, ties to even
    return (uint16_t)(u >> 16);
}

__device__ __forceinline__ v4s pack_bf(v4f v)
{
    v4s r;
    r[0] = (short)f2bf(v[0]);
    r[1] = (short)f2bf(v[1]);
    r[2] = (short)f2bf(v[2]);
    r[3] = (short)f2bf(v[3]);
    return r;
}

__device__ __forceinline__ float bf2f(short b) { return __uint_as_float(((uint32_t)(uint16_t)b) << 16); }

__device__ __forceinline__ float tanh_f(float z)
{
    const float e = __expf(2.0f * z);   // inf for large z gives 1, 0 for very negative z gives -1
    return 1.0f - 2.0f / (e + 1.0f);
}

__device__ __forceinline__ v4f mfma(v4s a, v4s b, v4f c)
{
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ v4s ld4(const uint16_t* p) { return *reinterpret_cast<const v4s*>(p); }

// Batch-contiguous copies (of activations and gradients, for the weight gradients) are kept in
// the operand order of products over the batch: 16 features x 32 rows are 64 lanes x 8 values,
// lane 16 (row % 16 / 4) + feature holding rows 4 (lane / 16) .. + 3 of the first 16 rows and
// then of the second, one such block after the other.  A load of both operands of a step is then
// 1024 consecutive bytes; in
// plain feature-major rows (2 B bytes apart, a power of two at the usual batches) the 16 lines
// of a load fell on one L2 channel.
//
// Store tile (ft, rt) from the layout of a D tile (lane 16 g + r: features 4 g .. 4 g + 3 of row
// r): transpose 4 x 4 values within each four lanes, then one 8-byte store.
__device__ __forceinline__ void store_t(uint16_t* dst, int B, int ft, int rt, v4s v)
{
    const int lane = threadIdx.x & 63, q = lane & 3;
    const uint2 p = __builtin_bit_cast(uint2, v);      // features (0, 1) and (2, 3)
    const bool hi = q & 2, odd = q & 1;
    // lanes q and q ^ 2 exchange a word: own features (q & 2) + {0, 1} of rows q and q ^ 2
    const uint32_t mine = hi ? p.y : p.x;
    const uint32_t far = (uint32_t)__builtin_amdgcn_mov_dpp((int)(hi ? p.x : p.y), 0x4E, 0xF, 0xF, true);
    // lanes q and q ^ 1 exchange both: own feature q of rows (q, q ^ 1) and (q ^ 2, q ^ 3)
    const uint32_t mine1 = (uint32_t)__builtin_amdgcn_mov_dpp((int)mine, 0xB1, 0xF, 0xF, true);
    const uint32_t far1 = (uint32_t)__builtin_amdgcn_mov_dpp((int)far, 0xB1, 0xF, 0xF, true);
    // the halves of the even and the odd row of each pair: low ones in even lanes, high in odd
    const uint32_t sel = odd ? 0x07060302u : 0x05040100u;
    const uint32_t a = __builtin_amdgcn_perm(odd ? mine : mine1, odd ? mine1 : mine, sel);
    const uint32_t b = __builtin_amdgcn_perm(odd ? far : far1, odd ? far1 : far, sel);
    const uint2 o = hi ? make_uint2(b, a) : make_uint2(a, b);
    // feature 4 g + q, rows 4 (r / 4) .. + 3
    const int at = ((lane & 15) >> 2) * 16 + 4 * (lane >> 4) + q;
    *reinterpret_cast<uint2*>(dst + ((size_t)ft * (B / 32) + (rt >> 1)) * 512 + at * 8 + 4 * (rt & 1)) = o;
}

// Forward pass: one workgroup of kFwdWaves wavefronts per 32 batch rows.  The wavefronts
// split the output features of every layer (wave v computes hidden tiles kMtPerWave v.. and
// output tiles v, v + kFwdWaves, ...) and exchange the BF16 activations through LDS between
// layers, already in B-operand order.  Each wavefront needs only its slice of the weights and
// loads all of it up front (straight from L2, one batch of independent loads), so the three
// layers wait for memory once.  The kernel is latency-bound (one workgroup per CU at the
// Monte Carlo batch); eight wavefronts measured faster than four (fewer output tiles each).
#ifndef APM_MLP_FWD_WAVES
#define APM_MLP_FWD_WAVES 8
#endif
#ifndef APM_MLP_W3PRE
#define APM_MLP_W3PRE 3
#endif
constexpr int kFwdWaves = APM_MLP_FWD_WAVES;   // 2, 4 or 8
constexpr int kMtPerWave = 8 / kFwdWaves;
constexpr int kW3Pre = APM_MLP_W3PRE;    // output tiles per wavefront whose weights are loaded up front
static_assert(kFwdWaves == 2 || kFwdWaves == 4 || kFwdWaves == 8, "hidden tiles split evenly over the wavefronts");

// This lane's A operands of row tile mt (k-steps 0..KS-1) of a layer, from the
// fragment-ordered weights: one address per tile, the k-steps at constant offsets of 512 B.
template <int KS>
__device__ __forceinline__ void load_tile(const uint16_t* __restrict__ W, int mt, v4s (&a)[KS])
{
    const uint16_t* p = W + (size_t)(uint32_t)mt * (KS * 256) + (threadIdx.x & 63) * 4;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) a[ks] = ld4(p + ks * 256);
}

template <int KS>
__device__ __forceinline__ void load_slice(const uint16_t* __restrict__ W, int mt0, v4s (&a)[kMtPerWave][KS])
{
#pragma unroll
    for (int m = 0; m < kMtPerWave; ++m) load_tile<KS>(W, mt0 + m, a[m]);
}

// the biases of this lane's features 16 (mt0 + m) + 4 (lane / 16) + 0..3 of the hidden tiles
// mt0 .. mt0+kMtPerWave-1
__device__ __forceinline__ void load_bias(const float* __restrict__ b, int mt0, v4f (&bb)[kMtPerWave])
{
    const int g = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int m = 0; m < kMtPerWave; ++m) bb[m] = *reinterpret_cast<const v4f*>(b + 16 * (mt0 + m) + 4 * g);
}

// tanh(W in + b) for the hidden tiles mt0 .. mt0+kMtPerWave-1 of both row tiles (bb: their
// biases, from load_bias)
template <int KS>
__device__ __forceinline__ void hidden_slice(const v4s (&a)[kMtPerWave][KS], const v4f (&bb)[kMtPerWave],
                                             const v4s (&in)[2][KS], int mt0, v4s* act_out, int row0, int B,
                                             float* save, uint16_t* save_t)
{
    const int lane = threadIdx.x & 63, r16 = lane & 15, g = lane >> 4;
#pragma unroll
    for (int m = 0; m < kMtPerWave; ++m) {
        const int mt = mt0 + m;
        v4f a0 = {0.f, 0.f, 0.f, 0.f}, a1 = a0;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            a0 = mfma(a[m][ks], in[0][ks], a0);
            a1 = mfma(a[m][ks], in[1][ks], a1);
        }
        const int f0 = 16 * mt + 4 * g;
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            const v4f z = (nt == 0 ? a0 : a1) + bb[m];
            v4f h;
            h[0] = tanh_f(z[0]);
            h[1] = tanh_f(z[1]);
            h[2] = tanh_f(z[2]);
            h[3] = tanh_f(z[3]);
            const v4s hb = pack_bf(h);
            act_out[(mt * 2 + nt) * 64 + lane] = hb;
            const int r = row0 + 16 * nt + r16;
            if (save) *reinterpret_cast<v4f*>(save + (size_t)r * H + f0) = h;
            if (save_t) store_t(save_t, B, mt, row0 / 16 + nt, hb);
        }
    }
}

template <int KS1>
__global__ __launch_bounds__(64 * kFwdWaves) void mlp_fwd_kernel(const uint16_t* __restrict__ w,
                                                                 const float* __restrict__ bias,
                                                                 const uint16_t* __restrict__ x, int B, int Op,
                                                                 float* __restrict__ out, float* h1s, float* h2s,
                                                                 uint16_t* actT)
{
    constexpr int DP = 16 * KS1;
    __shared__ v4s act1[8 * 2 * 64], act2[8 * 2 * 64];   // [feature tile][row tile][lane]
    const int lane = threadIdx.x & 63, r16 = lane & 15, g = lane >> 4, wv = threadIdx.x >> 6;
    const int row0 = blockIdx.x * 32;
    const uint16_t* W1 = w;
    const uint16_t* W2 = W1 + H * DP;
    const uint16_t* W3 = W2 + H * H;

    const int ntile = Op / 16;
    const float* b3 = bias + 2 * H;
    // every input, weight and bias this wavefront uses (a slice of each layer) is requested up
    // front, in the order the layers need them, so that each layer waits only for its own
    // operands and the three layers wait for memory about once
    v4s xo[2][KS1];
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
        for (int ks = 0; ks < KS1; ++ks) xo[nt][ks] = ld4(x + (size_t)(row0 + 16 * nt + r16) * DP + 16 * ks + 4 * g);
    v4s w1[kMtPerWave][KS1], w2[kMtPerWave][8], w3[kW3Pre][8];
    v4f bb1[kMtPerWave], bb2[kMtPerWave], bb3[kW3Pre];
    load_slice<KS1>(W1, kMtPerWave * wv, w1);
    load_bias(bias, kMtPerWave * wv, bb1);
    __builtin_amdgcn_sched_barrier(0);   // keep this issue order (the scheduler groups loads by size)
    load_slice<8>(W2, kMtPerWave * wv, w2);
    load_bias(bias + H, kMtPerWave * wv, bb2);
    __builtin_amdgcn_sched_barrier(0);
    // (tiles past the last one load the last tile again, unused: unconditional loads keep the
    // compiler's count of loads in flight exact, so no wait covers more than it needs)
#pragma unroll
    for (int u = 0; u < kW3Pre; ++u) {
        const int t = min(wv + u * kFwdWaves, ntile - 1);
        load_tile<8>(W3, t, w3[u]);
        bb3[u] = *reinterpret_cast<const v4f*>(b3 + 16 * t + 4 * g);
    }
    if (actT && wv == 0) {   // training: batch-contiguous copy of the input
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
            for (int ks = 0; ks < KS1; ++ks) store_t(actT, B, ks, row0 / 16 + nt, xo[nt][ks]);
    }
    hidden_slice<KS1>(w1, bb1, xo, kMtPerWave * wv, act1, row0, B, h1s, actT ? actT + (size_t)DP * B : nullptr);
    __syncthreads();

    v4s h1o[2][8];
#pragma unroll
    for (int kt = 0; kt < 8; ++kt)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) h1o[nt][kt] = act1[(kt * 2 + nt) * 64 + lane];
    hidden_slice<8>(w2, bb2, h1o, kMtPerWave * wv, act2, row0, B, h2s, actT ? actT + (size_t)(DP + H) * B : nullptr);
    __syncthreads();

    v4s h2o[2][8];
#pragma unroll
    for (int kt = 0; kt < 8; ++kt)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) h2o[nt][kt] = act2[(kt * 2 + nt) * 64 + lane];
    auto out_tile = [&](int t, const v4s (&a)[8], v4f bb) {
        v4f a0 = {0.f, 0.f, 0.f, 0.f}, a1 = a0;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
            a0 = mfma(a[ks], h2o[0][ks], a0);
            a1 = mfma(a[ks], h2o[1][ks], a1);
        }
        const int f0 = 16 * t + 4 * g;
        *reinterpret_cast<v4f*>(out + (size_t)(row0 + r16) * Op + f0) = a0 + bb;
        *reinterpret_cast<v4f*>(out + (size_t)(row0 + 16 + r16) * Op + f0) = a1 + bb;
    };
#pragma unroll
    for (int u = 0; u < kW3Pre; ++u) {
        const int t = wv + u * kFwdWaves;
        if (t < ntile) out_tile(t, w3[u], bb3[u]);
    }
    // tiles beyond the preloaded ones (wide output layers)
    for (int t = wv + kW3Pre * kFwdWaves; t < ntile; t += kFwdWaves) {
        v4s a[8];
        load_tile<8>(W3, t, a);
        out_tile(t, a, *reinterpret_cast<const v4f*>(b3 + 16 * t + 4 * g));
    }
}

// The gradient of the Monte Carlo regression at the outputs of row r: two entries, the proposed
// site's logit and the proposed bin's, hold the same value g[r]; all others are zero.
//   pred = site logit + bin logit, y = log|c'| clipped below at (batch maximum - clip),
//   g = 2 (pred - y) / B; the loss is the mean of (pred - y)^2.
// One thread per row of the workgroup's 32; the maximum from the acceptance kernel's partial
// ones.  Writes the rows' entries for the weight gradients and the workgroup's share of the
// loss, and leaves them in LDS for the hidden gradients.
struct Picked {
    uint32_t sel[32];    // entries: low and high half
    float g[32];         // rounded to BF16
};

__device__ __forceinline__ void pick_rows(const MlpPick& pk, int Op, int B, int row0, Picked& lds)
{
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        double mx = -INFINITY;
        for (int i = lane; i < pk.nmax; i += 64) mx = fmax(mx, pk.maxp[i]);
        for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o));
        double sq = 0.0;
        if (lane < 32) {
            const int r = row0 + lane;
            const uint32_t v = pk.prop[r];
            const int f1 = (int)(v & 0xFFFFu), f2 = pk.L2 + (int)(v >> 16) / pk.per_bin;
            float g = 0.0f;
            if (mx > -INFINITY) {
                const double floor_y = mx - pk.clip;
                double y = pk.logc[r];
                y = isfinite(y) ? fmax(y, floor_y) : floor_y;
                const double pred = (double)pk.logits[(size_t)r * Op + f1] + (double)pk.logits[(size_t)r * Op + f2];
                const double diff = pred - y;
                g = (float)(2.0 * diff / B);
                sq = diff * diff;
            }
            const uint32_t sel = (uint32_t)f1 | ((uint32_t)f2 << 16);
            const uint16_t gb = f2bf(g);
            lds.sel[lane] = sel;
            lds.g[lane] = bf2f((short)gb);
            pk.sel[r] = sel;
            pk.g[r] = gb;
        }
        for (int o = 16; o > 0; o >>= 1) sq += __shfl_xor(sq, o);
        if (lane == 0) pk.lpart[blockIdx.x] = sq;
    }
    __syncthreads();
}

// dz2 = (W3^T dout^T) * (1 - h2^2), dz1 = (W2^T dz2^T) * (1 - h1^2); batch-contiguous
// BF16 copies (store_t) of dout, dz2 and dz1 go to gT = [Op | H | H][B].  One workgroup of four wavefronts per 32
// rows; wavefront v computes the hidden tiles 2 v and 2 v + 1 of both gradients, dz2 passed on
// through LDS in B-operand order.  Picks: the output gradient has two entries a row
// (pick_rows), so W3^T dout^T is two rows of W3 times g (8-byte pieces of the operand-ordered
// copy, the same sum), and neither dout nor its copy is formed.
// Measured at 8192 rows (272 outputs): one wavefront per 32 rows with dense dout 18.5 us, and
// 33 us more to form it; now 7.6 us in all.
constexpr int kBwdWaves = 4;

template <bool Picks>
__global__ __launch_bounds__(64 * kBwdWaves) void mlp_bwd_act_kernel(const uint16_t* __restrict__ w,
                                                                     const uint16_t* __restrict__ wt, int DP, int Op,
                                                                     const float* __restrict__ dout, MlpPick pk, int B,
                                                                     const float* __restrict__ h1s,
                                                                     const float* __restrict__ h2s,
                                                                     uint16_t* __restrict__ gT)
{
    __shared__ v4s dz[8 * 2 * 64];   // [feature tile][row tile][lane]
    __shared__ Picked pick;
    const int lane = threadIdx.x & 63, r16 = lane & 15, g = lane >> 4, wv = threadIdx.x >> 6;
    const int row0 = blockIdx.x * 32, mt0 = 2 * wv;
    const uint16_t* W2T = wt + (size_t)H * DP;        // [H][H]
    const uint16_t* W3T = W2T + H * H;                // [H][Op]
    uint16_t* doT = gT;
    uint16_t* dz2T = gT + (size_t)Op * B;
    uint16_t* dz1T = dz2T + (size_t)H * B;

    // operands that depend on nothing: the transposed W2 rows and the activations
    v4s w2[2][8];
    v4f h2[2][2], h1[2][2];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
#pragma unroll
        for (int k = 0; k < 8; ++k) w2[m][k] = ld4(W2T + (size_t)(16 * (mt0 + m) + r16) * H + 16 * k + 4 * g);
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            const size_t at = (size_t)(row0 + 16 * nt + r16) * H + 16 * (mt0 + m) + 4 * g;
            h2[m][nt] = *reinterpret_cast<const v4f*>(h2s + at);
            h1[m][nt] = *reinterpret_cast<const v4f*>(h1s + at);
        }
    }
    v4f acc[2][2];
    if constexpr (Picks) {
        pick_rows(pk, Op, B, row0, pick);
        const uint16_t* W3 = w + (size_t)H * DP + H * H;   // operand order, K = H
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            const uint32_t sel = pick.sel[16 * nt + r16];
            const float gr = pick.g[16 * nt + r16];
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                // features 16 mt + 4 g .. + 3 of row f: lane 16 g + f % 16 of tile (f / 16, mt)
                auto piece = [&](uint32_t f) {
                    return ld4(W3 + ((size_t)((f >> 4) * (H / 16) + mt0 + m) * 64 + 16 * g + (f & 15)) * 4);
                };
                const v4s p1 = piece(sel & 0xFFFFu), p2 = piece(sel >> 16);
                // (the products are exact in fp32: one rounding, as in the matrix product)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[m][nt][j] = fmaf(gr, bf2f(p1[j]), gr * bf2f(p2[j]));
            }
        }
    } else {
#pragma unroll
        for (int m = 0; m < 2; ++m) acc[m][0] = acc[m][1] = v4f{0.f, 0.f, 0.f, 0.f};
        for (int ks = 0; ks < Op / 16; ++ks) {
            v4s bo[2];
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) {
                const int r = row0 + 16 * nt + r16;
                bo[nt] = pack_bf(*reinterpret_cast<const v4f*>(dout + (size_t)r * Op + 16 * ks + 4 * g));
                if ((ks & 3) == wv) store_t(doT, B, ks, row0 / 16 + nt, bo[nt]);
            }
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const v4s a = ld4(W3T + (size_t)(16 * (mt0 + m) + r16) * Op + 16 * ks + 4 * g);
                acc[m][0] = mfma(a, bo[0], acc[m][0]);
                acc[m][1] = mfma(a, bo[1], acc[m][1]);
            }
        }
    }
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            const v4f h = h2[m][nt];
            const v4s d = pack_bf(acc[m][nt] * (1.0f - h * h));
            dz[((mt0 + m) * 2 + nt) * 64 + lane] = d;
            store_t(dz2T, B, mt0 + m, row0 / 16 + nt, d);
        }
    __syncthreads();
    v4s b[2][8];
#pragma unroll
    for (int k = 0; k < 8; ++k)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) b[nt][k] = dz[(k * 2 + nt) * 64 + lane];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        v4f a0 = {0.f, 0.f, 0.f, 0.f}, a1 = a0;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            a0 = mfma(w2[m][k], b[0][k], a0);
            a1 = mfma(w2[m][k], b[1][k], a1);
        }
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            const v4f h = h1[m][nt];
            store_t(dz1T, B, mt0 + m, row0 / 16 + nt, pack_bf((nt == 0 ? a0 : a1) * (1.0f - h * h)));
        }
    }
}

// dW[f][k] = sum_r dZ[r][f] act[r][k] and db[f] = sum_r dZ[r][f].  A wavefront sums one 16 x 16
// tile of dW over the whole batch, 32 rows a step in two chains of products (rows 0..15 and
// 16..31 of each step), so the order of the sums does not depend on the launch.  Four tiles of
// one row of tiles share a workgroup and its A operands: the batch goes by in blocks of 16
// steps, each wavefront brings four steps of A to LDS (two buffers, one barrier a block) and
// loads its own B operands, both two blocks ahead.  Row tiles: layer 3 (Op/16, two workgroups each),
// layer 2 (8, two each), layer 1 (8).  Picks: layer 3's A is formed from the rows' two entries; an
// extra workgroup adds up the loss.
// Bound by the latency of the loads: with a step's loads issued at its start (one wavefront a
// workgroup, nothing shared) 8192 rows took 84 us, now 24.
constexpr int kGradWaves = 4, kGradSteps = 16;

template <bool Picks>
__global__ __launch_bounds__(64 * kGradWaves) __attribute__((amdgpu_waves_per_eu(1, 1))) void mlp_wgrad_kernel(const uint16_t* __restrict__ gT,
                                                                    const uint16_t* __restrict__ actT, MlpPick pk,
                                                                    int B, int DP, int Op, float* __restrict__ grad)
{
    constexpr int kOwn = kGradSteps / kGradWaves;   // steps of A a wavefront brings in
    __shared__ uint4 As[2][kGradSteps][64];
    const int lane = threadIdx.x & 63, r16 = lane & 15, g = lane >> 4, wv = threadIdx.x >> 6;
    const int T3 = (Op / 16) * 2;
    int t = blockIdx.x;
    if constexpr (Picks) {
        if (t == T3 + 16 + 8) {
            // the loss: the backward kernel's shares, one per 32 rows
            double sum = 0.0;
            for (int i = threadIdx.x; i < B / 32; i += 64 * kGradWaves) sum += pk.lpart[i];
            for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
            double* red = reinterpret_cast<double*>(&As[0][0][0]);
            if (lane == 0) red[wv] = sum;
            __syncthreads();
            if (threadIdx.x == 0) pk.loss[0] = (float)(((red[0] + red[1]) + (red[2] + red[3])) / B);
            return;
        }
    }
    const uint16_t* A;     // dZ^T [f][B]
    const uint16_t* Bm;    // act^T [k][B]
    float* dW;
    float* db;
    int ld, it, kt;
    bool picked = false;
    float* bias = grad + (size_t)H * DP + H * H + (size_t)Op * H;
    if (t < T3) {
        it = t / 2;
        kt = 4 * (t % 2) + wv;
        A = gT;
        Bm = actT + (size_t)(DP + H) * B;
        dW = grad + (size_t)H * DP + H * H;
        ld = H;
        db = bias + 2 * H;
        picked = Picks;
    } else if (t < T3 + 16) {
        t -= T3;
        it = t / 2;
        kt = 4 * (t % 2) + wv;
        A = gT + (size_t)Op * B;
        Bm = actT + (size_t)DP * B;
        dW = grad + (size_t)H * DP;
        ld = H;
        db = bias + H;
    } else {
        it = t - T3 - 16;
        kt = wv;
        A = gT + (size_t)(Op + H) * B;
        Bm = actT;
        dW = grad;
        ld = DP;
        db = bias;
    }
    const bool act = 16 * kt < ld;              // (layer 1 may have fewer tiles than wavefronts)
    const int steps = B / 32;
    const uint16_t* pa = A + (size_t)it * B * 16 + lane * 8;
    const uint16_t* pb = Bm + (size_t)(act ? kt : 0) * B * 16 + lane * 8;
    v4f c0 = {0.f, 0.f, 0.f, 0.f}, c1 = c0;
    float bs = 0.f;
    auto run = [&](auto is_picked) {
        constexpr bool kPicked = decltype(is_picked)::value;
        // operands of two blocks of steps in flight (past the end: the last step's, A taken as
        // zeros): this wavefront's share of A, and B.  Picks: A is a block of zeros in which each
        // thread sets the entries of two rows, and clears them when the buffer comes round again.
        constexpr int kRows = 32 * kGradSteps / (64 * kGradWaves);   // rows of a block per thread
        uint4 an[2][kPicked ? 1 : kOwn];
        uint32_t sn[2][kPicked ? kRows : 1];
        uint16_t gn[2][kPicked ? kRows : 1];
        int set[2][kPicked ? 2 * kRows : 1];       // entries set in each buffer (-1: none)
        uint4 bn[2][kGradSteps];
        auto load_a = [&](int s0, int p) {
            if constexpr (kPicked) {
#pragma unroll
                for (int i = 0; i < kRows; ++i) {
                    const int r = min(32 * s0 + (int)threadIdx.x + 64 * kGradWaves * i, B - 1);
                    sn[p][i] = pk.sel[r];
                    gn[p][i] = pk.g[r];
                }
            } else {
#pragma unroll
                for (int i = 0; i < kOwn; ++i)
                    an[p][i] = *reinterpret_cast<const uint4*>(pa + (size_t)min(s0 + kOwn * wv + i, steps - 1) * 512);
            }
        };
        auto load_b = [&](int s0, uint4 (&b)[kGradSteps]) {
#pragma unroll
            for (int i = 0; i < kGradSteps; ++i)
                b[i] = *reinterpret_cast<const uint4*>(pb + (size_t)min(s0 + i, steps - 1) * 512);
        };
        auto block = [&](int s0, int p, uint4 (&bn)[kGradSteps]) {
            uint4 (&lds)[kGradSteps][64] = As[p];
            if constexpr (kPicked) {
                uint16_t* e = reinterpret_cast<uint16_t*>(&lds[0][0]);
#pragma unroll
                for (int i = 0; i < 2 * kRows; ++i)
                    if (set[p][i] >= 0) e[set[p][i]] = 0;
#pragma unroll
                for (int i = 0; i < kRows; ++i) {
                    const int q = (int)threadIdx.x + 64 * kGradWaves * i;   // row of the block
                    // its place but for the feature: step, half, rows of four (see store_t)
                    const int at = (q >> 5) * 512 + ((q & 15) >> 2) * 128 + ((q >> 4) & 1) * 4 + (q & 3);
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const uint32_t f = h ? sn[p][i] >> 16 : sn[p][i] & 0xFFFFu;
                        const bool in = (int)(f >> 4) == it && 32 * s0 + q < B;
                        set[p][2 * i + h] = in ? at + (int)(f & 15) * 8 : -1;
                        if (in) e[set[p][2 * i + h]] = gn[p][i];
                    }
                }
            } else {
#pragma unroll
                for (int i = 0; i < kOwn; ++i) {
                    const uint32_t in = s0 + kOwn * wv + i < steps ? ~0u : 0u;
                    const uint4 w = an[p][i];
                    lds[kOwn * wv + i][lane] = make_uint4(w.x & in, w.y & in, w.z & in, w.w & in);
                }
            }
            load_a(s0 + 2 * kGradSteps, p);
            __syncthreads();
            uint4 a[kGradSteps];
#pragma unroll
            for (int i = 0; i < kGradSteps; ++i) a[i] = lds[i][lane];
            __builtin_amdgcn_sched_barrier(0);   // every read of the block in flight at once
            auto lo = [](uint4 v) { return __builtin_bit_cast(v4s, make_uint2(v.x, v.y)); };
            auto hi = [](uint4 v) { return __builtin_bit_cast(v4s, make_uint2(v.z, v.w)); };
#pragma unroll
            for (int i = 0; i < kGradSteps; ++i) {
                c0 = mfma(lo(a[i]), lo(bn[i]), c0);
                c1 = mfma(hi(a[i]), hi(bn[i]), c1);
            }
            load_b(s0 + 2 * kGradSteps, bn);
            if (kt == 0) {
#pragma unroll
                for (int i = 0; i < kGradSteps; ++i) {
                    const v4s a0 = lo(a[i]), a1 = hi(a[i]);
                    bs += (bf2f(a0[0]) + bf2f(a0[1])) + (bf2f(a0[2]) + bf2f(a0[3])) + (bf2f(a1[0]) + bf2f(a1[1])) +
                          (bf2f(a1[2]) + bf2f(a1[3]));
                }
            }
        };
        load_a(0, 0);
        load_b(0, bn[0]);
        load_a(kGradSteps, 1);
        load_b(kGradSteps, bn[1]);
        if constexpr (kPicked) {
#pragma unroll
            for (int i = 0; i < 2 * kRows; ++i) set[0][i] = set[1][i] = -1;
            for (int i = threadIdx.x; i < 2 * kGradSteps * 64; i += 64 * kGradWaves)
                (&As[0][0][0])[i] = make_uint4(0, 0, 0, 0);
            __syncthreads();
        }
        for (int s0 = 0; s0 < steps; s0 += 2 * kGradSteps) {
            block(s0, 0, bn[0]);
            block(s0 + kGradSteps, 1, bn[1]);
        }
    };
    if (picked)
        run(std::integral_constant<bool, Picks>{});
    else
        run(std::integral_constant<bool, false>{});
    const v4f c = c0 + c1;
    if (act) {
#pragma unroll
        for (int j = 0; j < 4; ++j) dW[(size_t)(16 * it + 4 * g + j) * ld + 16 * kt + r16] = c[j];
    }
    if (kt == 0) {
        bs += __shfl_xor(bs, 16);
        bs += __shfl_xor(bs, 32);
        if (g == 0) db[16 * it + r16] = bs;
    }
}

// Adam step (update != 0) and/or refresh of the BF16 copies w and wt from param.
__global__ __launch_bounds__(256) void mlp_adam_kernel(float* __restrict__ p, const float* __restrict__ gr,
                                                       float* __restrict__ m, float* __restrict__ v,
                                                       uint16_t* __restrict__ w, uint16_t* __restrict__ wt,
                                                       int64_t P, int DP, int Op, int update, float lr, float b1,
                                                       float b2, float eps, float c1, float c2)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= P) return;
    float x = p[i];
    if (update) {
        const float gi = gr[i];
        const float mi = b1 * m[i] + (1.0f - b1) * gi;
        const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        x -= lr * (mi * c1) / (sqrtf(vi * c2) + eps);
        p[i] = x;
    }
    const int64_t s2 = (int64_t)H * DP, s3 = s2 + H * H, nw = s3 + (int64_t)Op * H;
    if (i < nw) {
        const uint16_t bits = f2bf(x);
        // element (row, col) of the M x K layer at `base`: fragment copy at
        // ((row/16 (K/16) + col/16) 64 + lane) 4 + col % 4, lane = 16 ((col % 16) / 4) + row % 16;
        // transposed copy at col M + row
        int64_t base, K, M;
        if (i < s2) {
            base = 0, K = DP, M = H;
        } else if (i < s3) {
            base = s2, K = H, M = H;
        } else {
            base = s3, K = H, M = Op;
        }
        const int64_t row = (i - base) / K, col = (i - base) % K;
        const int64_t lane = 16 * ((col & 15) >> 2) + (row & 15);
        w[base + (((row >> 4) * (K >> 4) + (col >> 4)) * 64 + lane) * 4 + (col & 3)] = bits;
        wt[base + col * M + row] = bits;
    }
}

}  // namespace

int64_t mlp_param_count(int dp, int op) { return (int64_t)H * dp + H * H + (int64_t)op * H + H + H + op; }
int64_t mlp_weight_count(int dp, int op) { return (int64_t)H * dp + H * H + (int64_t)op * H; }

int64_t mlp_work_bytes(int dp, int op, int B)
{
    const int64_t f32 = 2 * (int64_t)B * H * 4;                       // h1, h2 fp32 [B][H]
    const int64_t act = (int64_t)(dp + 2 * H) * B * 2;                // x^T, h1^T, h2^T bf16
    const int64_t gra = (int64_t)(op + 2 * H) * B * 2;                // dout^T, dz2^T, dz1^T bf16
    auto al = [](int64_t v) { return (v + 255) & ~(int64_t)255; };
    return al(f32) + al(act) + al(gra);
}

MlpWork mlp_work_carve(void* work, int dp, int op, int B)
{
    auto al = [](int64_t v) { return (v + 255) & ~(int64_t)255; };
    char* p = static_cast<char*>(work);
    MlpWork wk;
    wk.h1 = reinterpret_cast<float*>(p);
    wk.h2 = wk.h1 + (size_t)B * H;
    p += al(2 * (int64_t)B * H * 4);
    wk.actT = reinterpret_cast<uint16_t*>(p);
    p += al((int64_t)(dp + 2 * H) * B * 2);
    wk.gT = reinterpret_cast<uint16_t*>(p);
    return wk;
}

hipError_t mlp_forward_launch(const MlpNet& net, const uint16_t* x, int B, float* out, const MlpWork* wk,
                              hipStream_t st)
{
    if (B == 0) return hipSuccess;
    const float* bias = net.param + mlp_weight_count(net.dp, net.op);
    float* h1 = wk ? wk->h1 : nullptr;
    float* h2 = wk ? wk->h2 : nullptr;
    uint16_t* actT = wk ? wk->actT : nullptr;
    const dim3 grid((unsigned)(B / 32)), block(64 * kFwdWaves);
    switch (net.dp / 16) {
    case 1: hipLaunchKernelGGL(mlp_fwd_kernel<1>, grid, block, 0, st, net.w, bias, x, B, net.op, out, h1, h2, actT); break;
    case 2: hipLaunchKernelGGL(mlp_fwd_kernel<2>, grid, block, 0, st, net.w, bias, x, B, net.op, out, h1, h2, actT); break;
    case 3: hipLaunchKernelGGL(mlp_fwd_kernel<3>, grid, block, 0, st, net.w, bias, x, B, net.op, out, h1, h2, actT); break;
    case 4: hipLaunchKernelGGL(mlp_fwd_kernel<4>, grid, block, 0, st, net.w, bias, x, B, net.op, out, h1, h2, actT); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

namespace {

template <bool Picks>
hipError_t backward(const MlpNet& net, const float* dout, const MlpPick& pk, int B, const MlpWork& wk, hipStream_t st)
{
    if (B == 0) return hipSuccess;
    hipLaunchKernelGGL(mlp_bwd_act_kernel<Picks>, dim3((unsigned)(B / 32)), dim3(64 * kBwdWaves), 0, st, net.w, net.wt,
                       net.dp, net.op, dout, pk, B, wk.h1, wk.h2, wk.gT);
    const int tiles = (net.op / 16) * 2 + 16 + 8;
    hipLaunchKernelGGL(mlp_wgrad_kernel<Picks>, dim3((unsigned)(tiles + (Picks && pk.loss ? 1 : 0))),
                       dim3(64 * kGradWaves), 0, st, wk.gT, wk.actT, pk, B, net.dp, net.op, net.grad);
    return hipGetLastError();
}

}  // namespace

hipError_t mlp_backward_launch(const MlpNet& net, const float* dout, int B, const MlpWork& wk, hipStream_t st)
{
    return backward<false>(net, dout, MlpPick{}, B, wk, st);
}

hipError_t mlp_backward_picked_launch(const MlpNet& net, const MlpPick& pk, int B, const MlpWork& wk, hipStream_t st)
{
    return backward<true>(net, nullptr, pk, B, wk, st);
}

hipError_t mlp_adam_launch(const MlpNet& net, bool update, float lr, float b1, float b2, float eps, int t,
                           hipStream_t st)
{
    const int64_t P = mlp_param_count(net.dp, net.op);
    const float c1 = update ? (float)(1.0 / (1.0 - pow((double)b1, (double)t))) : 1.0f;
    const float c2 = update ? (float)(1.0 / (1.0 - pow((double)b2, (double)t))) : 1.0f;
    hipLaunchKernelGGL(mlp_adam_kernel, dim3((unsigned)((P + 255) / 256)), dim3(256), 0, st, net.param, net.grad,
                       net.m, net.v, net.w, net.wt, P, net.dp, net.op, update ? 1 : 0, lr, b1, b2, eps, c1, c2);
    return hipGetLastError();
}

}  // namespace apm
