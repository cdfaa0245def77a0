// lead.hip -- leading principal minors by successive Schur complements (Sec. III) on gfx950.
//
// det A[:k, :k] for k = 1..n: elimination without row exchanges on the leading block, the
// k-th pivot being the ratio of consecutive leading minors (the ratio rule of Sec. II
// along the tree's rightmost path).  As the paper notes, no pivot correction is possible
// here (it would need minors that are never formed), so a zero pivot makes the later
// minors non-finite (info = -3).
//
// Mapping: a matrix is held by a row of 16 lanes, lane j holding column j (and column 16 + j
// above order 16) in registers; four matrices per wavefront.  The pivot column reaches the
// lanes by DPP row broadcast inside the multiply-adds (row_fma.h), the scaled pivot row is in
// its lanes already, so a step needs no memory and no synchronisation.  The order is rounded
// up to a multiple of 4 (the kernel's compile-time order R); the rows and columns past n repeat
// the last one and influence none before them.
// Bound by the input (8 n^2 bytes a matrix) and the chain of n pivots.  8192 matrices of order
// 16: one wavefront per matrix with the matrix in LDS 31 us, this 5.9 us (3.0 TB/s).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "apm_device.h"
#include "apm_kernels.h"
#include "row_fma.h"

namespace apm {
namespace {

constexpr int kLeadMax = 32;

template <class F, int R>
struct Lead {
    using E = typename F::E;
    static constexpr bool kTwo = R > 16;           // a second column per lane
    static constexpr int R2 = kTwo ? R : 1;
    E a[R], b[R2];                                 // columns j and 16 + j, by rows
    E o0, o1;                                      // leading minors j + 1 and 17 + j of lane j
    E mk;
    double chk;
    int l16;

    // rows I .. I + 3, all below pivot row K (rows above it in the first group of four are left)
    template <int K, int I>
    __device__ __forceinline__ void below(E wa, E wb)
    {
        if constexpr (I < R) {
            constexpr int P = K % 16;
            if constexpr (I > K) {
                if constexpr (K >= 16) {
                    row_elim<P>(b[I], b[I + 1], b[I + 2], b[I + 3], wb);
                } else {
                    if constexpr (kTwo) row_sub<P>(b[I], b[I + 1], b[I + 2], b[I + 3], a[I], a[I + 1], a[I + 2], a[I + 3], wb);
                    row_elim<P>(a[I], a[I + 1], a[I + 2], a[I + 3], wa);
                }
            } else {
                one<K, I>(wa, wb);
                one<K, I + 1>(wa, wb);
                one<K, I + 2>(wa, wb);
                one<K, I + 3>(wa, wb);
            }
            below<K, I + 4>(wa, wb);
        }
    }

    // row I alone
    template <int K, int I>
    __device__ __forceinline__ void one(E wa, E wb)
    {
        if constexpr (I > K) {
            constexpr int P = K % 16;
            if constexpr (K >= 16) {
                b[I] = F::upd(b[I], bcast<P>(b[I]), wb);
            } else {
                const E c = bcast<P>(a[I]);
                if constexpr (kTwo) b[I] = F::upd(b[I], c, wb);
                a[I] = F::upd(a[I], c, wa);
            }
        }
    }

    template <int P>
    static __device__ __forceinline__ double bcast(double v) { return row_bcast_after<P>(v); }
    template <int P>
    static __device__ __forceinline__ cd bcast(cd v) { return {row_bcast_after<P>(v.x), row_bcast_after<P>(v.y)}; }

    template <int K>
    __device__ __forceinline__ void steps(int n)
    {
        if constexpr (K < R) {
            if (K < n) {
                constexpr int P = K % 16;
                E pv;
                if constexpr (K >= 16)
                    pv = bcast<P>(b[K]);
                else
                    pv = bcast<P>(a[K]);
                mk = F::bmul(mk, pv, 0);
                chk += F::fincheck(mk);
                if (l16 == P) {
                    if constexpr (K >= 16)
                        o1 = mk;
                    else
                        o0 = mk;
                }
                if constexpr (K + 1 < R) {
                    const typename F::R r = F::recip(pv);
                    E wa = F::rowscale(a[K], r), wb = wa;
                    if constexpr (kTwo) wb = F::rowscale(b[K], r);
                    // in place: the pivot's lane keeps its column (its multipliers)
                    if (F::kComplex && l16 == P) {
                        if constexpr (K >= 16)
                            wb = F::zero();
                        else
                            wa = F::zero();
                    }
                    below<K, K / 4 * 4>(wa, wb);
                }
            }
            steps<K + 1>(n);
        }
    }
};

template <class F, int R>
__global__ __launch_bounds__(64) void lead_kernel(const typename F::E* __restrict__ A, typename F::E* __restrict__ out,
                                                  int32_t* __restrict__ info, int32_t batch, int n)
{
    using E = typename F::E;
    using L = Lead<F, R>;
    const int lane = threadIdx.x;
    const int64_t m = (int64_t)blockIdx.x * 4 + (lane >> 4);
    const bool valid = m < batch;
    const E* A0 = A + (valid ? m : batch - 1) * n * n;
    L s;
    s.l16 = lane & 15;
    const int ca = s.l16 < n ? s.l16 : n - 1, cb = 16 + s.l16 < n ? 16 + s.l16 : n - 1;
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const E* row = A0 + (i < n ? i : n - 1) * n;
        s.a[i] = load_reg(&row[ca]);
        if constexpr (L::kTwo) s.b[i] = load_reg(&row[cb]);
    }
    bool fin = true;
#pragma unroll
    for (int i = 0; i < R; ++i) {
        fin = fin && F::in_finite(s.a[i]);
        if constexpr (L::kTwo) fin = fin && F::in_finite(s.b[i]);
    }
    const bool finite = ((ballot(!fin) >> (lane & 48)) & 0xFFFF) == 0;
    s.mk = F::one();
    if (!finite) F::store_nan(&s.mk, nullptr, 0, false);   // makes every minor NaN
    s.o0 = s.o1 = F::zero();
    s.chk = 0.0;
    s.template steps<0>(n);
    if (!valid) return;
    E* ob = out + m * n;
    if (s.l16 < n) ob[s.l16] = s.o0;
    if (L::kTwo && 16 + s.l16 < n) ob[16 + s.l16] = s.o1;
    if (info && s.l16 == 0) info[m] = !finite ? -2 : s.chk != 0.0 ? -3 : 0;
}

template <class F, int R>
hipError_t launch(const void* A, void* out, int32_t* info, int32_t batch, int n, hipStream_t st)
{
    if constexpr (R > kLeadMax) {
        return hipErrorInvalidValue;
    } else {
        if (n > R) return launch<F, R + 4>(A, out, info, batch, n, st);
        hipLaunchKernelGGL((lead_kernel<F, R>), dim3((unsigned)((batch + 3) / 4)), dim3(64), 0, st,
                           static_cast<const typename F::E*>(A), static_cast<typename F::E*>(out), info, batch, n);
        return hipGetLastError();
    }
}

}  // namespace

hipError_t lead_launch(int dtype, const void* A, void* out, int32_t* info, int32_t batch, int n, hipStream_t st)
{
    if (n < 1 || n > kLeadMax) return hipErrorInvalidValue;
    if (dtype == 0) return launch<FR64, 4>(A, out, info, batch, n, st);
    if (dtype == 2) return launch<FC128, 4>(A, out, info, batch, n, st);
    return hipErrorInvalidValue;
}

}  // namespace apm
