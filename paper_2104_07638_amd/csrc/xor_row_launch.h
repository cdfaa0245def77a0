// xor_row_launch.h -- launch of the register block-minor kernels (xor_row.h) for one type.
#pragma once
#include "xor_row.h"

namespace apm {
namespace xrow {

__global__ static void xor_info_kernel(int32_t* info, int32_t batch)
{
    const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (i < batch) info[i] = 0;
}

template <class F, int MODE, int WAVES, int N>
hipError_t launch_n(const LaunchXor& L, hipStream_t st)
{
    if constexpr (N > 16) {
        return hipErrorInvalidValue;
    } else {
        if (L.n != N) return launch_n<F, MODE, WAVES, N + 1>(L, st);
        constexpr int T = top_levels(N);
        const int64_t units = (int64_t)L.batch << T;
        // Wavefronts per matrix: as many as bring the launch to four per wavefront slot (the
        // units share nothing, so a split costs only the input check of each wavefront).
        int split = 1;
        while (4 * split < (1 << T) && (int64_t)L.batch * split < 16 * kCus * WAVES) split *= 2;
        const int per_wave = T >= 2 ? (1 << T) / split : 4;
        const int64_t grid = (units + per_wave - 1) / per_wave;
        if (split > 1 && L.info)
            hipLaunchKernelGGL(xor_info_kernel, dim3((unsigned)((L.batch + 255) / 256)), dim3(256), 0, st, L.info,
                               L.batch);
        hipLaunchKernelGGL((xor_row_kernel<F, N, MODE, WAVES>), dim3((unsigned)grid), dim3(64), 0, st,
                           static_cast<const typename F::E*>(L.A), static_cast<typename F::E*>(L.out), L.info, units,
                           per_wave, split > 1 ? 1 : 0);
        return hipGetLastError();
    }
}

}  // namespace xrow
}  // namespace apm
