// What the kernels of the moment forms share.
#pragma once
#include <hip/hip_runtime.h>

namespace pufe {

typedef double dbl2 __attribute__((ext_vector_type(2)));

// Four independent 4x4 tiles, K = 4.
__device__ __forceinline__ double mfma4(double a, double b, double c) {
    return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}

// Value at t of Lagrange polynomial k on M equidistant nodes of [-1, 1].
template <int M>
__device__ __forceinline__ double lagrange_equi(int k, double t) {
    constexpr double h = 2.0 / (M - 1);
    // prod_{j != k} (k - j) h = (-1)^(M - 1 - k) k! (M - 1 - k)! h^(M - 1)
    constexpr double f[5] = {1.0, 1.0, 2.0, 6.0, 24.0};
    double v = 1.0, d = 1.0;
#pragma unroll
    for (int j = 0; j < M; ++j) {
        v *= j == k ? 1.0 : t - (-1.0 + j * h);
        const double inv = 1.0 / (f[j] * f[M - 1 - j] * (M == 3 ? h * h : (M == 4 ? h * h * h : h * h * h * h)));
        d = j == k ? ((M - 1 - j) & 1 ? -inv : inv) : d;
    }
    return v * d;
}

}  // namespace pufe
