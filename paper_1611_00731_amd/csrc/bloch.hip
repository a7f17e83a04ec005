// Bloch-periodic enrichment (eq. Psi with f(R) = exp(i k.R)): per-k image
// weights for the contraction.
#include <hip/hip_runtime.h>

#include "bloch.hpp"
#include "device_common.hpp"

namespace pufe {

// w[i] = cos(2 pi kappa.n_i) for the entries of the real-part groups and
// sin(2 pi kappa.n_i) for those of the imaginary-part copies; nk[4 i .. 4 i + 3]
// = (n_i, kind).
__global__ void image_weights_kernel(const int32_t *__restrict__ nk, int64_t n, double k0, double k1, double k2,
                                     double *__restrict__ w) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int32_t *e = nk + 4 * i;
    double sn, cs;
    sincos(2.0 * M_PI * (k0 * e[0] + k1 * e[1] + k2 * e[2]), &sn, &cs);
    w[i] = e[3] ? sn : cs;
}

hipError_t launch_image_weights(const int32_t *img_nk, int64_t n, const double kap[3], double *w, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    image_weights_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(img_nk, n, kap[0], kap[1], kap[2], w);
    return hipGetLastError();
}

}  // namespace pufe
