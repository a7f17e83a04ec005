// Launchers of the Bloch-periodic enrichment kernels (bloch.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tables.hpp"

namespace pufe {

// Image weights of one k-point: w[i] = cos or sin(2 pi kappa.n_i) by the
// kind of entry i (img_nk: 4 ints per entry, the lattice shift and the kind).
hipError_t launch_image_weights(const int32_t *img_nk, int64_t n, const double kap[3], double *w, hipStream_t st);

}  // namespace pufe
