// Moment form of the FP64 element contraction (moments.hip): plan constants
// and launchers.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tables.hpp"

namespace pufe {

constexpr int kMomMaxPoints = 288;   // points of one stage (whole planes of a leaf)

// Planes per stage and LDS bytes of an element of nt row tiles in a work
// group of nw waves: the most planes that keep two stages within the work
// group's share of a CU (one stage where two do not fit); planes = 0 when not
// even one plane fits.
struct MomStage {
    int planes, buffers;
    size_t lds;
};
MomStage mom_stage(int nt, int nimg, int n, int p, int nw);

hipError_t init_moment_attributes();
// Contraction of the items of one work group width (nw = 4 or 8) of problems
// whose rules have the same x steps (n points, 4 a step): moments of every
// item's tasks into its slots.  V and wimg: those of the problem of a
// single-problem launch (null: each problem's own).
hipError_t launch_moments(int nw, int n, int lmax, bool gen, bool skew, const CtxDev *ctxs, const MomItemDev *items,
                          int n_items, const int32_t *wave_task, const double *V, const double *wimg, size_t lds,
                          hipStream_t st);
// Moments of the classical part of the items' elements and leaves.
hipError_t launch_classical_moments(const CtxDev *ctxs, const MomItemDev *items, int n_items, const double *V,
                                    hipStream_t st);
// Sum of the K-chunk moments of every listed (element, slot, problem) into chunk 0.
hipError_t launch_moment_reduce(const CtxDev *ctxs, const int4 *list, int n, hipStream_t st);
// Element matrices (the upper 16x16 tiles of slot chunk 0) from the moments:
// list entries (element, kind, index, problem): an energy quad, a pair of
// enrichment functions, the classical part.
enum { MOM_X_ENR = 0, MOM_X_MIXED = 1, MOM_X_FE = 2 };
hipError_t launch_moment_expand(const CtxDev *ctxs, const int4 *list, int n, double *partial, hipStream_t st);

}  // namespace pufe
