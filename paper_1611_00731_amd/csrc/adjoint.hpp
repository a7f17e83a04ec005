// Adjoint of the assembly in moment form (adjoint.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tables.hpp"

namespace pufe {

// Stage of an element of nt row tiles and the work group that runs it: planes
// per stage, or lines of one plane (planes = 0) where a plane does not fit;
// waves 4 (two groups per CU) or 8.
// waves = 0: it does not fit at all.
struct AdjStage {
    int waves, planes, lines;
    size_t lds;
};
AdjStage adj_stage(int nt, int nimg, int n, int p);

// Doubles of an element's folded adjoint matrices.
int64_t adj_doubles(int nt, int p);
// Wave tasks of an element: three per quad of ordered tile pairs, two per group
// of 16 functions.
static inline __host__ __device__ int adj_tasks(int nt) { return 3 * mom_quads_b(nt) + 2 * ((nt + 3) / 4); }

// Item: element, leaf_b .. leaf_e - 1 its stages counted from the element's
// first leaf, tab = planes | lines << 8, chunk = the item's partial-force slot.
hipError_t init_adjoint_attributes();
enum { ADJ_PAIRS = 0, ADJ_MIXED = 1, ADJ_CLASSICAL = 2 };
// Fold Ps and Qs (either may be null: zero) of the listed (element, kind,
// index) into the coefficients of the element's moments, at lam + base[element].
hipError_t launch_adjoint_fold(const CtxDev *ctx, const int4 *list, int n, const int64_t *pt_off, const double *Ps,
                               const double *Qs, const int64_t *base, double *lam, hipStream_t st);
// dL/dV of the items' points (dV may be null) and the partial forces of every
// item and group, fpart[(slot max_ngrp + group) 3 + k].
hipError_t launch_adjoint_moments(int nw, const CtxDev *ctx, const MomItemDev *items, int n_items, const int64_t *base,
                                  const double *lam, const double *V, double *dV, double *fpart, int max_ngrp, size_t lds,
                                  hipStream_t st);

}  // namespace pufe
