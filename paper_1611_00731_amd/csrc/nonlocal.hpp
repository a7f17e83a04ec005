// Host launchers of the separable nonlocal term (nonlocal.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.hpp"
#include "tables.hpp"

namespace pufe {

size_t nl_lds_bytes(int npad, int ncol, int nfun, int nimg, int nleaf, int n3);
hipError_t init_nonlocal_attributes();
hipError_t launch_nl_f(int lmax, const KParams &kp, int n_items, const NlItemDev *items, const ElemDev *elems,
                       const GroupDev *groups, const double *img, const int32_t *edof, const uint32_t *leaves,
                       const PGroupDev *pgroups, double *Fp, size_t lds, hipStream_t st);
// The same in moment form (orders 1 and 2): planes of a leaf per stage, LDS of
// an element, tasks of an item at most.
int nl_moment_planes(int n);
size_t nl_moment_lds(int nfun, int ncol, int nimg, int n, int planes);
static inline int nl_moment_tasks(int nfun, int ncol) {
    const int nt = (nfun + 3) / 4, ntc = (ncol + 3) / 4;
    return (nt * ntc + 3) / 4 + (ntc + 3) / 4;
}
constexpr int kNlMomentTasks = 16;
hipError_t launch_nl_moments(const KParams &kp, int n_items, const NlItemDev *items, const ElemDev *elems,
                             const GroupDev *groups, const double *img, const int32_t *edof, const uint32_t *leaves,
                             const PGroupDev *pgroups, int planes, double *Fp, size_t lds, hipStream_t st);
hipError_t launch_nl_reduce(const ElemDev *elems, const int32_t *nl_elems, int n, double *Fp, hipStream_t st);
// bpart: the partner table of the Bloch-periodic enrichment's rows (null for
// the periodic form)
hipError_t launch_nl_gather(const KParams &kp, const ElemDev *elems, const PGroupDev *pgroups, const int32_t *edof,
                            const int32_t *bpart, const int64_t *dof_el_off, const int2 *dof_el, const double *Fp,
                            const KPoints &kps, int n_pfun, int64_t n_dof, double2 *f, hipStream_t st);

}  // namespace pufe
