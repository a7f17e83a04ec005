// Launchers of the self-consistent field kernels (scf.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tables.hpp"

namespace pufe {

// Load vector of the classical FE space, b[v * nfs + s] = sum_q w_q phi f_q:
// per-element sums into be (nel x 32), then a gather per DOF over its
// (element, local function) pairs.
hipError_t launch_fe_load(const KParams &kp, const ElemDev *elems, int64_t nel, const uint32_t *leaves,
                          const double *f, double *be, int64_t nv, int nfs, const int64_t *dof_off,
                          const int64_t *dof_el_off, const int2 *dof_el, double *b, hipStream_t st);
// out_q = sum_i u_i phi_i(x_q) over the classical FE functions.
hipError_t launch_fe_eval(const KParams &kp, const ElemDev *elems, const int32_t *edof, const uint32_t *leaves,
                          const int32_t *leaf_elem, int64_t n_qp, const double *u, double *out, hipStream_t st);
// The nfs x nfs classical FE corner of every BSR block of A, times scale.
hipError_t launch_fe_blocks(int64_t nnzb, int nfs, const int32_t *bcol, const int64_t *bval_off,
                            const int64_t *dof_off, const double *A, double scale, double *K, hipStream_t st);
// *out = a . b in a fixed order; part holds dot_partial_slots() doubles.
hipError_t launch_dot(int64_t n, const double *a, const double *b, double *part, double *out, hipStream_t st);
// The dot_partial_slots() block partials of a . b alone.
hipError_t launch_dot_partials(int64_t n, const double *a, const double *b, double *part, hipStream_t st);
int dot_partial_slots();

// Conjugate gradients on the classical FE space with their scalars on the
// device: |r|^2 of the last two iterations, the first residual's norm, the
// relative residual, iterations done, and whether the solve is over: `done` is
// written by the products (the tolerance or the iteration limit is met, or
// `ended` was set), `ended` by the updates (p . Ap <= 0, or `done` was set).
struct CgState {
    double rr[2], r0, rel;
    int32_t it, done, ended;
};
struct CgSolve {
    int64_t nv;
    int nfs;
    const int64_t *brow_ptr;
    const int32_t *bcol;
    const double *K;
    double *r, *p0, *p1, *Ap, *x;
    double *part;   // cg_partial_slots(nv) doubles
    CgState *state;
};
int64_t cg_partial_slots(int64_t nv);
// r = 4 pi (b - nbar m) with nbar = (sum of the partials bpart) / msum, x = 0
hipError_t launch_cg_start(const CgSolve &c, const double *b, const double *m, const double *bpart, double msum,
                           hipStream_t st);
// Iteration it (no effect once the solve has ended); check: the test of the
// residual after the last iteration only.
hipError_t launch_cg_iteration(const CgSolve &c, int it, double tol, bool check, hipStream_t st);
// x -= (sum of the partials mpart) / msum, also into out if it is not null
hipError_t launch_cg_mean(const CgSolve &c, const double *mpart, double msum, double *out, hipStream_t st);
hipError_t launch_lda_xc(int64_t n, const double *rho, double *vxc, double *exc, hipStream_t st);

}  // namespace pufe
