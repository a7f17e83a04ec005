// Separable nonlocal term of the PUFE Hamiltonian (eq. disceig3d) on gfx950:
//   H_ij += sum_J h_J f_J^i conj(f_J^j),
//   f_J^i = int phi_i^* sum_n exp(i k . a_n) v_J(x - tau - a_n) dx.
// Formulation with Bloch phases on the FE and PU functions (phi_i = p_a N_a
// on an element) and projector images n:
//   f_J^i = sum_{(e, a) -> i} conj(p_a) sum_{images n of J reaching e}
//           exp(2 pi i kappa . n) F_e[a][col(J, n)],
//   F_e[a][c] = sum_q w_q N_a(x_q) v_c(x_q)          (real, k-independent)
// F_e is a contraction of the element's basis values with its projector
// values over the quadrature points, on FP64 MFMA (nl_f_kernel); with the
// Bloch-periodic enrichment the element's rows are its real rows and the
// imaginary parts of its enriched functions (images weighted per k-point), so
// F_e is per k-point and the gather takes conj(phi) = real - i imaginary, with
// the boundary phase on the classical FE rows only; the
// phases and the sum over the elements of a DOF are a gather per (J, DOF)
// (nl_gather_kernel), and the assembly adds the low-rank term to the blocks that
// a projector image couples (gather.hip).  No atomics; fixed order.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "basis.hpp"
#include "device_common.hpp"
#include "kernels.hpp"
#include "nonlocal.hpp"
#include "stage.hpp"
#include "tables.hpp"

namespace pufe {

typedef double double4_t __attribute__((ext_vector_type(4)));

constexpr int kNlQ = 16;        // points per stage
constexpr int kNlQU = kNlQ + 1; // row stride (doubles) of the value and projector tables: offset banks
constexpr int kNlThreads = 256;

// LDS map (per work item):
//   sU[npad][QU]     sqrt(w) N_a at the stage points (rows past nloc zero)
//   sPv[ncp][QU]     sqrt(w) v_c at the stage points (columns past ncol zero)
//   sPsi[f][4 Q]     enrichment functions (value, gradient)
//   sGeo[GEO][Q]     per-point geometry
//   sImg, sG, sPG, sEd, sCS, sLeaf, sPt, sGx, sGs
struct NlLds {
    static __host__ __device__ size_t bytes(int npad, int ncp, int nfun, int nimg, int nleaf, int n3) {
        return sizeof(double) * ((size_t)npad * kNlQU + (size_t)ncp * kNlQU + (size_t)nfun * 4 * kNlQ +
                                 (size_t)40 * kNlQ + (size_t)nimg * 3 + 2 * kMaxGauss) +
               sizeof(GroupDev) * kMaxGroups + sizeof(PGroupDev) * kMaxPGroups + sizeof(int32_t) * (kMaxNloc + 16) +
               sizeof(uint32_t) * ((size_t)nleaf + n3) + 64;
    }
};

// Projector coefficients of one element over one range of leaves, for the
// item's row tiles R0 .. R0 + nR - 1 against every column tile: FP64 MFMAs
// (v_mfma_f64_16x16x4f64, k = 4 points per instruction).
template <int LMAX>
__global__ __launch_bounds__(kNlThreads) void nl_f_kernel(
    const KParams kpg, const NlItemDev *__restrict__ items, const ElemDev *__restrict__ elems,
    const GroupDev *__restrict__ groups, const double *__restrict__ img, const int32_t *__restrict__ edof,
    const uint32_t *__restrict__ leaves, const PGroupDev *__restrict__ pgroups, double *__restrict__ Fp) {
    constexpr int Q = kNlQ, QU = kNlQU, NT = kNlThreads;
    extern __shared__ __attribute__((aligned(16))) double smem[];
    const NlItemDev it = items[blockIdx.x];
    const KLocal kp = load_klocal(kpg);
    const ElemDev &el = elems[it.elem];
    const int nloc = el.nloc, nfe = el.nfe, ngrp = el.ngrp, nfun = el.nfun, npg = el.npg, ncol = el.ncol;
    const int T = (nloc + 15) / 16, npad = 16 * T, TC = (ncol + 15) / 16, ncp = 16 * TC;
    const int img0 = ngrp > 0 ? groups[el.grp_off].img_off : 0;
    const int nimg = ngrp > 0 ? groups[el.grp_off + ngrp - 1].img_off + groups[el.grp_off + ngrp - 1].nimg - img0 : 0;
    const uint32_t n3 = (uint32_t)kp.n3, n = (uint32_t)kp.n;
    double *sU = smem;
    double *sPv = sU + (size_t)npad * QU;
    double *sPsi = sPv + (size_t)ncp * QU;
    double *sGeo = sPsi + (size_t)nfun * 4 * Q;
    double *sImg = sGeo + 40 * Q;
    double *sGx = sImg + 3 * (size_t)nimg, *sGs = sGx + kMaxGauss;
    GroupDev *sG = (GroupDev *)(sGs + kMaxGauss);
    PGroupDev *sPG = (PGroupDev *)(sG + kMaxGroups);
    int32_t *sEd = (int32_t *)(sPG + kMaxPGroups);
    int *sCS = sEd + kMaxNloc;
    uint32_t *sLeaf = (uint32_t *)(sCS + 16);
    uint32_t *sPt = sLeaf + (it.leaf_e - it.leaf_b);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t nli = (uint32_t)((it.leaf_e - it.leaf_b) * n3);
    for (int k = tid; k < nloc - nfe; k += NT) sEd[k] = edof[el.edof_off + k];
    corner_starts((const PUFE_GLOBAL int32_t *)(edof + el.edof_off), nloc - nfe, sCS, tid, NT);
    for (int g = tid; g < ngrp; g += NT) {
        GroupDev G = groups[el.grp_off + g];
        G.img_off -= img0;
        sG[g] = G;
    }
    for (int g = tid; g < npg; g += NT) sPG[g] = pgroups[el.pg_off + g];
    for (int k = tid; k < 3 * nimg; k += NT) sImg[k] = img[3 * (size_t)img0 + k];
    for (int64_t k = tid; k < it.leaf_e - it.leaf_b; k += NT) sLeaf[k] = leaves[it.leaf_b + k];
    for (uint32_t j = tid; j < n3; j += NT) sPt[j] = (j % n) | (((j / n) % n) << 8) | ((j / (n * n)) << 16);
    // padding rows and columns stay zero
    for (int k = tid; k < (npad - nloc) * QU; k += NT) sU[(size_t)nloc * QU + k] = 0.0;
    for (int k = tid; k < (ncp - ncol) * QU; k += NT) sPv[(size_t)ncol * QU + k] = 0.0;
    if (tid < kp.n) {
        sGx[tid] = kpg.gx[tid];
        sGs[tid] = sqrt(kpg.gw[tid]);
    }
    const double org[3] = {el.ijk[0] * kp.E[0] + el.ijk[1] * kp.E[3] + el.ijk[2] * kp.E[6],
                           el.ijk[0] * kp.E[1] + el.ijk[1] * kp.E[4] + el.ijk[2] * kp.E[7],
                           el.ijk[0] * kp.E[2] + el.ijk[1] * kp.E[5] + el.ijk[2] * kp.E[8]};
    // tile pairs (row tile, column tile) of the item, round-robin over waves
    const int npairs = it.nR * TC;
    int pr_row[4], pr_col[4];
    double4_t acc[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int pidx = wave + 4 * u;
        pr_row[u] = pidx < npairs ? 16 * (it.R0 + pidx / TC) : -1;
        pr_col[u] = pidx < npairs ? 16 * (pidx % TC) : -1;
        acc[u] = (double4_t){0.0, 0.0, 0.0, 0.0};
    }
    const int nfu = fe_units(kp.p);
    const int r16 = lane & 15, k4 = lane >> 4;
    __syncthreads();
    for (uint32_t lb = 0; lb < nli; lb += Q) {
        // ---- phase 1: geometry, enrichment functions, projector values
        const int gq = tid - (NT - Q);
        if (gq >= 0) {
            double xi[3], sw;
            item_point(kp, sLeaf, sPt, sGx, sGs, lb + gq, nli, n3, xi, &sw);
            point_geometry<Q>(kp, org, xi, sw, sGeo + gq);
        }
        for (int idx = tid; idx < ngrp * Q; idx += NT) {
            const int g = idx / Q, q = idx - g * Q;
            const GroupDev &G = sG[g];
            double xi[3], sw, x[3];
            item_point(kp, sLeaf, sPt, sGx, sGs, lb + q, nli, n3, xi, &sw);
            point_position(kp, org, xi, x);
            group_eval_upto<LMAX, Q>(G, sImg, kp.spl, kp.wimg ? kp.wimg + img0 : nullptr, x,
                                     sPsi + (size_t)G.fbase * 4 * Q + q);
        }
        for (int idx = tid; idx < npg * Q; idx += NT) {
            const int g = idx / Q, q = idx - g * Q;
            const PGroupDev &G = sPG[g];
            double xi[3], sw, x[3];
            item_point(kp, sLeaf, sPt, sGx, sGs, lb + q, nli, n3, xi, &sw);
            point_position(kp, org, xi, x);
            const double rx = x[0] - G.c[0], ry = x[1] - G.c[1], rz = x[2] - G.c[2];
            const double s = rx * rx + ry * ry + rz * rz, rc2 = G.rc * G.rc;
            double rad = 0.0;
            if (s < rc2) {
                const double c = 1.0 - s / rc2;
                rad = sw * exp(-G.a * s) * c * c * c;
            }
            double S[7], dS[21];
            solid_harmonics(G.l, rx, ry, rz, S, dS);
            for (int m = 0; m <= 2 * G.l; ++m) sPv[(size_t)(G.col0 + m) * QU + q] = rad * S[m];
        }
        __syncthreads();
        // ---- phase 2: sqrt(w) N_a of every local function (grouped units)
        for (int idx = tid; idx < (nfu + 8) * Q; idx += NT) {
            const int u = idx / Q, q = idx - u * Q;
            auto put = [&](int a, double, double, double, double w) { sU[(size_t)a * QU + q] = w; };
            if (u >= nfu) {
                const int c = u - nfu;
                pu_unit<Q>(kp, sGeo + q, sPsi + q, sEd, c, sCS[c], sCS[c + 1], nfe, put);
            } else {
                fe_unit_any<Q>(kp, sGeo + q, u, put);
            }
        }
        __syncthreads();
        // ---- phase 3: F[a][c] += sum_q U[a][q] P[c][q], 4 points per MFMA
#pragma unroll
        for (int s4 = 0; s4 < Q / 4; ++s4) {
            const int o = 4 * s4 + k4;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (pr_row[u] < 0) continue;
                const double a = sU[(size_t)(pr_row[u] + r16) * QU + o];
                const double b = sPv[(size_t)(pr_col[u] + r16) * QU + o];
                acc[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc[u], 0, 0, 0);
            }
        }
        __syncthreads();
    }
    // slot of this K-chunk: F[col][npad], FP64 16x16x4 accumulator layout:
    // register r of lane l is row (l / 16) + 4 r, column l % 16
    double *dst = Fp + el.pf_base + (int64_t)it.chunk * ncp * npad;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        if (pr_row[u] < 0) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            dst[(size_t)(pr_col[u] + r16) * npad + pr_row[u] + k4 + 4 * r] = acc[u][r];
    }
}

// Projector coefficients in moment form (tensor-product elements): an enriched
// row is M_c Psi_f, so its eight corners share the sums of Psi_f v_c over M_0
// and M_1 along each direction, and a classical row is a product of three
// Lagrange factors.  The sum over a line of points runs on v_mfma_f64_4x4x4
// (functions x projector values at 4 points), those over lines and planes on
// the accumulators: 2 matrix operations per pair and 4 points for eight rows,
// where nl_f_kernel evaluates every row at every point.  What is left to bound
// it is the evaluation of the functions.  Measured on 512 elements of one and
// two row tiles with 20 projector functions: 590 us there, 111 us here.
// An item's tasks R0 .. R0 + nR - 1 (quads of tile pairs, then groups of four
// projector tiles for the classical rows), at most four per wave; stages are
// planes of a leaf.
// 1D tables of a leaf, with the rule's weights: hats and Lagrange factors, z
// with the leaf's volume factor too.
struct NlTab {
    int h, l, size;   // h + (2 d + c) n, l + (3 d + i) n
    __host__ __device__ explicit NlTab(int n) : h(0), l(6 * n), size(15 * n) {}
};

__host__ __device__ inline int nl_stride(int points) { return ((points + 15) / 16) * 16 + 4; }

struct NlMomLds {
    static __host__ __device__ size_t bytes(int nfun, int ncol, int nimg, int n, int planes) {
        return sizeof(double) * ((size_t)(nfun + ncol) * nl_stride(planes * n * n) + NlTab(n).size + 2 * kMaxGauss +
                                 3 * (size_t)nimg) +
               sizeof(GroupDev) * kMaxGroups + sizeof(PGroupDev) * kMaxPGroups + sizeof(int16_t) * 8 * kMaxFun + 64;
    }
};

template <int L>
__device__ __forceinline__ void nl_group_value(const GroupDev &G, const double *__restrict__ img,
                                               const double *__restrict__ spl, const double *__restrict__ wimg,
                                               const double *x, double *o, int stride) {
    constexpr int NM = 2 * L + 1;
    const double rc2 = G.rc * G.rc, inv_rc2 = 1.0 / rc2;
    const double *c0 = img + 3 * G.img_off;
    double v[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m) v[m] = 0.0;
    for (int k = 0; k < G.nimg; ++k) {
        const double rx = x[0] - c0[3 * k], ry = x[1] - c0[3 * k + 1], rz = x[2] - c0[3 * k + 2];
        const double s = rx * rx + ry * ry + rz * rz;
        if (s >= rc2) continue;
        double g0, g1, g2;
        if (G.nspl > 0) {
            spline_radial<false>(G, spl, s, g0, g1, g2);
        } else {
            const double c = 1.0 - s * inv_rc2, c2 = c * c;
            g0 = exp(-G.a * s) * c2 * c;
        }
        if (wimg) g0 *= wimg[G.img_off + k];
        double S[7], dS[21];
        solid_harmonics(L, rx, ry, rz, S, dS);
#pragma unroll
        for (int m = 0; m < NM; ++m) v[m] += g0 * S[m];
    }
#pragma unroll
    for (int m = 0; m < NM; ++m) o[m * stride] = v[m];
}

template <int L>
__device__ __forceinline__ void nl_projector_value(const PGroupDev &G, const double *x, double *o, int stride) {
    const double rx = x[0] - G.c[0], ry = x[1] - G.c[1], rz = x[2] - G.c[2];
    const double s = rx * rx + ry * ry + rz * rz, rc2 = G.rc * G.rc;
    double rad = 0.0;
    if (s < rc2) {
        const double c = 1.0 - s / rc2;
        rad = exp(-G.a * s) * c * c * c;
    }
    double S[7], dS[21];
    solid_harmonics(L, rx, ry, rz, S, dS);
#pragma unroll
    for (int m = 0; m <= 2 * L; ++m) o[m * stride] = rad * S[m];
}

template <int P>
__global__ __launch_bounds__(kNlThreads) void nl_moment_kernel(
    const KParams kp, const NlItemDev *__restrict__ items, const ElemDev *__restrict__ elems,
    const GroupDev *__restrict__ groups, const double *__restrict__ img, const int32_t *__restrict__ edof,
    const uint32_t *__restrict__ leaves, const PGroupDev *__restrict__ pgroups, int planes, double *__restrict__ Fp) {
    constexpr int NT = kNlThreads, NU = kNlMomentTasks / 4, KS = kMaxGauss / 4, NA = P + 1;
    extern __shared__ __attribute__((aligned(16))) double smem[];
    const NlItemDev it = items[blockIdx.x];
    const ElemDev &el = elems[it.elem];
    const int n = kp.n, n2 = n * n, nfun = el.nfun, ncol = el.ncol, ngrp = el.ngrp, npg = el.npg, nfe = el.nfe;
    const int img0 = ngrp > 0 ? groups[el.grp_off].img_off : 0;
    const int nimg = ngrp > 0 ? groups[el.grp_off + ngrp - 1].img_off + groups[el.grp_off + ngrp - 1].nimg - img0 : 0;
    const int RS = nl_stride(planes * n2);
    const NlTab tb(n);
    double *sR = smem;                       // [nfun + ncol][RS]
    double *sT = sR + (nfun + ncol) * RS, *sGx = sT + tb.size, *sGw = sGx + kMaxGauss, *sImg = sGw + kMaxGauss;
    GroupDev *sG = (GroupDev *)(sImg + 3 * nimg);
    PGroupDev *sPG = (PGroupDev *)(sG + kMaxGroups);
    int16_t *sPos = (int16_t *)(sPG + kMaxPGroups);   // local index of (corner, function)
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (int g = tid; g < ngrp; g += NT) {
        GroupDev G = groups[el.grp_off + g];
        G.img_off -= img0;
        sG[g] = G;
    }
    for (int g = tid; g < npg; g += NT) sPG[g] = pgroups[el.pg_off + g];
    for (int k = tid; k < 3 * nimg; k += NT) sImg[k] = img[3 * (size_t)img0 + k];
    for (int k = tid; k < 8 * kMaxFun; k += NT) sPos[k] = -1;
    if (tid < n) {
        sGx[tid] = kp.gx[tid];
        sGw[tid] = kp.gw[tid];
    }
    double org[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) org[c] = el.ijk[0] * kp.E[c] + el.ijk[1] * kp.E[3 + c] + el.ijk[2] * kp.E[6 + c];
    __syncthreads();
    for (int k = tid; k < el.nloc - nfe; k += NT) {
        const int pk = edof[el.edof_off + k];
        sPos[(pk & 7) * kMaxFun + ((pk >> 3) & 255)] = (int16_t)k;
    }
    const int nt = (nfun + 3) / 4, ntc = (ncol + 3) / 4, npairs = nt * ntc, nquad = (npairs + 3) / 4;
    const int blk = (lane >> 2) & 3, i4 = lane & 3, k4 = lane >> 4;
    int ra[NU], rb[NU];   // this lane's rows of the table; the classical tasks have none on the left
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        const int t = it.R0 + wave + 4 * u;
        const int pr = min(4 * t + blk, max(npairs - 1, 0)), I = ntc > 0 ? pr / ntc : 0, J = pr - I * ntc;
        ra[u] = min(4 * I + i4, max(nfun - 1, 0)) * RS;
        const int col = t < nquad ? 4 * J + i4 : 4 * (4 * (t - nquad) + blk) + i4;
        rb[u] = (nfun + min(col, ncol - 1)) * RS;
    }
    double Z[NU][9];
#pragma unroll
    for (int u = 0; u < NU; ++u)
#pragma unroll
        for (int k = 0; k < 9; ++k) Z[u][k] = 0.0;
    const int spl = (n + planes - 1) / planes, nst = (int)(it.leaf_e - it.leaf_b) * spl, steps = (n + 3) / 4;
#pragma unroll 1
    for (int st = 0; st < nst; ++st) {
        const int lf = st / spl, ss = st - lf * spl, z0 = ss * planes, npl = min(planes, n - z0), npts = npl * n2;
        const uint32_t code = leaves[it.leaf_b + lf];
        const double h = 1.0 / (double)(1u << (code >> 27));
        const double c0 = 2.0 * (code & 511u) + 1.0, c1 = 2.0 * ((code >> 9) & 511u) + 1.0,
                     c2 = 2.0 * ((code >> 18) & 511u) + 1.0;
        if (ss == 0)
            for (int e = tid; e < tb.size; e += NT) {
                const bool hat = e < tb.l;
                const int j = hat ? e : e - tb.l, r = j / n, i = j - r * n, d = hat ? r >> 1 : r / 3;
                const int c = hat ? r & 1 : r - 3 * d;
                const double t = -1.0 + ((d == 0 ? c0 : (d == 1 ? c1 : c2)) + sGx[i]) * h;
                double v = c ? 0.5 * (1.0 + t) : 0.5 * (1.0 - t);
                if (!hat) {
                    double L[3] = {0.0, 0.0, 0.0}, D[3];
                    lagrange_1d(P, t, L, D);
                    v = c == 0 ? L[0] : (c == 1 ? L[1] : L[2]);
                }
                sT[e] = v * sGw[i] * (d == 2 ? h * h * h * kp.jac : 1.0);
            }
        for (int u = tid; u < (ngrp + npg) * npts; u += NT) {
            const int g = u / npts, q = u - g * npts, z = q / n2, yx = q - z * n2, y = yx / n;
            const double xi[3] = {-1.0 + (c0 + sGx[yx - y * n]) * h, -1.0 + (c1 + sGx[y]) * h, -1.0 + (c2 + sGx[z0 + z]) * h};
            double x[3];
#pragma unroll
            for (int c = 0; c < 3; ++c)
                x[c] = org[c] + 0.5 * (xi[0] + 1.0) * kp.E[c] + 0.5 * (xi[1] + 1.0) * kp.E[3 + c] +
                       0.5 * (xi[2] + 1.0) * kp.E[6 + c];
            if (g < ngrp) {
                const GroupDev &G = sG[g];
                double *o = sR + G.fbase * RS + q;
                const double *wi = kp.wimg ? kp.wimg + img0 : nullptr;
                switch (G.l) {
                    case 0: nl_group_value<0>(G, sImg, kp.spl, wi, x, o, RS); break;
                    case 1: nl_group_value<1>(G, sImg, kp.spl, wi, x, o, RS); break;
                    case 2: nl_group_value<2>(G, sImg, kp.spl, wi, x, o, RS); break;
                    default: nl_group_value<3>(G, sImg, kp.spl, wi, x, o, RS); break;
                }
            } else {
                const PGroupDev &G = sPG[g - ngrp];
                double *o = sR + (nfun + G.col0) * RS + q;
                switch (G.l) {
                    case 0: nl_projector_value<0>(G, x, o, RS); break;
                    case 1: nl_projector_value<1>(G, x, o, RS); break;
                    case 2: nl_projector_value<2>(G, x, o, RS); break;
                    default: nl_projector_value<3>(G, x, o, RS); break;
                }
            }
        }
        __syncthreads();
        // this lane's x weights: hats on the right, a Lagrange factor on the left
        int xo[KS];
        double w0[KS], w1[KS], wl[KS];
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int x = 4 * s + k4;
            xo[s] = min(x, n - 1);
            w0[s] = x < n ? sT[tb.h + x] : 0.0;
            w1[s] = x < n ? sT[tb.h + n + x] : 0.0;
            wl[s] = x < n && i4 < NA ? sT[tb.l + i4 * n + x] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int t = wave + 4 * u;
            if (t >= it.nR) continue;
            const bool quad = it.R0 + t < nquad;
#pragma unroll 1
            for (int z = 0; z < npl; ++z) {
                double Y[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
                for (int y = 0; y < n; ++y) {
                    const int o = (z * n + y) * n;
                    double t0 = 0.0, t1 = 0.0;
#pragma unroll
                    for (int s = 0; s < KS; ++s) {
                        if (s >= steps) continue;
                        const double b = sR[rb[u] + o + xo[s]];
                        if (quad) {
                            const double a = sR[ra[u] + o + xo[s]];
                            t0 = __builtin_amdgcn_mfma_f64_4x4x4f64(a, b * w0[s], t0, 0, 0, 0);
                            t1 = __builtin_amdgcn_mfma_f64_4x4x4f64(a, b * w1[s], t1, 0, 0, 0);
                        } else {
                            t0 = __builtin_amdgcn_mfma_f64_4x4x4f64(wl[s], b, t0, 0, 0, 0);
                        }
                    }
                    if (quad) {
                        const double y0 = sT[tb.h + 2 * n + y], y1 = sT[tb.h + 3 * n + y];
                        Y[0] += y0 * t0;
                        Y[1] += y0 * t1;
                        Y[2] += y1 * t0;
                        Y[3] += y1 * t1;
                    } else {
#pragma unroll
                        for (int i = 0; i < NA; ++i) Y[i] += sT[tb.l + (3 + i) * n + y] * t0;
                    }
                }
                if (quad) {
                    const double q0 = sT[tb.h + 4 * n + z0 + z], q1 = sT[tb.h + 5 * n + z0 + z];
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        Z[u][k] += q0 * Y[k];
                        Z[u][4 + k] += q1 * Y[k];
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < NA; ++i) {
                        const double q = sT[tb.l + (6 + i) * n + z0 + z];
#pragma unroll
                        for (int k = 0; k < NA; ++k) Z[u][NA * i + k] += q * Y[k];
                    }
                }
            }
        }
        __syncthreads();
    }
    // slot of this K-chunk: F[col][npad]; lane l holds function l / 16, column l % 4 of its block
    const int npad = 16 * ((el.nloc + 15) / 16), ncp = 16 * ((ncol + 15) / 16);
    double *dst = Fp + el.pf_base + (int64_t)it.chunk * ncp * npad;
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        const int t = it.R0 + wave + 4 * u;
        if (wave + 4 * u >= it.nR) continue;
        if (t < nquad) {
            const int pr = 4 * t + blk;
            if (pr >= npairs) continue;
            const int f = 4 * (pr / ntc) + k4, c = 4 * (pr % ntc) + i4;
            if (f >= nfun || c >= ncol) continue;
#pragma unroll
            for (int k = 0; k < 8; ++k) {   // Z runs over z, y, x of the corner
                const int loc = sPos[k * kMaxFun + f];
                if (loc >= 0) dst[(size_t)c * npad + nfe + loc] = Z[u][k];
            }
        } else {
            const int c = 4 * (4 * (t - nquad) + blk) + i4;
            if (c >= ncol || k4 >= NA) continue;
#pragma unroll
            for (int k = 0; k < NA * NA; ++k) dst[(size_t)c * npad + k4 + NA * k] = Z[u][k];
        }
    }
}

// Sum of the K-chunk slots of one element's projector coefficients, in chunk
// order, into the first slot.
__global__ __launch_bounds__(256) void nl_reduce_kernel(const ElemDev *__restrict__ elems,
                                                        const int32_t *__restrict__ nl_elems,
                                                        double *__restrict__ Fp) {
    const ElemDev &el = elems[nl_elems[blockIdx.x]];
    const int npad = 16 * ((el.nloc + 15) / 16), ncp = 16 * ((el.ncol + 15) / 16);
    const int64_t slot = (int64_t)ncp * npad;
    double *F = Fp + el.pf_base;
    for (int64_t k = threadIdx.x; k < slot; k += blockDim.x) {
        double s = 0.0;
        for (int c = 0; c < el.pf_nchunk; ++c) s += F[c * slot + k];
        F[k] = s;
    }
}

// f_J^i for the k-points of kps: one thread per (J, DOF i); the DOF's
// (element, local function) pairs in element order, each element's
// projector images of J in group order.  bpart (Bloch-periodic enrichment,
// one k-point; null otherwise): the partner table of the enriched rows, -1
// marking an imaginary part, which enters conj(phi) with the factor -i.
__global__ __launch_bounds__(256) void nl_gather_kernel(const KParams kp, const ElemDev *__restrict__ elems,
                                                        const PGroupDev *__restrict__ pgroups,
                                                        const int32_t *__restrict__ edof,
                                                        const int32_t *__restrict__ bpart,
                                                        const int64_t *__restrict__ dof_el_off,
                                                        const int2 *__restrict__ dof_el,
                                                        const double *__restrict__ Fp, const KPoints kps,
                                                        int n_pfun, int64_t n_dof, double2 *__restrict__ f) {
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (int64_t)n_pfun * n_dof) return;
    const int J = (int)(idx / n_dof);
    const int64_t i = idx - (int64_t)J * n_dof;
    double2 acc[kMaxKPerLaunch];
    for (int k = 0; k < kps.nk; ++k) acc[k] = make_double2(0.0, 0.0);
    for (int64_t t = dof_el_off[i]; t < dof_el_off[i + 1]; ++t) {
        const int2 ea = dof_el[t];
        const ElemDev &el = elems[ea.x];
        if (el.npg == 0) continue;
        const int npad = 16 * ((el.nloc + 15) / 16);
        int corner, slot;
        local_slot(el, edof, kp.p, ea.y, &corner, &slot);
        const bool enr = ea.y >= el.nfe;
        // Bloch-periodic enrichment: periodic PU (no boundary phase on the
        // enriched rows), imaginary parts with the factor -i
        const bool imag = bpart && enr && bpart[el.edof_off + (ea.y - el.nfe)] < 0;
        const int sh_on = (bpart && enr) ? 0 : 1;
        const double *F = Fp + el.pf_base;
        for (int g = 0; g < el.npg; ++g) {
            const PGroupDev &G = pgroups[el.pg_off + g];
            const int m = J - G.J0;
            if (m < 0 || m > 2 * G.l) continue;
            const double val = F[(size_t)(G.col0 + m) * npad + ea.y];
            for (int k = 0; k < kps.nk; ++k) {
                // conj(p_a) exp(2 pi i kappa . n): phase of kappa . (n - shift_a)
                double t2 = 0.0;
                for (int d = 0; d < 3; ++d)
                    t2 += kps.kap[k][d] * (double)(G.n[d] - sh_on * ((el.shifts >> (3 * corner + d)) & 1));
                double sn, cs;
                sincos(2.0 * M_PI * t2, &sn, &cs);
                if (imag) {   // (cs + i sn)(-i val)
                    acc[k].x += sn * val;
                    acc[k].y -= cs * val;
                } else {
                    acc[k].x += cs * val;
                    acc[k].y += sn * val;
                }
            }
        }
    }
    for (int k = 0; k < kps.nk; ++k) f[((int64_t)k * n_pfun + J) * n_dof + i] = acc[k];
}

size_t nl_lds_bytes(int npad, int ncol, int nfun, int nimg, int nleaf, int n3) {
    return NlLds::bytes(npad, 16 * ((ncol + 15) / 16), nfun, nimg, nleaf, n3);
}

hipError_t init_nonlocal_attributes() {
    const void *ks[4] = {(const void *)nl_f_kernel<1>, (const void *)nl_f_kernel<3>, (const void *)nl_moment_kernel<1>,
                         (const void *)nl_moment_kernel<2>};
    for (const void *k : ks) {
        const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxDynLds);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

int nl_moment_planes(int n) {
    // stages of up to 128 points: two to five work groups on a compute unit
    return std::max(1, std::min(n, 128 / (n * n)));
}

size_t nl_moment_lds(int nfun, int ncol, int nimg, int n, int planes) { return NlMomLds::bytes(nfun, ncol, nimg, n, planes); }

hipError_t launch_nl_moments(const KParams &kp, int n_items, const NlItemDev *items, const ElemDev *elems,
                             const GroupDev *groups, const double *img, const int32_t *edof, const uint32_t *leaves,
                             const PGroupDev *pgroups, int planes, double *Fp, size_t lds, hipStream_t st) {
    if (n_items == 0) return hipSuccess;
    auto *k = kp.p == 2 ? nl_moment_kernel<2> : nl_moment_kernel<1>;
    k<<<n_items, kNlThreads, lds, st>>>(kp, items, elems, groups, img, edof, leaves, pgroups, planes, Fp);
    return hipGetLastError();
}

hipError_t launch_nl_f(int lmax, const KParams &kp, int n_items, const NlItemDev *items, const ElemDev *elems,
                       const GroupDev *groups, const double *img, const int32_t *edof, const uint32_t *leaves,
                       const PGroupDev *pgroups, double *Fp, size_t lds, hipStream_t st) {
    if (n_items == 0) return hipSuccess;
    if (lmax <= 1)
        hipLaunchKernelGGL((nl_f_kernel<1>), dim3(n_items), dim3(kNlThreads), lds, st, kp, items, elems, groups, img,
                           edof, leaves, pgroups, Fp);
    else
        hipLaunchKernelGGL((nl_f_kernel<3>), dim3(n_items), dim3(kNlThreads), lds, st, kp, items, elems, groups, img,
                           edof, leaves, pgroups, Fp);
    return hipGetLastError();
}

hipError_t launch_nl_reduce(const ElemDev *elems, const int32_t *nl_elems, int n, double *Fp, hipStream_t st) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(nl_reduce_kernel, dim3(n), dim3(256), 0, st, elems, nl_elems, Fp);
    return hipGetLastError();
}

hipError_t launch_nl_gather(const KParams &kp, const ElemDev *elems, const PGroupDev *pgroups, const int32_t *edof,
                            const int32_t *bpart, const int64_t *dof_el_off, const int2 *dof_el, const double *Fp,
                            const KPoints &kps, int n_pfun, int64_t n_dof, double2 *f, hipStream_t st) {
    const int64_t n = (int64_t)n_pfun * n_dof;
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(nl_gather_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, kp, elems, pgroups, edof,
                       bpart, dof_el_off, dof_el, Fp, kps, n_pfun, n_dof, f);
    return hipGetLastError();
}

}  // namespace pufe
