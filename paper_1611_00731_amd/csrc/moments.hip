// Moment form of the FP64 element contraction (gfx950).
//
// The functions of an element are the classical FE functions N_i and the
// products M_c Psi_f of its 8 trilinear partition-of-unity functions with its
// few enrichment functions (eq. pufebasis).  Every product of two of them is a
// polynomial of low degree per direction times one of
//   1,  Psi_f,  d_d Psi_f,  Psi_f Psi_g,  Psi_g d_d Psi_f,  grad Psi_f . grad Psi_g,
// so the element matrices are linear in the moments of these against fixed
// polynomials, summed over the same quadrature points with the same weights:
//   A, E  (f <= g)  27 each: M_c M_d spans the triquadratics; A carries w,
//                   E carries grad Psi_f . grad Psi_g + 2 V Psi_f Psi_g
//   B_d   (f, g)    18 each: M_c d_d M_d is linear in direction d
//   mixed (f)       5 (p + 2)^3: w, 2 V w and the three derivatives against the
//                   degree p + 1 polynomials N_i M_c
//   classical       2 (2 p + 1)^3: w and 2 V w against the products N_i N_j
// The rule of a leaf is a tensor product, so each moment is three nested 1D
// sums.  The sum along x runs on v_mfma_f64_4x4x4 (four independent 4x4 tiles
// of function pairs; K = 4 points of a line; the x polynomial scales the
// column operand), the sums along y and z on the accumulators.  Per point and
// pair of enrichment functions this is about 31 multiply-adds on the matrix
// cores and 12 on the VALU, where the products of the element's own functions
// need 5 for each of the 64 (64/2 on the diagonal) pairs of corners: 380.
//
// The polynomials: x of A, E, B_y, B_z: 1, xi, xi^2 and of B_x: 1, xi (no
// scaling for the first); y and z: the products of the two hat functions
// m_0 m_0, m_0 m_1, m_1 m_1 (index c + d) and, along the derivative, m_0, m_1;
// mixed and classical: Lagrange polynomials on p + 2 and 2 p + 1 equidistant
// nodes, so that a moment is the weight of a node of an equivalent rule.
//
// Bound by issue on the FP64 pipes, matrix and vector in turn (they do not
// overlap on a SIMD).  Measured on 1728 elements of up to 41 functions, 27.3 M
// points: the contraction 198 ms with the products of the element's own
// functions, 40 ms here, 30 of them in work groups of eight waves (1.03e9 matrix
// operations, 7.1 ms at their rate; 7.7e9 vector instructions, about 15 ms, half
// of them the sums along y and z, a quarter the evaluation of the functions; a
// third of the cycles wait at a stage's two barriers or on LDS).  512 elements
// of up to 10 functions, 1.52 M points: 0.89 and 0.45 ms.
// Roles of at most 40 sums a lane: with the 54 of E and A in one wave the sums
// spill through the evaluation of the functions (111 ms for the 46 that the
// first form without spills took).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "basis.hpp"
#include "device_common.hpp"
#include "enrich.hpp"
#include "moment_math.hpp"
#include "moments.hpp"
#include "stage.hpp"
#include "tables.hpp"

namespace pufe {

namespace {

// 1D tables of one leaf, doubles: x coordinate [n]; y and z polynomials
// [n][5] (m0 m0, m0 m1, m1 m1, m0, m1); mixed x, y, z [n][p + 2] times the
// square root of the 1D weight (z also carries the leaf's volume factor).
struct MomTab {
    int yt, zt, fx, fy, fz, size;
    __host__ __device__ MomTab(int n, int p) {
        const int nf = p + 2;
        yt = n;
        zt = yt + 5 * n;
        fx = zt + 5 * n;
        fy = fx + nf * n;
        fz = fy + nf * n;
        size = fz + nf * n;
    }
};

// Points of a row of the enrichment table with the three past the end that the
// last operand read of a line may touch (never written, so zero), and its
// stride in doubles: value and gradient of a point are neighbours, and the
// stride is odd in 16-byte units, so that the eight rows of a 128-bit read
// phase start at distinct banks.  Other accesses still conflict: 2.06e9 cycles a
// launch of the eight-wave groups on 1728 elements of up to 41 functions.
__host__ __device__ inline int mom_points(int points) { return points + 3; }
__host__ __device__ inline int mom_stride(int points) { return 4 * mom_points(points) + 2; }

// ---------------------------------------------------------- wave roles

// One line of an operand table: lane l supplies k = l / 16, rows by block and
// row (or column) l % 4.
struct MomLane {
    int oa, ob;      // offsets of the row and column operands at the lane's first point
    int k4;
};

// Value and gradient of one function at one point.
struct MomOp {
    dbl2 lo, hi;
    __device__ __forceinline__ void load(const double *p) {
        lo = *(const dbl2 *)p;
        hi = *(const dbl2 *)(p + 2);
    }
};

// Energy moments of one quad, with the overlap moments of x^2 (whose operands
// they share): Z[9 k + 3 ky + kz] E of x^k, Z[27 + 3 ky + kz] A of x^2.  The
// operands of a line are read while the MFMAs of the line before it run.
template <int KS, bool SKEW>
__device__ __forceinline__ void mom_e(const double *__restrict__ sP, const MomLane &ln, const double *__restrict__ T,
                                      const MomTab &mt, const double *__restrict__ sV, int n, int z0, int np,
                                      const double *__restrict__ Gi, double *Z) {
    double xi[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) xi[s] = T[min(4 * s + ln.k4, n - 1)];
    const bool cut = 4 * (KS - 1) + ln.k4 >= n, ragged = 4 * KS != n;   // ragged: uniform
    const double *pa = sP + ln.oa, *pb = sP + ln.ob, *pv = sV + ln.k4;
    MomOp A[KS], B[KS];
    double v[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        A[s].load(pa + 16 * s);
        B[s].load(pb + 16 * s);
        v[s] = pv[4 * s];
    }
    for (int pz = 0; pz < np; ++pz) {
        double Y[4][3];
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int y = 0; y < 3; ++y) Y[k][y] = 0.0;
        const double *ty = T + mt.yt;
#pragma unroll 1
        for (int y = 0; y < n; ++y) {
            // the last line of the stage is read again in place of a next one
            const int step = pz + 1 < np || y + 1 < n ? n : 0;
            pa += 4 * step;
            pb += 4 * step;
            pv += step;
            double X[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                double a[4] = {A[s].lo[0], A[s].lo[1], A[s].hi[0], A[s].hi[1]};
                double b[4] = {B[s].lo[0], B[s].lo[1], B[s].hi[0], B[s].hi[1]};
                if (s == KS - 1 && ragged) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) a[c] = cut ? 0.0 : a[c];
                }
                const double av = a[0] * v[s];
                A[s].load(pa + 16 * s);
                B[s].load(pb + 16 * s);
                v[s] = pv[4 * s];
                if (SKEW) {
                    const double g0 = b[1], g1 = b[2], g2 = b[3];
#pragma unroll
                    for (int d = 0; d < 3; ++d) b[1 + d] = Gi[3 * d] * g0 + Gi[3 * d + 1] * g1 + Gi[3 * d + 2] * g2;
                }
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    if (k > 0) {
#pragma unroll
                        for (int c = 0; c < 4; ++c) b[c] *= xi[s];
                    }
                    X[k] = mfma4(av, b[0], X[k]);
                    if (k == 2) X[3] = mfma4(a[0], b[0], X[3]);
#pragma unroll
                    for (int d = 0; d < 3; ++d) X[k] = mfma4(a[1 + d], b[1 + d], X[k]);
                }
            }
            const double w0 = ty[0], w1 = ty[1], w2 = ty[2];
            ty += 5;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                Y[k][0] += w0 * X[k];
                Y[k][1] += w1 * X[k];
                Y[k][2] += w2 * X[k];
            }
        }
        const double *tz = T + mt.zt + 5 * (z0 + pz);
        const double w[3] = {tz[0], tz[1], tz[2]};
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int y = 0; y < 3; ++y)
#pragma unroll
                for (int z = 0; z < 3; ++z) Z[9 * k + 3 * y + z] += w[z] * Y[k][y];
    }
}

// Overlap moments of x^0 and x^1 of one quad: Z[9 k + 3 ky + kz].
template <int KS>
__device__ __forceinline__ void mom_a(const double *__restrict__ sP, const MomLane &ln, const double *__restrict__ T,
                                      const MomTab &mt, int n, int z0, int np, double *Z) {
    double xi[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) xi[s] = T[min(4 * s + ln.k4, n - 1)];
    const bool cut = 4 * (KS - 1) + ln.k4 >= n, ragged = 4 * KS != n;   // ragged: uniform
    const double *pa = sP + ln.oa, *pb = sP + ln.ob;
    double a[KS], b[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        a[s] = pa[16 * s];
        b[s] = pb[16 * s];
    }
    for (int pz = 0; pz < np; ++pz) {
        double Y[2][3] = {{0.0, 0.0, 0.0}, {0.0, 0.0, 0.0}};
        const double *ty = T + mt.yt;
#pragma unroll 1
        for (int y = 0; y < n; ++y) {
            const int step = pz + 1 < np || y + 1 < n ? n : 0;
            pa += 4 * step;
            pb += 4 * step;
            double X[2] = {0.0, 0.0};
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const double a0 = a[s];
                double b0 = b[s];
                if (s == KS - 1 && ragged) b0 = cut ? 0.0 : b0;
                a[s] = pa[16 * s];
                b[s] = pb[16 * s];
                X[0] = mfma4(a0, b0, X[0]);
                X[1] = mfma4(a0, b0 * xi[s], X[1]);
            }
            const double w0 = ty[0], w1 = ty[1], w2 = ty[2];
            ty += 5;
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                Y[k][0] += w0 * X[k];
                Y[k][1] += w1 * X[k];
                Y[k][2] += w2 * X[k];
            }
        }
        const double *tz = T + mt.zt + 5 * (z0 + pz);
        const double w[3] = {tz[0], tz[1], tz[2]};
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int y = 0; y < 3; ++y)
#pragma unroll
                for (int z = 0; z < 3; ++z) Z[9 * k + 3 * y + z] += w[z] * Y[k][y];
    }
}

// Derivative moments B_d(f, g) = sum w P D_d Psi_f Psi_g of one quad: with XY
// Z[9 kx + 3 ky + kz] (B_x) and Z[18 + 6 kx + 3 ky + kz] (B_y), else
// Z[6 kx + 2 ky + kz] (B_z).
template <int KS, bool XY>
__device__ __forceinline__ void mom_b(const double *__restrict__ sP, const MomLane &ln, const double *__restrict__ T,
                                      const MomTab &mt, int n, int z0, int np, double *Z) {
    double xi[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) xi[s] = T[min(4 * s + ln.k4, n - 1)];
    const bool cut = 4 * (KS - 1) + ln.k4 >= n, ragged = 4 * KS != n;   // ragged: uniform
    const double *pa = sP + ln.oa + (XY ? 1 : 3), *pb = sP + ln.ob;
    double a0[KS], a1[KS], b[KS];   // d_x (or d_z) and d_y of the row function, the column function
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        a0[s] = pa[16 * s];
        a1[s] = XY ? pa[16 * s + 1] : 0.0;
        b[s] = pb[16 * s];
    }
    for (int pz = 0; pz < np; ++pz) {
        double Yx[2][3], Yy[3][2], Yz[3][3];
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                if (i < 2) Yx[i][j] = 0.0;
                if (j < 2) Yy[i][j] = 0.0;
                Yz[i][j] = 0.0;
            }
        const double *ty = T + mt.yt;
#pragma unroll 1
        for (int y = 0; y < n; ++y) {
            const int step = pz + 1 < np || y + 1 < n ? n : 0;
            pa += 4 * step;
            pb += 4 * step;
            double Xx[2] = {0.0, 0.0}, X[3] = {0.0, 0.0, 0.0};   // X: B_y or B_z
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const double c0 = a0[s], c1 = a1[s];
                double b0 = b[s];
                if (s == KS - 1 && ragged) b0 = cut ? 0.0 : b0;
                a0[s] = pa[16 * s];
                if (XY) a1[s] = pa[16 * s + 1];
                b[s] = pb[16 * s];
                const double b1 = b0 * xi[s], b2 = b1 * xi[s];
                if (XY) {
                    Xx[0] = mfma4(c0, b0, Xx[0]);
                    X[0] = mfma4(c1, b0, X[0]);
                    Xx[1] = mfma4(c0, b1, Xx[1]);
                    X[1] = mfma4(c1, b1, X[1]);
                    X[2] = mfma4(c1, b2, X[2]);
                } else {
                    X[0] = mfma4(c0, b0, X[0]);
                    X[1] = mfma4(c0, b1, X[1]);
                    X[2] = mfma4(c0, b2, X[2]);
                }
            }
            const double w0 = ty[0], w1 = ty[1], w2 = ty[2], l0 = ty[3], l1 = ty[4];
            ty += 5;
            if (XY) {
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    Yx[k][0] += w0 * Xx[k];
                    Yx[k][1] += w1 * Xx[k];
                    Yx[k][2] += w2 * Xx[k];
                }
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    Yy[k][0] += l0 * X[k];
                    Yy[k][1] += l1 * X[k];
                }
            } else {
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    Yz[k][0] += w0 * X[k];
                    Yz[k][1] += w1 * X[k];
                    Yz[k][2] += w2 * X[k];
                }
            }
        }
        const double *tz = T + mt.zt + 5 * (z0 + pz);
        const double w[3] = {tz[0], tz[1], tz[2]}, l[2] = {tz[3], tz[4]};
        if (XY) {
#pragma unroll
            for (int z = 0; z < 3; ++z) {
#pragma unroll
                for (int k = 0; k < 2; ++k)
#pragma unroll
                    for (int y = 0; y < 3; ++y) Z[9 * k + 3 * y + z] += w[z] * Yx[k][y];
#pragma unroll
                for (int k = 0; k < 3; ++k)
#pragma unroll
                    for (int y = 0; y < 2; ++y) Z[18 + 6 * k + 3 * y + z] += w[z] * Yy[k][y];
            }
        } else {
#pragma unroll
            for (int z = 0; z < 2; ++z)
#pragma unroll
                for (int k = 0; k < 3; ++k)
#pragma unroll
                    for (int y = 0; y < 3; ++y) Z[6 * k + 2 * y + z] += l[z] * Yz[k][y];
        }
    }
}

// Mixed moments of two row tiles (8 enrichment functions): rows are functions,
// the 16 columns of an MFMA the (kx, ky) products of the plane polynomials, K
// the points of a plane.  Z[(5 r + c) NF + kz], c = 0: w, 1: 2 V w, 2..4: the
// derivatives.
template <int NF>
__device__ __forceinline__ void mom_f(const double *__restrict__ sP, int o0, int o1, int col, int k4,
                                      const double *__restrict__ T, const MomTab &mt, const double *__restrict__ sV,
                                      const uint32_t *__restrict__ sPt, int n, int z0, int np, double *Z) {
    const bool live = col < NF * NF;
    const int kx = live ? col % NF : 0, ky = live ? col / NF : 0, n2 = n * n;
    const double *tx = T + mt.fx + kx, *ty = T + mt.fy + ky;
    for (int pz = 0; pz < np; ++pz) {
        double X[2][5];
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int c = 0; c < 5; ++c) X[r][c] = 0.0;
#pragma unroll 2
        for (int s = 0; s < n2; s += 4) {
            const int q = min(s + k4, n2 - 1);
            const uint32_t pt = sPt[q];
            double b = tx[(int)(pt & 255u) * NF] * ty[(int)((pt >> 8) & 255u) * NF];
            b = s + k4 < n2 ? b : 0.0;
            const int o = pz * n2 + q;
            const double v2 = sV[o];
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                MomOp A;
                A.load(sP + (r ? o1 : o0) + 4 * o);
                X[r][0] = mfma4(A.lo[0], b, X[r][0]);
                X[r][1] = mfma4(A.lo[0] * v2, b, X[r][1]);
                X[r][2] = mfma4(A.lo[1], b, X[r][2]);
                X[r][3] = mfma4(A.hi[0], b, X[r][3]);
                X[r][4] = mfma4(A.hi[1], b, X[r][4]);
            }
        }
        const double *tz = T + mt.fz + (z0 + pz) * NF;
#pragma unroll
        for (int z = 0; z < NF; ++z) {
            const double w = tz[z];
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int c = 0; c < 5; ++c) Z[(5 * r + c) * NF + z] += w * X[r][c];
        }
    }
}

// Enrichment functions of one group at one point, times sw, with gradients
// (skewed cells: Jt^T grad, so that a reference derivative d_d of a polynomial
// meets component d): function m, component c at o[m MS + c].  The sums over
// images accumulate in place.
template <int L, bool TAB>
__device__ __forceinline__ void mom_group(const GroupDev &G, const double *__restrict__ img,
                                          const double *__restrict__ spl, const double *__restrict__ wimg,
                                          const double *x, double sw, bool skew, const double *__restrict__ Jt,
                                          double *o, int MS) {
    constexpr int NM = 2 * L + 1;
    const double rc2 = G.rc * G.rc, inv_rc2 = 1.0 / rc2;
    const double *c0 = img + 3 * G.img_off;
    bool first = true;
    for (int k = 0; k < G.nimg; ++k) {
        const double rx = x[0] - c0[3 * k], ry = x[1] - c0[3 * k + 1], rz = x[2] - c0[3 * k + 2];
        const double s = rx * rx + ry * ry + rz * rz;
        if (s >= rc2) continue;
        double g0, g1;
        if (TAB && G.nspl > 0) {
            double unused;
            spline_radial<false>(G, spl, s, g0, g1, unused);
            g0 *= sw;
            g1 *= sw;
        } else {
            const double ex = sw * exp(-G.a * s), c = 1.0 - s * inv_rc2, c2 = c * c;
            g0 = ex * c2 * c;
            g1 = -ex * c2 * (G.a * c + 3.0 * inv_rc2);
        }
        if (TAB && wimg) {
            const double wk = wimg[G.img_off + k];
            g0 *= wk;
            g1 *= wk;
        }
        double S[7], dS[21];
        solid_harmonics(L, rx, ry, rz, S, dS);
        const double tx = 2.0 * g1 * rx, ty = 2.0 * g1 * ry, tz = 2.0 * g1 * rz;
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            double *om = o + m * MS;
            double v[4] = {g0 * S[m], tx * S[m] + g0 * dS[3 * m], ty * S[m] + g0 * dS[3 * m + 1],
                           tz * S[m] + g0 * dS[3 * m + 2]};
            if (skew) {
                const double u0 = v[1], u1 = v[2], u2 = v[3];
#pragma unroll
                for (int d = 0; d < 3; ++d) v[1 + d] = Jt[d] * u0 + Jt[3 + d] * u1 + Jt[6 + d] * u2;
            }
            dbl2 *ov = (dbl2 *)om;
            const dbl2 lo = {v[0], v[1]}, hi = {v[2], v[3]};
            if (first) {
                ov[0] = lo;
                ov[1] = hi;
            } else {
                ov[0] += lo;
                ov[1] += hi;
            }
            // one function at a time: with all 2 L + 1 read-modify-writes in
            // flight the moment sums of the wave would spill
            __builtin_amdgcn_sched_barrier(0);
        }
        first = false;
    }
    if (first)
#pragma unroll
        for (int m = 0; m < NM; ++m)
#pragma unroll
            for (int c = 0; c < 4; ++c) o[m * MS + c] = 0.0;
}

}  // namespace

// LDS map: nbuf stages of the enrichment table [4 nt rows][points][4] and of
// 2 V, two 1D tables, Gauss rule, cell constants (E, origin, Jt, G^-1), image
// centres, groups, point digits.
constexpr int kMomConst = 30;
static size_t mom_lds_bytes(int nt, int nimg, int n, int p, int planes, int nbuf) {
    const int pts = n * n * planes;
    return sizeof(double) * ((size_t)nbuf * (4 * (size_t)nt * mom_stride(pts) + ((mom_points(pts) + 1) & ~1)) +
                             2 * (size_t)MomTab(n, p).size + 2 * kMaxGauss + kMomConst + 3 * (size_t)nimg) +
           sizeof(GroupDev) * kMaxGroups + sizeof(uint32_t) * (size_t)(n * n * planes) + 64;
}

MomStage mom_stage(int nt, int nimg, int n, int p, int nw) {
    // 4-wave work groups share a CU in pairs; the static LDS of the kernel
    // stays free
    const size_t room = nw == 4 ? (size_t)79 * 1024 : kMaxDynLds;
    MomStage s{0, 2, 0};
    for (int nbuf = 2; nbuf >= 1 && s.planes == 0; --nbuf)
        for (int groups = 1; groups <= n; ++groups) {
            const int planes = (n + groups - 1) / groups;
            if (n * n * planes > kMomMaxPoints && planes > 1) continue;
            const size_t b = mom_lds_bytes(nt, nimg, n, p, planes, nbuf);
            if (b > room) continue;
            s.planes = planes;
            s.buffers = nbuf;
            s.lds = b;
            break;
        }
    return s;
}

// One work group of NW waves per item.  Each stage (a few planes of a leaf)
// alternates two halves: the moment sums, one task per wave on the whole
// stage, and the enrichment functions of the next stage's points, one (group,
// point) pair per lane, into the other buffer (one barrier interval; two with
// a single buffer).
template <int NW, int KS, int LMAX, bool GEN, bool SKEW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2))) void moment_kernel(
    const CtxDev *__restrict__ ctxs, const MomItemDev *__restrict__ items, const int32_t *__restrict__ wave_task,
    const double *__restrict__ V1, const double *__restrict__ wimg1) {
    extern __shared__ __attribute__((aligned(16))) double smem[];
    constexpr int NT = 64 * NW;
    const MomItemDev it = items[blockIdx.x];
    const CtxDev &cx = ctxs[it.ctx];
    const KParams &kp = cx.kp;
    const PUFE_GLOBAL ElemDev &el = ((const PUFE_GLOBAL ElemDev *)cx.elems)[it.elem];
    const PUFE_GLOBAL GroupDev *gGroups = (const PUFE_GLOBAL GroupDev *)cx.groups + el.grp_off;
    const PUFE_GLOBAL double *gV = (const PUFE_GLOBAL double *)(V1 ? V1 : cx.V);
    const PUFE_GLOBAL uint32_t *gLeaves = (const PUFE_GLOBAL uint32_t *)cx.leaves;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int task = __builtin_amdgcn_readfirstlane(wave_task[(it.tab & 0xffffff) + wave]);
    const int role = task & 255, idx = (task >> 8) & 4095;
    const int n = kp.n, n2 = n * n, p = kp.p, ngrp = el.ngrp, nt = el.nt, rows = 4 * nt;
    const int img0 = ngrp > 0 ? gGroups[0].img_off : 0;
    const int nimg = ngrp > 0 ? gGroups[ngrp - 1].img_off + gGroups[ngrp - 1].nimg - img0 : 0;
    const double *wimg0 = wimg1 ? wimg1 : kp.wimg;
    const double *wimg = (GEN && wimg0) ? wimg0 + img0 : nullptr;
    const int planes = (it.tab >> 24) & 15, nbuf = (it.tab >> 28) & 3;
    const int RS = mom_stride(n2 * planes), BUF = rows * RS, VS = (mom_points(n2 * planes) + 1) & ~1;
    const MomTab mt(n, p);
    double *sP = smem;                                 // [nbuf][rows][RS]
    double *sV = sP + nbuf * BUF;                      // [nbuf][VS]
    double *sT = sV + nbuf * VS;                       // [2][mt.size]
    double *sGx = sT + 2 * mt.size, *sGw = sGx + kMaxGauss;
    // the cell's constants are read from LDS where they are used: held in
    // scalar registers over the whole loop they would not fit
    double *sE = sGw + kMaxGauss, *sOrg = sE + 9, *sJt = sOrg + 3, *sGi = sJt + 9;
    double *sImg = sGi + 9;
    GroupDev *sG = (GroupDev *)(sImg + 3 * nimg);
    uint32_t *sPt = (uint32_t *)(sG + kMaxGroups);     // x | y << 8 | z << 16 of the stage's points

    for (int k = tid; k < 3 * nimg; k += NT) sImg[k] = ((const PUFE_GLOBAL double *)cx.img)[3 * (size_t)img0 + k];
    for (int g = tid; g < ngrp; g += NT) {
        GroupDev G;
        const PUFE_GLOBAL GroupDev &Gg = gGroups[g];
        G.atom = Gg.atom;
        G.desc = Gg.desc;
        G.l = Gg.l;
        G.fbase = Gg.fbase;
        G.img_off = Gg.img_off - img0;   // rebased onto sImg
        G.nimg = Gg.nimg;
        G.nspl = Gg.nspl;
        G.spl_off = Gg.spl_off;
        G.a = Gg.a;
        G.rc = Gg.rc;
        sG[g] = G;
    }
    for (int q = tid; q < n2 * planes; q += NT) sPt[q] = (q % n) | (((q / n) % n) << 8) | ((q / n2) << 16);
    if (tid < n) {
        sGx[tid] = kp.gx[tid];
        sGw[tid] = sqrt(kp.gw[tid]);   // square roots of the 1D weights
    }
    if (tid < 9) {
        sE[tid] = kp.E[tid];
        sJt[tid] = kp.Jt[tid];
        sGi[tid] = kp.Gi[tid];
    }
    if (tid < 3) sOrg[tid] = el.ijk[0] * kp.E[tid] + el.ijk[1] * kp.E[3 + tid] + el.ijk[2] * kp.E[6 + tid];
    // rows past the element's functions and the points past a row's end stay
    // zero, and what a shorter stage leaves behind is finite
    for (int k = tid; k < nbuf * (BUF + VS); k += NT) sP[k] = 0.0;
    const bool skew = SKEW && kp.skew != 0;

    int oa = 0, ob = 0, oa2 = 0, ob2 = 0;   // operand offsets; those of the second task of a wave
    {
        const int blk = (lane >> 2) & 3, r4 = lane & 3, k = 4 * (lane >> 4);
        auto energy = [&](int q) {
            const int pr = min(4 * q + blk, nt * (nt + 1) / 2 - 1);
            int J = 0;
            while ((J + 1) * (J + 2) / 2 <= pr) ++J;
            oa = (4 * (pr - J * (J + 1) / 2) + r4) * RS + k;
            ob = (4 * J + r4) * RS + k;
        };
        auto gradient = [&](int q, int &o1, int &o2) {
            const int pr = min(4 * q + blk, nt * nt - 1), I = pr / nt;
            o1 = (4 * I + r4) * RS + k;
            o2 = (4 * (pr - I * nt) + r4) * RS + k;
        };
        if (role == MOM_E || role == MOM_A || role == MOM_A_BZ) energy(idx);
        if (role == MOM_BXY) gradient(idx, oa, ob);
        if (role == MOM_BZ || role == MOM_A_BZ) gradient(task >> 20, oa2, ob2);
        if (role == MOM_F) {
            oa = (8 * idx + r4) * RS;
            ob = (min(8 * idx + 4, rows - 4) + r4) * RS;
        }
    }
    const double sqrt_jac = sqrt(kp.jac);
    double Z[40];
#pragma unroll
    for (int i = 0; i < 40; ++i) Z[i] = 0.0;

    const int npg = (n + planes - 1) / planes;
    const int nst = (int)(it.leaf_e - it.leaf_b) * npg;
    // enrichment functions, V and (on a leaf's first stage) the 1D tables
    auto fill = [&](int st) {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        const int lf = st / npg, z0 = (st - lf * npg) * planes, npl = min(planes, n - z0), npts = n2 * npl;
        const int64_t leaf = it.leaf_b + lf;
        const uint32_t code = gLeaves[leaf];
        const int buf = nbuf == 2 ? st & 1 : 0;
        double v2 = 0.0;
        if (tid < npts) v2 = 2.0 * gV[leaf * kp.n3 + (int64_t)z0 * n2 + tid];
        const int lev = (int)(code >> 27);
        const double h = 1.0 / (double)(1u << lev);
        const double c[3] = {2.0 * (code & 511u) + 1.0, 2.0 * ((code >> 9) & 511u) + 1.0,
                             2.0 * ((code >> 18) & 511u) + 1.0};
        // square root of the leaf's volume factor, h^(3/2) = 2^(-3 lev / 2)
        const double s0 = ldexp((lev & 1) ? M_SQRT2 : 1.0, -((3 * lev + (lev & 1)) >> 1)) * sqrt_jac;
        if (z0 == 0) {
            double *T = sT + (lf & 1) * mt.size;
            const int nf = p + 2;
            for (int e = tid; e < n * (11 + 3 * nf); e += NT) {
                int j = e;
                if (j < n) {
                    T[j] = -1.0 + (c[0] + sGx[j]) * h;
                    continue;
                }
                j -= n;
                if (j < 10 * n) {
                    const int d = j < 5 * n ? 1 : 2, i = (j - 5 * n * (d - 1)) / 5, k = j % 5;
                    const double x = -1.0 + (c[d] + sGx[i]) * h, m0 = 0.5 * (1.0 - x), m1 = 0.5 * (1.0 + x);
                    T[mt.yt + j] = k == 0 ? m0 * m0 : (k == 1 ? m0 * m1 : (k == 2 ? m1 * m1 : (k == 3 ? m0 : m1)));
                    continue;
                }
                j -= 10 * n;
                const int i = nf == 4 ? j >> 2 : j / 3, k = j - i * nf, d = i < n ? 0 : (i < 2 * n ? 1 : 2);
                const double x = -1.0 + (c[d] + sGx[i - d * n]) * h, w = sGw[i - d * n] * (d == 2 ? s0 : 1.0);
                T[mt.fx + j] = (nf == 4 ? lagrange_equi<4>(k, x) : lagrange_equi<3>(k, x)) * w;
            }
        }
        const int total = ngrp * npts;
        // groups come with l ascending: the second wave of a SIMD takes them
        // from the far end
        const int turn = NW == 8 && wave >= 4 ? 11 - wave : wave;
        for (int u = 64 * turn + (tid & 63); u < total; u += NT) {
            const int g = u / npts, q = u - g * npts;
            const uint32_t pt = sPt[q];
            const int k[3] = {(int)(pt & 255u), (int)((pt >> 8) & 255u), (int)(pt >> 16) + z0};
            double xi[3], x[3];
#pragma unroll
            for (int d = 0; d < 3; ++d) xi[d] = -1.0 + (c[d] + sGx[k[d]]) * h;
#pragma unroll
            for (int cc = 0; cc < 3; ++cc)
                x[cc] = sOrg[cc] + 0.5 * (xi[0] + 1.0) * sE[cc] + 0.5 * (xi[1] + 1.0) * sE[3 + cc] +
                        0.5 * (xi[2] + 1.0) * sE[6 + cc];
            const double sw = s0 * (sGw[k[0]] * sGw[k[1]] * sGw[k[2]]);
            const GroupDev &G = sG[g];
            double *o = sP + buf * BUF + G.fbase * RS + 4 * q;
            switch (G.l) {
                case 0: mom_group<0, GEN>(G, sImg, kp.spl, wimg, x, sw, skew, sJt, o, RS); break;
                case 1: mom_group<1, GEN>(G, sImg, kp.spl, wimg, x, sw, skew, sJt, o, RS); break;
                case 2: if (LMAX >= 2) mom_group<2, GEN>(G, sImg, kp.spl, wimg, x, sw, skew, sJt, o, RS); break;
                default: if (LMAX >= 3) mom_group<3, GEN>(G, sImg, kp.spl, wimg, x, sw, skew, sJt, o, RS); break;
            }
        }
        // the host keeps a stage within kMomMaxPoints: at most two V per thread
        if (tid < npts) sV[buf * VS + tid] = v2;
        if (tid + NT < npts) sV[buf * VS + tid + NT] = 2.0 * gV[leaf * kp.n3 + (int64_t)z0 * n2 + tid + NT];
    };
    auto sums = [&](int st) {
        int lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane));
        MomLane ln{oa, ob, lane >> 4};
        const int lf = st / npg, z0 = (st - lf * npg) * planes, npl = min(planes, n - z0);
        const int buf = nbuf == 2 ? st & 1 : 0;
        const double *P = sP + buf * BUF, *v = sV + buf * VS, *T = sT + (lf & 1) * mt.size;
        switch (role) {
            case MOM_E:
                if (SKEW && skew) mom_e<KS, true>(P, ln, T, mt, v, n, z0, npl, sGi, Z);
                else mom_e<KS, false>(P, ln, T, mt, v, n, z0, npl, sGi, Z);
                break;
            case MOM_BXY: mom_b<KS, true>(P, ln, T, mt, n, z0, npl, Z); break;
            case MOM_F:
                if (p == 2) mom_f<4>(P, oa, ob, lane & 15, ln.k4, T, mt, v, sPt, n, z0, npl, Z);
                else mom_f<3>(P, oa, ob, lane & 15, ln.k4, T, mt, v, sPt, n, z0, npl, Z);
                break;
            default:
                if (role == MOM_A || role == MOM_A_BZ) mom_a<KS>(P, ln, T, mt, n, z0, npl, Z);
                if (role == MOM_BZ || role == MOM_A_BZ)
                    mom_b<KS, false>(P, MomLane{oa2, ob2, ln.k4}, T, mt, n, z0, npl, Z + 18);
                break;
        }
    };
    __syncthreads();
    if (nst > 0) fill(0);
    __syncthreads();
    // one path through both halves for one and two buffers: the moment sums then
    // keep their registers from stage to stage
#pragma unroll 1
    for (int st = 0; st < nst; ++st) {
        sums(st);
        if (nbuf == 1) __syncthreads();
        if (st + 1 < nst) fill(st + 1);
        __syncthreads();
    }
    if (role == MOM_IDLE) return;
    // slots: energy quads (A[k][9] and E[k][9] per x power k), gradient quads
    // (B_x, B_y, B_z), mixed groups
    const int qa = mom_quads_ae(nt), qb = mom_quads_b(nt), second = task >> 20;
    PUFE_GLOBAL double *dst =
        (PUFE_GLOBAL double *)cx.mom + el.mom_base + (int64_t)it.chunk * mom_slots(nt) * kMomSlot + lane;
    if (role == MOM_E) {
        PUFE_GLOBAL double *d = dst + (int64_t)idx * kMomSlot;
#pragma unroll
        for (int i = 0; i < 27; ++i) d[(18 * (i / 9) + 9 + i % 9) * 64] = Z[i];
#pragma unroll
        for (int i = 0; i < 9; ++i) d[(36 + i) * 64] = Z[27 + i];
    } else if (role == MOM_BXY) {
        PUFE_GLOBAL double *d = dst + (int64_t)(qa + idx) * kMomSlot;
#pragma unroll
        for (int i = 0; i < 36; ++i) d[i * 64] = Z[i];
    } else if (role == MOM_F) {
        PUFE_GLOBAL double *d = dst + (int64_t)(qa + qb + idx) * kMomSlot;
        const int cnt = 10 * (p + 2);
#pragma unroll
        for (int i = 0; i < 40; ++i)
            if (i < cnt) d[i * 64] = Z[i];
    }
    if (role == MOM_A || role == MOM_A_BZ) {
        PUFE_GLOBAL double *d = dst + (int64_t)idx * kMomSlot;
#pragma unroll
        for (int i = 0; i < 18; ++i) d[(18 * (i / 9) + i % 9) * 64] = Z[i];
    }
    if (role == MOM_BZ || role == MOM_A_BZ) {
        PUFE_GLOBAL double *d = dst + (int64_t)(qa + second) * kMomSlot;
#pragma unroll
        for (int i = 0; i < 18; ++i) d[(36 + i) * 64] = Z[18 + i];
    }
}

// Classical moments: one work group per (element, range of leaves), its waves
// taking the leaves in turn without barriers.  Per plane, row 0 of the row
// operand carries 1 and row 1 carries 2 V; the columns are the (kx, ky)
// products of the classical polynomials times the 1D weights, 16 per MFMA; K
// the points of the plane.  Bound by reading V and by the tables of each leaf.
template <int NG>
__device__ __forceinline__ void classical_leaves(const CtxDev &cx, const MomItemDev &it, const double *__restrict__ V,
                                                 double *__restrict__ smem) {
    constexpr int NC = (NG * NG + 15) / 16;
    const KParams &kp = cx.kp;
    const int n = kp.n, n2 = n * n, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const PUFE_GLOBAL uint32_t *gLeaves = (const PUFE_GLOBAL uint32_t *)cx.leaves;
    const PUFE_GLOBAL double *gV = (const PUFE_GLOBAL double *)V;
    double *sT = smem + wave * (3 * NG * kMaxGauss + kMaxGauss * kMaxGauss), *sV = sT + 3 * NG * kMaxGauss;
    const int k4 = lane >> 4, row = lane & 3;
    int ox[NC], oy[NC];
#pragma unroll
    for (int t = 0; t < NC; ++t) {
        const int col = 16 * t + (lane & 15), cc = col < NG * NG ? col : 0;
        ox[t] = cc % NG;
        oy[t] = NG * n + cc / NG;
    }
    double Z[NC][NG];
#pragma unroll
    for (int t = 0; t < NC; ++t)
#pragma unroll
        for (int z = 0; z < NG; ++z) Z[t][z] = 0.0;
    for (int64_t leaf = it.leaf_b + wave; leaf < it.leaf_e; leaf += 4) {
        const uint32_t code = gLeaves[leaf];
        const double h = 1.0 / (double)(1u << (code >> 27));
        const double c[3] = {2.0 * (code & 511u) + 1.0, 2.0 * ((code >> 9) & 511u) + 1.0, 2.0 * ((code >> 18) & 511u) + 1.0};
        for (int e = lane; e < 3 * NG * n; e += 64) {
            const int i = e / NG, k = e - i * NG, d = i < n ? 0 : (i < 2 * n ? 1 : 2);
            const double x = -1.0 + (c[d] + kp.gx[i - d * n]) * h;
            sT[e] = lagrange_equi<NG>(k, x) * kp.gw[i - d * n] * (d == 2 ? h * h * h * kp.jac : 1.0);
        }
        const PUFE_GLOBAL double *v = gV + leaf * kp.n3;
        // V of a plane is read while the plane before it is summed
        double vn[3];
#pragma unroll
        for (int r = 0; r < 3; ++r) vn[r] = 64 * r + lane < n2 ? v[64 * r + lane] : 0.0;
        for (int z = 0; z < n; ++z) {
#pragma unroll
            for (int r = 0; r < 3; ++r) {
                const int q = 64 * r + lane;
                if (q < n2) {
                    sV[q] = 2.0 * vn[r];
                    if (z + 1 < n) vn[r] = v[(z + 1) * n2 + q];
                }
            }
            // the wave's own LDS writes above, then its reads below
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            double X[NC];
#pragma unroll
            for (int t = 0; t < NC; ++t) X[t] = 0.0;
            int x = k4, y = 0;
            for (int s = 0; s < n2; s += 4) {
                while (x >= n) x -= n, ++y;
                const bool in = s + k4 < n2;
                const int px = in ? x * NG : 0, py = in ? y * NG : 0;
                double a = row == 0 ? 1.0 : (row == 1 ? sV[in ? s + k4 : 0] : 0.0);
                a = in ? a : 0.0;
#pragma unroll
                for (int t = 0; t < NC; ++t) X[t] = mfma4(a, sT[ox[t] + px] * sT[oy[t] + py], X[t]);
                x += 4;
            }
#pragma unroll
            for (int k = 0; k < NG; ++k) {
                const double w = sT[2 * NG * n + z * NG + k];
#pragma unroll
                for (int t = 0; t < NC; ++t) Z[t][k] += w * X[t];
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
    }
    // sum over the waves in order; rows 0 and 1 are lanes 0..31
    __syncthreads();
    if (lane < 32)
#pragma unroll
        for (int t = 0; t < NC; ++t)
#pragma unroll
            for (int k = 0; k < NG; ++k) smem[(wave * NC * NG + t * NG + k) * 32 + lane] = Z[t][k];
    __syncthreads();
    PUFE_GLOBAL double *dst = (PUFE_GLOBAL double *)cx.mom + cx.elems[it.elem].ff_base + (int64_t)it.chunk * kMomFFSlot;
    for (int e = threadIdx.x; e < NC * NG * 32; e += 256)
        dst[e] = ((smem[e] + smem[NC * NG * 32 + e]) + smem[2 * NC * NG * 32 + e]) + smem[3 * NC * NG * 32 + e];
}

__global__ __launch_bounds__(256) void classical_moment_kernel(const CtxDev *__restrict__ ctxs,
                                                               const MomItemDev *__restrict__ items,
                                                               const double *__restrict__ V1) {
    __shared__ double smem[4 * (15 * kMaxGauss + kMaxGauss * kMaxGauss)];
    const MomItemDev it = items[blockIdx.x];
    const CtxDev &cx = ctxs[it.ctx];
    if (cx.kp.p == 2) classical_leaves<5>(cx, it, V1 ? V1 : cx.V, smem);
    else classical_leaves<3>(cx, it, V1 ? V1 : cx.V, smem);
}

// Sum of the K-chunk moments of one slot, in chunk order, into chunk 0.
__global__ __launch_bounds__(256) void moment_reduce_kernel(const CtxDev *__restrict__ ctxs,
                                                            const int4 *__restrict__ list) {
    const int4 e = list[blockIdx.x];
    const CtxDev &cx = ctxs[e.w];
    const ElemDev &el = cx.elems[e.x];
    const int64_t stride = (int64_t)mom_slots(el.nt) * kMomSlot;
    double *dst = cx.mom + el.mom_base + (int64_t)e.y * kMomSlot;
    const int nch = el.mchunk;
    for (int k = threadIdx.x; k < e.z; k += 256) {
        double acc = 0.0;
        int c = 0;
        for (; c + 4 <= nch; c += 4) {
            const double v0 = dst[c * stride + k], v1 = dst[(c + 1) * stride + k];
            const double v2 = dst[(c + 2) * stride + k], v3 = dst[(c + 3) * stride + k];
            acc += v0;
            acc += v1;
            acc += v2;
            acc += v3;
        }
        for (; c < nch; ++c) acc += dst[c * stride + k];
        dst[k] = acc;
    }
}

// ---------------------------------------------------------------- launchers

// Every variant: work group width, x steps of a line, and l <= 1, l <= 3 or the
// general one (tabulated radials, image weights), the last also for skewed
// cells (of any radial).
template <class F>
static hipError_t with_moment_kernel(int nw, int ks, int lmax, bool gen, bool skew, F &&f) {
#define PUFE_MOM_L(NW, KS)                                              \
    do {                                                                \
        if (skew) return f(moment_kernel<NW, KS, 3, true, true>);       \
        if (gen) return f(moment_kernel<NW, KS, 3, true, false>);       \
        if (lmax <= 1) return f(moment_kernel<NW, KS, 1, false, false>); \
        return f(moment_kernel<NW, KS, 3, false, false>);               \
    } while (0)
#define PUFE_MOM_K(NW)                    \
    do {                                  \
        if (ks == 1) PUFE_MOM_L(NW, 1);   \
        if (ks == 2) PUFE_MOM_L(NW, 2);   \
        PUFE_MOM_L(NW, 3);                \
    } while (0)
    if (nw == 4) PUFE_MOM_K(4);
    PUFE_MOM_K(8);
#undef PUFE_MOM_K
#undef PUFE_MOM_L
}

hipError_t init_moment_attributes() {
    for (int nw = 4; nw <= 8; nw += 4)
        for (int ks = 1; ks <= 3; ++ks)
            for (int v = 0; v < 4; ++v) {
                const hipError_t e = with_moment_kernel(nw, ks, v == 0 ? 1 : 3, v >= 2, v == 3, [](auto *k) {
                    return hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxDynLds);
                });
                if (e != hipSuccess) return e;
            }
    return hipSuccess;
}

hipError_t launch_moments(int nw, int n, int lmax, bool gen, bool skew, const CtxDev *ctxs, const MomItemDev *items,
                          int n_items, const int32_t *wave_task, const double *V, const double *wimg, size_t lds,
                          hipStream_t st) {
    if (n_items == 0) return hipSuccess;
    return with_moment_kernel(nw, (n + 3) / 4, lmax, gen, skew, [&](auto *k) {
        k<<<n_items, 64 * nw, lds, st>>>(ctxs, items, wave_task, V, wimg);
        return hipGetLastError();
    });
}

hipError_t launch_classical_moments(const CtxDev *ctxs, const MomItemDev *items, int n_items, const double *V,
                                    hipStream_t st) {
    if (n_items == 0) return hipSuccess;
    classical_moment_kernel<<<n_items, 256, 0, st>>>(ctxs, items, V);
    return hipGetLastError();
}

hipError_t launch_moment_reduce(const CtxDev *ctxs, const int4 *list, int n, hipStream_t st) {
    if (n == 0) return hipSuccess;
    moment_reduce_kernel<<<n, 256, 0, st>>>(ctxs, list);
    return hipGetLastError();
}

}  // namespace pufe
