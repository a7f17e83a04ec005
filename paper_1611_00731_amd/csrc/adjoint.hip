// Adjoint of the assembly in moment form (gfx950), orthorhombic cells.
//
// L = Re<P, H> + Re<Q, S> is linear in the moments of moments.hip.  Folding
// the element's Ps and Qs onto them (once per element) leaves polynomials of
// low degree as coefficients,
//   L = sum_q w_q [ 1/2 sum_fg (LA Psi_f Psi_g + LE (grad Psi_f . grad Psi_g + 2 V Psi_f Psi_g))
//                   + sum_fg LB_d(f, g) d_d Psi_f Psi_g + sum_f (lp Psi_f + lv 2 V Psi_f + ld . grad Psi_f) + lc 2 V ],
// all functions of the point, so with y_f = sum_g LE Psi_g
//   dL/dPsi_f   = w [ sum_g LA Psi_g + 2 V y_f + sum_g LB_d(g, f) d_d Psi_g + lp + 2 V lv ]
//   dL/d d_d Psi_f = w [ sum_g LE d_d Psi_g + LB_d(f, g) Psi_g + ld ]
//   dL/dV       = w [ sum_f Psi_f (y_f + 2 lv) + 2 lc ]
// and a centre's force is -sum (dL/dPsi_f d_k Psi_f + dL/d d_d Psi_f d_dk Psi_f).
// Along a line of points the polynomials in z and y are evaluated on the
// coefficients (as on the accumulators of the forward sums), and the sum over
// g and the polynomials in x run on v_mfma_f64_4x4x4: row operand the coefficients,
// column operand the polynomial times the functions at 4 points.  The polynomials of
// each direction are the products of its two hats, m_0 m_0 (1, t, t^2) with t =
// m_1 / m_0, and m_0 (1, t): the powers of t scale the operand, m_0 the results.  The
// powers of x itself add up to a product of hats with cancellation near the face
// where it vanishes: with them dL/dV of one vertex was off by up to 1.2e-12 of itself
// there, by 1e-14 now as through the functions' own products.  Per point and ordered
// pair that is 31 multiply-adds on the matrix cores, where the products of Ps
// with the element's own functions take 256; P and Q share one pass.
// Bound by issue and latency between the matrix instructions (two waves a SIMD,
// a dozen LDS reads and as many FP64 operations per 15 of them), not by these.
// Measured, P and Q together: 512 elements of one or two row tiles, 7036 leaves
// of 216 points 0.97 ms (8.1 ms through the element's own functions), 216
// elements of up to eleven, 664 leaves 1.50 ms (17.4 ms).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "adjoint.hpp"
#include "basis.hpp"
#include "device_common.hpp"
#include "enrich.hpp"
#include "moment_math.hpp"
#include "moments.hpp"
#include "stage.hpp"
#include "tables.hpp"

namespace pufe {

namespace {

constexpr int kAdjPair = 108 * 64;   // doubles of a quad: LE, LA (27 each), LB_x, LB_y, LB_z (18 each)

// (kx, ky) products of the mixed polynomials, four per MFMA
__host__ __device__ constexpr int adj_steps(int p) { return ((p + 2) * (p + 2) + 3) / 4; }
__host__ __device__ inline int adj_mixed_doubles(int p) { return 5 * adj_steps(p) * (p + 2) * 64; }

// 1D tables of a leaf, unweighted: x [n][2] (m_0, m_1 / m_0 of the two hats); y, z
// [n][5] (m_0 m_0, m_0 m_1, m_1 m_1, m_0, m_1); mixed [n][p + 2] and classical
// [n][2 p + 1] Lagrange values for x, y, z; weights [3][n] (z with the leaf's volume
// factor).
struct AdjTab {
    int yt, zt, fx, fy, fz, gx, gy, gz, w, size;
    __host__ __device__ AdjTab(int n, int p) {
        const int nf = p + 2, ng = 2 * p + 1;
        yt = 2 * n;
        zt = yt + 5 * n;
        fx = zt + 5 * n;
        fy = fx + nf * n;
        fz = fy + nf * n;
        gx = fz + nf * n;
        gy = gx + ng * n;
        gz = gy + ng * n;
        w = gz + ng * n;
        size = w + 3 * n;
    }
};

// Row stride (doubles) of the table: value, gradient and Hessian of a point
// (10 doubles) side by side, an odd number of 16-byte units per row.
__host__ __device__ inline int adj_stride(int points) { return 10 * ((points + 1) & ~1) + 2; }

// Enrichment functions of a group with gradients and Hessians (xx yy zz xy xz
// yz) at one point: function m at o + m MS.  Hessian of g(s) S(r):
// 4 g'' r r^T S + 2 g' (S I + r grad S^T + grad S r^T) + g Hess S.
template <int L>
__device__ __forceinline__ void adj_group(const GroupDev &G, const double *__restrict__ img,
                                          const double *__restrict__ spl, const double *x, double *o, int MS) {
    constexpr int NM = 2 * L + 1;
    const double rc2 = G.rc * G.rc, inv_rc2 = 1.0 / rc2;
    const double *c0 = img + 3 * G.img_off;
    bool first = true;
    for (int k = 0; k < G.nimg; ++k) {
        const double r[3] = {x[0] - c0[3 * k], x[1] - c0[3 * k + 1], x[2] - c0[3 * k + 2]};
        const double s = r[0] * r[0] + r[1] * r[1] + r[2] * r[2];
        if (s >= rc2) continue;
        double g0, g1, g2;
        if (G.nspl > 0) {
            spline_radial<true>(G, spl, s, g0, g1, g2);
        } else {
            const double ex = exp(-G.a * s), c = 1.0 - s * inv_rc2, c2 = c * c;
            g0 = ex * c2 * c;
            g1 = -ex * c2 * (G.a * c + 3.0 * inv_rc2);
            g2 = ex * c * (G.a * G.a * c2 + 6.0 * G.a * c * inv_rc2 + 6.0 * inv_rc2 * inv_rc2);
        }
        double S[7], dS[21], hS[42];
        solid_harmonics(L, r[0], r[1], r[2], S, dS);
        solid_harmonics_hess(L, r[0], r[1], r[2], hS);
        constexpr int ii[6] = {0, 1, 2, 0, 0, 1}, jj[6] = {0, 1, 2, 1, 2, 2};
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            double v[10];
            v[0] = g0 * S[m];
#pragma unroll
            for (int d = 0; d < 3; ++d) v[1 + d] = 2.0 * g1 * r[d] * S[m] + g0 * dS[3 * m + d];
#pragma unroll
            for (int t = 0; t < 6; ++t) {
                const int i = ii[t], j = jj[t];
                v[4 + t] = 4.0 * g2 * r[i] * r[j] * S[m] +
                           2.0 * g1 * ((i == j ? S[m] : 0.0) + r[i] * dS[3 * m + j] + dS[3 * m + i] * r[j]) +
                           g0 * hS[6 * m + t];
            }
            dbl2 *om = (dbl2 *)(o + m * MS);
#pragma unroll
            for (int c = 0; c < 5; ++c) {
                const dbl2 u = {v[2 * c], v[2 * c + 1]};
                om[c] = first ? u : om[c] + u;
            }
        }
        first = false;
    }
    if (first)
#pragma unroll
        for (int m = 0; m < NM; ++m)
#pragma unroll
            for (int c = 0; c < 5; ++c) ((dbl2 *)(o + m * MS))[c] = (dbl2){0.0, 0.0};
}

// What dL/dPsi_f = u + 2 V y and dL/d grad Psi_f = (gx, gy, gz) at one point do
// to the forces (times the weight): lane l holds function row l / 16 of its
// block at point l % 4.
__device__ __forceinline__ void adj_force_val(const double *__restrict__ pf, double ub, double w, double *fr) {
    const dbl2 a = *(const dbl2 *)pf, b = *(const dbl2 *)(pf + 2);
    fr[0] += w * (ub * a[1]);
    fr[1] += w * (ub * b[0]);
    fr[2] += w * (ub * b[1]);
}

__device__ __forceinline__ void adj_force_grad(const double *__restrict__ pf, double gx, double gy, double gz, double w,
                                               double *fr) {
    // Hessian xx, yy, zz, xy, xz, yz
    const dbl2 c = *(const dbl2 *)(pf + 4), d = *(const dbl2 *)(pf + 6), e = *(const dbl2 *)(pf + 8);
    fr[0] += w * (gx * c[0] + gy * d[1] + gz * e[0]);
    fr[1] += w * (gx * d[1] + gy * c[1] + gz * e[1]);
    fr[2] += w * (gx * e[0] + gy * e[1] + gz * d[0]);
}

// v summed over the functions of the lanes of one point, which are all blocks
// (rep 1), blocks of one parity (rep 2) or one block (rep 4); every lane of the
// point gets the sum.  Rows of a block: ones times v on the matrix cores;
// blocks: rotations within the 16 lanes.
__device__ __forceinline__ double adj_sum_functions(double v, int rep) {
    double s = mfma4(1.0, v, 0.0);
    auto rot = [](double v, auto ctrl) {
        const uint64_t x = __builtin_bit_cast(uint64_t, v);
        const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)x, decltype(ctrl)::value, 0xf, 0xf, true);
        const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(x >> 32), decltype(ctrl)::value, 0xf, 0xf, true);
        return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
    };
    if (rep < 4) s += rot(s, std::integral_constant<int, 0x128>());   // row_ror:8
    if (rep < 2) s += rot(s, std::integral_constant<int, 0x124>());   // row_ror:4
    return s;
}

// A stage as the wave tasks see it: nyl lines per plane from (z0, y0), planes
// npl, n points per line.
struct AdjView {
    const double *P, *T, *V, *W;
    int n, z0, y0, nyl, npl, lane;
};

// One quad of ordered tile pairs (f in tile I, g in tile J) over a stage, in
// three roles whose coefficients stay in registers over the stage (27 + 27 of
// LE and LA, or 54 of LB), folded per plane and per line; lane l carries the
// coefficient of function row l % 4, column l / 16, and rep lines lie side by
// side in the blocks.
//   ADJ_EA  y, LE grad Psi, LA Psi and dL/dV     15 MFMAs per 4 points
//   ADJ_B   LB(f, g) Psi                          8
//   ADJ_BT  LB(g, f) . grad Psi                   8
enum { ADJ_EA = 0, ADJ_B = 1, ADJ_BT = 2 };

template <int ROLE>
__device__ __forceinline__ void adj_pairs(const double *__restrict__ lam, const AdjTab &mt, const AdjView &v, int og, int of,
                                          int rep, double *__restrict__ sDV, double *fr) {
    constexpr int NX = ROLE == ADJ_EA ? 27 : 18;   // coefficients of the first part
    const int n = v.n, lane = v.lane;
    const int nyg = (v.nyl + rep - 1) / rep, sub = (lane >> 2) & (rep - 1);
    double c[54];
#pragma unroll
    for (int m = 0; m < 54; ++m) c[m] = lam[m * 64];
#pragma unroll 1
    for (int pz = 0; pz < v.npl; ++pz) {
        const double *tz = v.T + mt.zt + 5 * (v.z0 + pz);
        const double w0 = tz[0], w1 = tz[1], w2 = tz[2], l0 = tz[3], l1 = tz[4];
        double q1[9], q2[9], q3[9];   // EA: E, A; B: x (6), y (6), z (9)
        if (ROLE == ADJ_EA) {
#pragma unroll
            for (int e = 0; e < 9; ++e) {
                q1[e] = w0 * c[3 * e] + w1 * c[3 * e + 1] + w2 * c[3 * e + 2];
                q2[e] = w0 * c[NX + 3 * e] + w1 * c[NX + 3 * e + 1] + w2 * c[NX + 3 * e + 2];
            }
        } else {
#pragma unroll
            for (int e = 0; e < 6; ++e) {
                q1[e] = w0 * c[3 * e] + w1 * c[3 * e + 1] + w2 * c[3 * e + 2];
                q2[e] = w0 * c[NX + 3 * e] + w1 * c[NX + 3 * e + 1] + w2 * c[NX + 3 * e + 2];
            }
#pragma unroll
            for (int e = 0; e < 9; ++e) q3[e] = l0 * c[36 + 2 * e] + l1 * c[36 + 2 * e + 1];
        }
#pragma unroll 1
        for (int yg = 0; yg < nyg; ++yg) {
            const int yr = yg * rep + sub, yl = min(yr, v.nyl - 1);
            const double *ty = v.T + mt.yt + 5 * (v.y0 + yl);
            const double y0 = ty[0], y1 = ty[1], y2 = ty[2], m0 = ty[3], m1 = ty[4];
            double e[3], a[3], b[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                if (ROLE == ADJ_EA) {
                    e[k] = y0 * q1[3 * k] + y1 * q1[3 * k + 1] + y2 * q1[3 * k + 2];
                    a[k] = y0 * q2[3 * k] + y1 * q2[3 * k + 1] + y2 * q2[3 * k + 2];
                } else {
                    if (k < 2) e[k] = y0 * q1[3 * k] + y1 * q1[3 * k + 1] + y2 * q1[3 * k + 2];
                    a[k] = m0 * q2[2 * k] + m1 * q2[2 * k + 1];
                    b[k] = y0 * q3[3 * k] + y1 * q3[3 * k + 1] + y2 * q3[3 * k + 2];
                }
            }
            const int q0 = (pz * v.nyl + yl) * n;
#pragma unroll 1
            for (int x = lane & 3; x < ((n + 3) & ~3); x += 4) {
                const int xo = min(x, n - 1), q = q0 + xo;
                const bool in = x < n && yr < v.nyl;
                const double mx = v.T[2 * xo], t = v.T[2 * xo + 1], w = in ? v.W[q] : 0.0;
                const double *pg = v.P + og + 10 * q, *pf = v.P + of + 10 * q;
                const dbl2 g0 = *(const dbl2 *)pg, g1 = *(const dbl2 *)(pg + 2);
                double p = g0[0], dx = g0[1], dy = g1[0], dz = g1[1];
                if (ROLE == ADJ_EA) {
                    double y = 0.0, u = 0.0, gx = 0.0, gy = 0.0, gz = 0.0;
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        y = mfma4(e[k], p, y);
                        gx = mfma4(e[k], dx, gx);
                        gy = mfma4(e[k], dy, gy);
                        gz = mfma4(e[k], dz, gz);
                        u = mfma4(a[k], p, u);
                        if (k < 2) {
                            p *= t;
                            dx *= t;
                            dy *= t;
                            dz *= t;
                        }
                    }
                    const double h = mx * mx, wh = w * h;
                    adj_force_val(pf, u + v.V[q] * y, wh, fr);
                    adj_force_grad(pf, gx, gy, gz, wh, fr);
                    const double dv = h * adj_sum_functions(pf[0] * y, rep);
                    if (lane < 4 * rep && in) sDV[q] = dv;
                } else if (ROLE == ADJ_B) {
                    double gx = 0.0, gy = 0.0, gz = 0.0;
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        gy = mfma4(a[k], p, gy);
                        gz = mfma4(b[k], p, gz);
                        if (k < 2) gx = mfma4(e[k], p, gx);
                        if (k < 2) p *= t;
                    }
                    adj_force_grad(pf, gx, mx * gy, mx * gz, w * mx, fr);
                } else {
                    double u = 0.0, u1 = 0.0, u2 = 0.0;
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        u = mfma4(a[k], dy, u);
                        u2 = mfma4(b[k], dz, u2);
                        if (k < 2) {
                            u1 = mfma4(e[k], dx, u1);
                            dx *= t;
                            dy *= t;
                            dz *= t;
                        }
                    }
                    adj_force_val(pf, u1 + mx * (u + u2), w * mx, fr);
                }
            }
        }
    }
}

// The mixed part of 16 functions (4 row tiles, one per block): with GRAD the
// three gradient polynomials, else lp and lv (which gives dL/dV its part).
template <int P, bool GRAD>
__device__ __forceinline__ void adj_mixed(const double *__restrict__ lam, const AdjTab &mt, const AdjView &v, int of, int rep,
                                          double *__restrict__ sDV, double *fr) {
    constexpr int NF = P + 2, NS = adj_steps(P), ND = GRAD ? 3 : 2, D0 = GRAD ? 2 : 0;
    const int n = v.n, lane = v.lane;
    const int nyg = (v.nyl + rep - 1) / rep, sub = (lane >> 2) & (rep - 1);
    double c[ND][NS][NF];
#pragma unroll
    for (int d = 0; d < ND; ++d)
#pragma unroll
        for (int t = 0; t < NS; ++t)
#pragma unroll
            for (int z = 0; z < NF; ++z) c[d][t][z] = lam[(((D0 + d) * NS + t) * NF + z) * 64];
    int ix[NS], iy[NS];   // polynomials of this lane's k = l / 16 in each step
    bool live[NS];
#pragma unroll
    for (int t = 0; t < NS; ++t) {
        const int k = 4 * t + (lane >> 4);
        live[t] = k < NF * NF;
        ix[t] = live[t] ? k % NF : 0;
        iy[t] = live[t] ? k / NF : 0;
    }
#pragma unroll 1
    for (int pz = 0; pz < v.npl; ++pz) {
        const double *tz = v.T + mt.fz + NF * (v.z0 + pz);
        double q1[ND][NS];
#pragma unroll
        for (int d = 0; d < ND; ++d)
#pragma unroll
            for (int t = 0; t < NS; ++t) {
                double s = 0.0;
#pragma unroll
                for (int z = 0; z < NF; ++z) s += tz[z] * c[d][t][z];
                q1[d][t] = s;
            }
#pragma unroll 1
        for (int yg = 0; yg < nyg; ++yg) {
            const int yr = yg * rep + sub, yl = min(yr, v.nyl - 1);
            double fy[NS];
#pragma unroll
            for (int t = 0; t < NS; ++t) fy[t] = live[t] ? v.T[mt.fy + NF * (v.y0 + yl) + iy[t]] : 0.0;
            const int q0 = (pz * v.nyl + yl) * n;
#pragma unroll 1
            for (int x = lane & 3; x < ((n + 3) & ~3); x += 4) {
                const int xo = min(x, n - 1), q = q0 + xo;
                const bool in = x < n && yr < v.nyl;
                const double w = in ? v.W[q] : 0.0;
                double o[ND];
#pragma unroll
                for (int d = 0; d < ND; ++d) o[d] = 0.0;
#pragma unroll
                for (int t = 0; t < NS; ++t) {
                    const double b = v.T[mt.fx + NF * xo + ix[t]] * fy[t];
#pragma unroll
                    for (int d = 0; d < ND; ++d) o[d] = mfma4(q1[d][t], b, o[d]);
                }
                const double *pf = v.P + of + 10 * q;
                if (GRAD) {
                    adj_force_grad(pf, o[0], o[1], o[ND - 1], w, fr);
                } else {
                    adj_force_val(pf, o[0] + v.V[q] * o[1], w, fr);
                    const double dv = adj_sum_functions(2.0 * pf[0] * o[1], rep);
                    if (lane < 4 * rep && in) sDV[q] = dv;
                }
            }
        }
    }
}

}  // namespace

int64_t adj_doubles(int nt, int p) {
    const int ng = 2 * p + 1;
    return (int64_t)mom_quads_b(nt) * kAdjPair + (int64_t)((nt + 3) / 4) * adj_mixed_doubles(p) + ((ng * ng * ng + 7) & ~7);
}

// Lines side by side in the blocks of an MFMA where a task has fewer than four
// tiles or tile pairs.
__host__ __device__ static inline int adj_rep(int nt, bool pairs) { return nt == 1 ? 4 : (nt == 2 && !pairs ? 2 : 1); }

// Task un of an element: role and quad or group.
enum { ADJ_M_GRAD = 3, ADJ_M_VAL = 4 };
struct AdjTask {
    int role, idx;
};
__device__ __forceinline__ AdjTask adj_task(int un, int qb, int gf) {
    if (un < qb) return {ADJ_EA, un};
    un -= qb;
    if (un < gf) return {ADJ_M_GRAD, un};
    un -= gf;
    if (un < gf) return {ADJ_M_VAL, un};
    un -= gf;
    return un < qb ? AdjTask{ADJ_B, un} : AdjTask{ADJ_BT, un - qb};
}

// LDS map: the table [4 nt rows], 2 V, weights, dL/dV of every quad and group, 1D tables,
// classical coefficients of a plane, force sums of every task, Gauss
// rule, cell constants, image centres, groups (each has one function at least).
static size_t adj_lds_bytes(int nt, int nimg, int n, int p, int points, int planes) {
    const int ng = 2 * p + 1, sums = mom_quads_b(nt) + (nt + 3) / 4;
    return sizeof(double) * ((size_t)4 * nt * adj_stride(points) + (size_t)(2 + sums) * points + AdjTab(n, p).size +
                             (size_t)planes * ng * ng + (size_t)adj_tasks(nt) * 48 + 2 * kMaxGauss + 12 + 3 * (size_t)nimg) +
           sizeof(GroupDev) * std::min(kMaxGroups, 4 * nt) + 64;
}

AdjStage adj_stage(int nt, int nimg, int n, int p) {
    AdjStage s{0, 0, 0, 0};
    for (int nw = nt <= 3 ? 4 : 8; nw <= 8 && s.waves == 0; nw += 4) {
        const size_t room = nw == 4 ? (size_t)79 * 1024 : kMaxDynLds;
        auto take = [&](int planes, int lines) {
            const size_t b = adj_lds_bytes(nt, nimg, n, p, (planes > 0 ? planes * n : lines) * n, std::max(planes, 1));
            if (b > room) return false;
            s = AdjStage{nw, planes, lines, b};
            return true;
        };
        bool ok = false;
        for (int groups = 1; groups <= n && !ok; ++groups) {
            const int planes = (n + groups - 1) / groups;
            if (n * n * planes > 256 && planes > 1) continue;
            ok = take(planes, 0);
        }
        for (int groups = 2; groups <= n && !ok; ++groups) ok = take(0, (n + groups - 1) / groups);
    }
    return s;
}

// One work group of NW waves per item (a range of an element's stages).  Stages
// alternate the functions, the tasks, and dL/dV.
template <int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2))) void adjoint_moment_kernel(
    const CtxDev *__restrict__ ctx, const MomItemDev *__restrict__ items, const int64_t *__restrict__ base,
    const double *__restrict__ lam0, const double *__restrict__ V, double *__restrict__ dV, double *__restrict__ fpart,
    int max_ngrp) {
    extern __shared__ __attribute__((aligned(16))) double smem[];
    constexpr int NT = 64 * NW;
    const MomItemDev it = items[blockIdx.x];
    const CtxDev &cx = *ctx;
    const KParams &kp = cx.kp;
    const ElemDev &el = cx.elems[it.elem];
    const GroupDev *gGroups = cx.groups + el.grp_off;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = kp.n, n2 = n * n, p = kp.p, ng = 2 * p + 1, nf = p + 2;
    const int ngrp = el.ngrp, nt = el.nt, nfun = el.nfun, rows = 4 * nt;
    const int img0 = ngrp > 0 ? gGroups[0].img_off : 0;
    const int nimg = ngrp > 0 ? gGroups[ngrp - 1].img_off + gGroups[ngrp - 1].nimg - img0 : 0;
    const int planes = it.tab & 255, lines = it.tab >> 8;
    const int nyl = planes > 0 ? n : lines, maxpl = planes > 0 ? planes : 1, points = maxpl * nyl * n;
    const int qb = mom_quads_b(nt), gf = (nt + 3) / 4, tasks = adj_tasks(nt);
    const AdjTab mt(n, p);
    const int RS = adj_stride(points);
    double *sP = smem;
    double *sV = sP + rows * RS, *sW = sV + points, *sDV = sW + points;   // sDV[qb + gf][points]
    double *sT = sDV + (qb + gf) * points;
    double *sC = sT + mt.size;                                             // [planes][ng ng]
    double *sF = sC + maxpl * ng * ng;                                 // [tasks][block][row][3]
    double *sGx = sF + tasks * 48, *sGw = sGx + kMaxGauss;
    double *sE = sGw + kMaxGauss, *sOrg = sE + 9, *sImg = sOrg + 3;
    GroupDev *sG = (GroupDev *)(sImg + 3 * nimg);
    const double *lam = lam0 + base[it.elem];
    const double *lamc = lam + (int64_t)qb * kAdjPair + (int64_t)gf * adj_mixed_doubles(p);

    for (int k = tid; k < 3 * nimg; k += NT) sImg[k] = cx.img[3 * (size_t)img0 + k];
    for (int g = tid; g < ngrp; g += NT) {
        GroupDev G = gGroups[g];
        G.img_off -= img0;
        sG[g] = G;
    }
    if (tid < n) {
        sGx[tid] = kp.gx[tid];
        sGw[tid] = kp.gw[tid];
    }
    if (tid < 9) sE[tid] = kp.E[tid];
    if (tid < 3) sOrg[tid] = el.ijk[0] * kp.E[tid] + el.ijk[1] * kp.E[3 + tid] + el.ijk[2] * kp.E[6 + tid];
    for (int k = nfun * RS + tid; k < rows * RS; k += NT) sP[k] = 0.0;   // padding rows stay zero
    for (int k = tid; k < tasks * 48; k += NT) sF[k] = 0.0;
    const int spl = planes > 0 ? (n + planes - 1) / planes : n * ((n + lines - 1) / lines);   // stages per leaf
    const int sb = (int)it.leaf_b, se = (int)it.leaf_e;
    __syncthreads();
#pragma unroll 1
    for (int st = sb; st < se; ++st) {
        const int lf = st / spl, ss = st - lf * spl;
        int z0, y0, npl, ny;   // the stage's planes and lines
        if (planes > 0) {
            z0 = ss * planes;
            npl = min(planes, n - z0);
            y0 = 0;
            ny = n;
        } else {
            const int per = (n + lines - 1) / lines;
            z0 = ss / per;
            npl = 1;
            y0 = (ss - z0 * per) * lines;
            ny = min(lines, n - y0);
        }
        const int npts = npl * ny * n;
        const int64_t leaf = el.leaf_off + lf, qbase = leaf * kp.n3 + (int64_t)z0 * n2 + y0 * n;
        {
            const uint32_t code = cx.leaves[leaf];
            const int lev = (int)(code >> 27);
            const double h = 1.0 / (double)(1u << lev);
            const double c[3] = {2.0 * (code & 511u) + 1.0, 2.0 * ((code >> 9) & 511u) + 1.0,
                                 2.0 * ((code >> 18) & 511u) + 1.0};
            if (ss == 0 || st == sb) {
                const double vol = h * h * h * kp.jac;
                for (int e = tid; e < mt.size; e += NT) {
                    int j = e;
                    double v;
                    if (j < mt.fx) {
                        const int d = j < mt.yt ? 0 : (j < mt.zt ? 1 : 2), m = d == 0 ? 2 : 5;
                        j -= d == 0 ? 0 : (d == 1 ? mt.yt : mt.zt);
                        const int i = j / m, k = j - i * m;
                        const double x = -1.0 + ((d == 0 ? c[0] : (d == 1 ? c[1] : c[2])) + sGx[i]) * h;
                        const double m0 = 0.5 * (1.0 - x), m1 = 0.5 * (1.0 + x);
                        if (d == 0) v = k == 0 ? m0 : m1 / m0;
                        else v = k == 0 ? m0 * m0 : (k == 1 ? m0 * m1 : (k == 2 ? m1 * m1 : (k == 3 ? m0 : m1)));
                    } else if (j < mt.w) {
                        const bool mixed = j < mt.gx;
                        j -= mixed ? mt.fx : mt.gx;
                        const int m = mixed ? nf : ng, i = j / m, k = j - i * m, d = i < n ? 0 : (i < 2 * n ? 1 : 2);
                        const double x = -1.0 + ((d == 0 ? c[0] : (d == 1 ? c[1] : c[2])) + sGx[i - d * n]) * h;
                        v = m == 5 ? lagrange_equi<5>(k, x) : (m == 4 ? lagrange_equi<4>(k, x) : lagrange_equi<3>(k, x));
                    } else {
                        j -= mt.w;
                        v = sGw[j % n] * (j >= 2 * n ? vol : 1.0);
                    }
                    sT[e] = v;
                }
            }
            for (int u = tid; u < ngrp * npts; u += NT) {
                const int g = u / npts, q = u - g * npts;
                const int k[3] = {q % n, y0 + (q / n) % ny, z0 + q / (n * ny)};
                double xi[3], x[3];
#pragma unroll
                for (int d = 0; d < 3; ++d) xi[d] = -1.0 + (c[d] + sGx[k[d]]) * h;
#pragma unroll
                for (int cc = 0; cc < 3; ++cc)
                    x[cc] = sOrg[cc] + 0.5 * (xi[0] + 1.0) * sE[cc] + 0.5 * (xi[1] + 1.0) * sE[3 + cc] +
                            0.5 * (xi[2] + 1.0) * sE[6 + cc];
                const GroupDev &G = sG[g];
                double *o = sP + G.fbase * RS + 10 * q;
                switch (G.l) {
                    case 0: adj_group<0>(G, sImg, kp.spl, x, o, RS); break;
                    case 1: adj_group<1>(G, sImg, kp.spl, x, o, RS); break;
                    case 2: adj_group<2>(G, sImg, kp.spl, x, o, RS); break;
                    default: adj_group<3>(G, sImg, kp.spl, x, o, RS); break;
                }
            }
            for (int q = tid; q < npts; q += NT) sV[q] = 2.0 * V[qbase + q];
        }
        __syncthreads();   // tables complete
        for (int q = tid; q < npts; q += NT) {
            const int x = q % n, y = y0 + (q / n) % ny, z = z0 + q / (n * ny);
            sW[q] = sT[mt.w + x] * sT[mt.w + n + y] * sT[mt.w + 2 * n + z];
        }
        for (int k = tid; k < npl * ng * ng; k += NT) {   // classical coefficients of the planes
            const int pz = k / (ng * ng), c = k - pz * ng * ng;
            double v = 0.0;
            for (int z = 0; z < ng; ++z) v += sT[mt.gz + ng * (z0 + pz) + z] * lamc[z * ng * ng + c];
            sC[k] = v;
        }
        __syncthreads();
        // tasks in descending weight, dealt to the waves there and back
        for (int rd = 0; rd * NW < tasks; ++rd) {
            const int un = rd * NW + (rd & 1 ? NW - 1 - wave : wave);
            if (un >= tasks) continue;
            const AdjTask tk = adj_task(un, qb, gf);
            const int rep = adj_rep(nt, tk.role <= ADJ_BT);
            const int blk = ((lane >> 2) & 3) / rep, k4 = lane >> 4, j4 = lane & 3;
            const int op = 16 * k4 + 4 * blk + j4;
            const AdjView v{sP, sT, sV, sW, n, z0, y0, ny, npl, lane};
            double fr[3] = {0.0, 0.0, 0.0};
            if (tk.role <= ADJ_BT) {
                // a quad past the last pair repeats it: its coefficients are zero in the fold
                const bool pad = 4 * tk.idx + blk >= nt * nt;
                const int pr = pad ? nt * nt - 1 : 4 * tk.idx + blk, I = pr / nt, J = pr - I * nt, prT = J * nt + I;
                const double *m = lam + (int64_t)tk.idx * kAdjPair + op;
                const int og = (4 * J + k4) * RS, of = (4 * I + k4) * RS;
                if (tk.role == ADJ_EA) {
                    adj_pairs<ADJ_EA>(m, mt, v, og, of, rep, sDV + tk.idx * points, fr);
                } else if (tk.role == ADJ_B) {
                    adj_pairs<ADJ_B>(m + 54 * 64, mt, v, og, of, rep, nullptr, fr);
                } else {
                    const double *mT = pad ? m : lam + (int64_t)(prT >> 2) * kAdjPair + 16 * j4 + 4 * (prT & 3) + k4;
                    adj_pairs<ADJ_BT>(mT + 54 * 64, mt, v, og, of, rep, nullptr, fr);
                }
            } else {
                const int tile = min(4 * tk.idx + blk, nt - 1), of = (4 * tile + k4) * RS;
                const double *m = lam + (int64_t)qb * kAdjPair + (int64_t)tk.idx * adj_mixed_doubles(p) + op;
                double *dv = sDV + (qb + tk.idx) * points;
                if (p == 2) {
                    if (tk.role == ADJ_M_GRAD) adj_mixed<2, true>(m, mt, v, of, rep, dv, fr);
                    else adj_mixed<2, false>(m, mt, v, of, rep, dv, fr);
                } else {
                    if (tk.role == ADJ_M_GRAD) adj_mixed<1, true>(m, mt, v, of, rep, dv, fr);
                    else adj_mixed<1, false>(m, mt, v, of, rep, dv, fr);
                }
            }
            // points of a row, then into the task's own sums
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                fr[k] += __shfl_xor(fr[k], 1, 64);
                fr[k] += __shfl_xor(fr[k], 2, 64);
            }
            if (j4 == 0)
#pragma unroll
                for (int k = 0; k < 3; ++k) sF[un * 48 + (4 * ((lane >> 2) & 3) + k4) * 3 + k] += fr[k];
        }
        __syncthreads();
        if (dV)
            for (int q = tid; q < npts; q += NT) {
                const int x = q % n, yl = (q / n) % ny, pz = q / (n * ny);
                double s = 0.0;
                for (int t = 0; t < qb + gf; ++t) s += sDV[t * points + q];
                double cl = 0.0;
                for (int b = 0; b < ng; ++b) {
                    double r = 0.0;
                    for (int a = 0; a < ng; ++a) r += sT[mt.gx + ng * x + a] * sC[pz * ng * ng + b * ng + a];
                    cl += sT[mt.gy + ng * (y0 + yl) + b] * r;
                }
                dV[qbase + q] = sW[q] * (s + 2.0 * cl);
            }
        __syncthreads();
    }
    // forces: tasks in order per function, functions in order per group
    double *sS = sP;   // [rows][3]
    for (int e = tid; e < 3 * rows; e += NT) {
        const int f = e / 3, k = e - 3 * f, I = f >> 2, r = f & 3;
        double s = 0.0;
        for (int un = 0; un < tasks; ++un) {
            const AdjTask tk = adj_task(un, qb, gf);
            const bool pair = tk.role <= ADJ_BT;
            const int rep = adj_rep(nt, pair);
            for (int b = 0; b < 4; ++b) {
                const int pr = 4 * tk.idx + b / rep;
                const bool mine = pair ? pr < nt * nt && pr / nt == I : pr == I;
                if (mine) s += sF[un * 48 + (4 * b + r) * 3 + k];
            }
        }
        sS[e] = s;
    }
    __syncthreads();
    for (int e = tid; e < 3 * max_ngrp; e += NT) {
        const int g = e / 3, k = e - 3 * g;
        double s = 0.0;
        if (g < ngrp)
            for (int f = sG[g].fbase; f < sG[g].fbase + 2 * sG[g].l + 1 && f < nfun; ++f) s += sS[3 * f + k];
        const int64_t at = ((int64_t)it.chunk * max_ngrp) * 3 + e;
        fpart[at] = -s;
    }
}

// ------------------------------------------------------------------- fold

// One ordered quad per wave: coefficients of the moments of pair (f, g) from
// the 64 corner pairs of Ps and Qs.
__device__ __forceinline__ void fold_pairs(const KParams &kp, const ElemDev &el, int quad, const int16_t *__restrict__ pos,
                                           const double *__restrict__ Ps, const double *__restrict__ Qs, int npad,
                                           double *__restrict__ out) {
    const int lane = threadIdx.x & 63, nt = el.nt, nfe = el.nfe;
    const int blk = (lane >> 2) & 3, pr = 4 * quad + blk;
    const int I = pr / nt, J = pr - I * nt, f = 4 * I + (lane & 3), g = 4 * J + (lane >> 4);
    double *o = out + (int64_t)quad * kAdjPair + lane;
    if (pr >= nt * nt || f >= el.nfun || g >= el.nfun) {
        for (int m = 0; m < 108; ++m) o[m * 64] = 0.0;
        return;
    }
    double E[3][3][3], A[3][3][3], X[2][3][3], Y[3][2][3], Z[3][3][2];
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int y = 0; y < 3; ++y)
#pragma unroll
            for (int z = 0; z < 3; ++z) {
                E[k][y][z] = A[k][y][z] = 0.0;
                if (k < 2) X[k][y][z] = 0.0;
                if (y < 2) Y[k][y][z] = 0.0;
                if (z < 2) Z[k][y][z] = 0.0;
            }
#pragma unroll
    for (int cdz = 0; cdz < 4; ++cdz) {
        const int cz = cdz & 1, dz = cdz >> 1, iz = cz + dz;
        const double hz[2] = {cz ? 0.5 : -0.5, dz ? 0.5 : -0.5};
        double e9[3][3], a9[3][3], x6[2][3], y6[3][2];
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int y = 0; y < 3; ++y) {
                e9[k][y] = a9[k][y] = 0.0;
                if (k < 2) x6[k][y] = 0.0;
                if (y < 2) y6[k][y] = 0.0;
            }
#pragma unroll
        for (int cd = 0; cd < 16; ++cd) {
            const int cx = cd & 1, dx = (cd >> 1) & 1, cy = (cd >> 2) & 1, dy = cd >> 3, iy = cy + dy;
            const int ka = pos[(cx | (cy << 1) | (cz << 2)) * kMaxFun + f], kb = pos[(dx | (dy << 1) | (dz << 2)) * kMaxFun + g];
            const bool ok = ka >= 0 && kb >= 0;
            const int64_t at = ok ? (int64_t)(nfe + ka) * npad + nfe + kb : 0;
            const double pv = ok && Ps ? Ps[at] : 0.0, qv = ok && Qs ? 2.0 * Qs[at] : 0.0;
            const double hx[2] = {cx ? 0.5 : -0.5, dx ? 0.5 : -0.5}, hy[2] = {cy ? 0.5 : -0.5, dy ? 0.5 : -0.5};
            // one is m_0 m_0 + 2 m_0 m_1 + m_1 m_1 in the direction of the derivatives
            const double xx = kp.G[0] * hx[0] * hx[1] * pv, yy = kp.G[4] * hy[0] * hy[1] * pv;
            const int ix = cx + dx;
            e9[ix][iy] += pv;
            a9[ix][iy] += qv;
            a9[0][iy] += xx;
            a9[1][iy] += 2.0 * xx;
            a9[2][iy] += xx;
            a9[ix][0] += yy;
            a9[ix][1] += 2.0 * yy;
            a9[ix][2] += yy;
            x6[cx][iy] += hx[1] * kp.sd[0] * pv;
            y6[ix][cy] += hy[1] * kp.sd[1] * pv;
        }
        const double zz = kp.G[8] * hz[0] * hz[1];
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int y = 0; y < 3; ++y) {
                E[k][y][iz] += e9[k][y];
                A[k][y][iz] += a9[k][y];
                A[k][y][0] += zz * e9[k][y];
                A[k][y][1] += 2.0 * zz * e9[k][y];
                A[k][y][2] += zz * e9[k][y];
                if (k < 2) X[k][y][iz] += x6[k][y];
                if (y < 2) Y[k][y][iz] += y6[k][y];
                Z[k][y][cz] += hz[1] * kp.sd[2] * e9[k][y];
            }
    }
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int y = 0; y < 3; ++y)
#pragma unroll
            for (int z = 0; z < 3; ++z) {
                o[(9 * k + 3 * y + z) * 64] = E[k][y][z];
                o[(27 + 9 * k + 3 * y + z) * 64] = A[k][y][z];
                if (k < 2) o[(54 + 9 * k + 3 * y + z) * 64] = X[k][y][z];
                if (y < 2) o[(72 + 6 * k + 3 * y + z) * 64] = Y[k][y][z];
                if (z < 2) o[(90 + 6 * k + 2 * y + z) * 64] = Z[k][y][z];
            }
}

// Classical shape functions of a column of Ps contracted at one node: v with
// the values, d with the reference derivatives.
template <int P>
__device__ __forceinline__ void fold_column(const double *__restrict__ col, int64_t stride, const double (&L)[3][3],
                                            const double (&D)[3][3], double *v, double *d) {
    constexpr int N1 = P + 1;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int i2 = 0; i2 < N1; ++i2) {
        double r[3] = {0.0, 0.0, 0.0};   // value, x and y derivative
#pragma unroll
        for (int i1 = 0; i1 < N1; ++i1) {
            double q0 = 0.0, q1 = 0.0;
#pragma unroll
            for (int i0 = 0; i0 < N1; ++i0) {
                const double c = col[(int64_t)(i0 + N1 * (i1 + N1 * i2)) * stride];
                q0 += L[0][i0] * c;
                q1 += D[0][i0] * c;
            }
            r[0] += L[1][i1] * q0;
            r[1] += L[1][i1] * q1;
            r[2] += D[1][i1] * q0;
        }
        s[0] += L[2][i2] * r[0];
        s[1] += L[2][i2] * r[1];
        s[2] += L[2][i2] * r[2];
        s[3] += D[2][i2] * r[0];
    }
    *v = s[0];
    d[0] = s[1];
    d[1] = s[2];
    d[2] = s[3];
}

// A row tile: wave w takes its function w, lanes the nodes.
template <int P>
__device__ __forceinline__ void fold_mixed(const KParams &kp, const ElemDev &el, int tile, const int16_t *__restrict__ pos,
                                           const double *__restrict__ Ps, const double *__restrict__ Qs, int npad,
                                           double *__restrict__ out) {
    constexpr int NF = P + 2, NS = adj_steps(P), N3 = NF * NF * NF;
    const int lane = threadIdx.x & 63, row = threadIdx.x >> 6, f = 4 * tile + row, nfe = el.nfe;
    double *o = out + (int64_t)mom_quads_b(el.nt) * kAdjPair + (int64_t)(tile >> 2) * adj_mixed_doubles(P) + 4 * (tile & 3) + row;
    double m[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    const int kx = lane % NF, ky = (lane / NF) % NF, kz = lane / (NF * NF);
    if (lane < N3 && f < el.nfun) {
        const double t[3] = {-1.0 + kx * (2.0 / (NF - 1)), -1.0 + ky * (2.0 / (NF - 1)), -1.0 + kz * (2.0 / (NF - 1))};
        double L[3][3], D[3][3];
#pragma unroll
        for (int d = 0; d < 3; ++d) lagrange_1d(P, t[d], L[d], D[d]);
        for (int c = 0; c < 8; ++c) {
            const int k = pos[c * kMaxFun + f];
            if (k < 0) continue;
            const double b[3] = {c & 1 ? 0.5 : -0.5, c & 2 ? 0.5 : -0.5, c & 4 ? 0.5 : -0.5};
            const double h[3] = {0.5 + b[0] * t[0], 0.5 + b[1] * t[1], 0.5 + b[2] * t[2]};
            const double M = h[0] * h[1] * h[2], dM[3] = {b[0] * h[1] * h[2], h[0] * b[1] * h[2], h[0] * h[1] * b[2]};
            if (Ps) {
                double v, d[3];
                fold_column<P>(Ps + nfe + k, npad, L, D, &v, d);
                m[0] += kp.G[0] * dM[0] * d[0] + kp.G[4] * dM[1] * d[1] + kp.G[8] * dM[2] * d[2];
                m[1] += M * v;
#pragma unroll
                for (int e = 0; e < 3; ++e) m[2 + e] += kp.sd[e] * M * d[e];
            }
            if (Qs) {
                double v, d[3];
                fold_column<P>(Qs + nfe + k, npad, L, D, &v, d);
                m[0] += 2.0 * M * v;
            }
        }
    }
    // polynomial (kx, ky) is column 4 step + k, k = lane / 16 of the operand
    const int cc = ky * NF + kx, at = 16 * (cc & 3);
    if (lane < N3)
#pragma unroll
        for (int d = 0; d < 5; ++d) o[((d * NS + (cc >> 2)) * NF + kz) * 64 + at] = m[d];
    // polynomials past the last one
    for (int e = lane; e < 5 * NF * (4 * NS - NF * NF); e += 64) {
        const int x = NF * NF + e / (5 * NF), d = (e / NF) % 5, z = e % NF;
        o[((d * NS + (x >> 2)) * NF + z) * 64 + 16 * (x & 3)] = 0.0;
    }
}

template <int P>
__device__ __forceinline__ void fold_classical(const ElemDev &el, const double *__restrict__ Ps, int npad,
                                               double *__restrict__ sum, double *__restrict__ out) {
    constexpr int NG = 2 * P + 1, N1 = P + 1, N3 = NG * NG * NG;
    double *o = out + (int64_t)mom_quads_b(el.nt) * kAdjPair + (int64_t)((el.nt + 3) / 4) * adj_mixed_doubles(P);
    // 128 threads per half of the rows
    const int e = threadIdx.x & 127, half = threadIdx.x >> 7;
    const int kx = e % NG, ky = (e / NG) % NG, kz = e / (NG * NG);
    double L[3][3], D[3][3], s = 0.0;
    lagrange_1d(P, -1.0 + kx * (2.0 / (NG - 1)), L[0], D[0]);
    lagrange_1d(P, -1.0 + ky * (2.0 / (NG - 1)), L[1], D[1]);
    lagrange_1d(P, -1.0 + kz * (2.0 / (NG - 1)), L[2], D[2]);
    if (Ps)
#pragma unroll 2
        for (int i = half; i < N1 * N1 * N1; i += 2) {
            double v, d[3];
            fold_column<P>(Ps + (int64_t)i * npad, 1, L, D, &v, d);
            const int i0 = i % N1, i1 = (i / N1) % N1, i2 = i / (N1 * N1);
            auto at = [](const double (&x)[3], int k) { return k == 0 ? x[0] : (k == 1 ? x[1] : x[2]); };
            s += at(L[0], i0) * at(L[1], i1) * at(L[2], i2) * v;
        }
    if (half) sum[e] = s;
    __syncthreads();
    if (!half && e < N3) o[e] = 0.5 * (s + sum[e]);
}

__global__ __launch_bounds__(256) void adjoint_fold_kernel(const CtxDev *__restrict__ ctx, const int4 *__restrict__ list,
                                                           const int64_t *__restrict__ pt_off, const double *__restrict__ P,
                                                           const double *__restrict__ Q, const int64_t *__restrict__ base,
                                                           double *__restrict__ lam) {
    __shared__ __attribute__((aligned(8))) int16_t pos[8 * kMaxFun];   // the classical part's sums where it has no use for positions
    static_assert(sizeof(int16_t) * 8 * kMaxFun >= sizeof(double) * 128, "128 partial sums");
    const int4 e = list[blockIdx.x];
    const CtxDev &cx = *ctx;
    const ElemDev &el = cx.elems[e.x];
    const int npad = 16 * ((el.nloc + 15) / 16);
    const double *Ps = P ? P + pt_off[e.x] : nullptr, *Qs = Q ? Q + pt_off[e.x] : nullptr;
    for (int k = threadIdx.x; k < 8 * kMaxFun; k += 256) pos[k] = -1;
    __syncthreads();
    for (int k = threadIdx.x; k < el.nloc - el.nfe; k += 256) {
        const int pk = cx.edof[el.edof_off + k];
        pos[(pk & 7) * kMaxFun + ((pk >> 3) & 255)] = (int16_t)k;
    }
    __syncthreads();
    double *out = lam + base[e.x];
    if (e.y == ADJ_PAIRS) {
        const int quad = 4 * e.z + (threadIdx.x >> 6);
        if (quad < mom_quads_b(el.nt)) fold_pairs(cx.kp, el, quad, pos, Ps, Qs, npad, out);
    } else if (e.y == ADJ_MIXED) {
        if (cx.kp.p == 2) fold_mixed<2>(cx.kp, el, e.z, pos, Ps, Qs, npad, out);
        else fold_mixed<1>(cx.kp, el, e.z, pos, Ps, Qs, npad, out);
    } else {
        if (cx.kp.p == 2) fold_classical<2>(el, Ps, npad, (double *)pos, out);
        else fold_classical<1>(el, Ps, npad, (double *)pos, out);
    }
}

hipError_t init_adjoint_attributes() {
    const hipError_t e = hipFuncSetAttribute((const void *)adjoint_moment_kernel<4>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxDynLds);
    if (e != hipSuccess) return e;
    return hipFuncSetAttribute((const void *)adjoint_moment_kernel<8>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)kMaxDynLds);
}

hipError_t launch_adjoint_fold(const CtxDev *ctx, const int4 *list, int n, const int64_t *pt_off, const double *Ps,
                               const double *Qs, const int64_t *base, double *lam, hipStream_t st) {
    if (n == 0) return hipSuccess;
    adjoint_fold_kernel<<<n, 256, 0, st>>>(ctx, list, pt_off, Ps, Qs, base, lam);
    return hipGetLastError();
}

hipError_t launch_adjoint_moments(int nw, const CtxDev *ctx, const MomItemDev *items, int n_items, const int64_t *base,
                                  const double *lam, const double *V, double *dV, double *fpart, int max_ngrp, size_t lds,
                                  hipStream_t st) {
    if (n_items == 0) return hipSuccess;
    auto *k = nw == 4 ? adjoint_moment_kernel<4> : adjoint_moment_kernel<8>;
    k<<<n_items, 64 * nw, lds, st>>>(ctx, items, base, lam, V, dV, fpart, max_ngrp);
    return hipGetLastError();
}

}  // namespace pufe
