// Element matrices from the moments of moments.hip: every entry of the upper
// 16x16 tiles of H_e and S_e is a short sum of moments.  Bound by reading the
// moments and by launch latency on small problems: the work is a few hundred
// multiply-adds per entry, once per element instead of once per point.  0.88 ms
// for 1096 elements of up to 283 functions, 98 us for 512 of up to 67.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "basis.hpp"
#include "moments.hpp"
#include "tables.hpp"

namespace pufe {

// v[i] for a run-time i of three values, without an indexed register array
__device__ __forceinline__ double pick(int i, const double (&v)[3]) { return i == 0 ? v[0] : (i == 1 ? v[1] : v[2]); }

// Place of the upper entry (a, b), a <= b, among the element's 16x16 tiles.
__device__ __forceinline__ int64_t tile_at(int a, int b) {
    const int I = a >> 4, J = b >> 4;
    return ((int64_t)J * (J + 1) / 2 + I) * 512 + (a & 15) * 16 + (b & 15);
}

// Enriched pairs of one quad (four 4x4 tiles of (f, g), f <= g): wave w takes
// the corner bits (cz, dz) = (w & 1, w >> 1) of the two rows, lane l the pair
// its MFMA result held, and forms the 16 entries of the other corner bits.
__device__ __forceinline__ void expand_enriched(const KParams &kp, const ElemDev &el, const double *__restrict__ mom,
                                                int quad, const int16_t *__restrict__ pos, double *__restrict__ out) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int cz = wave & 1, dz = wave >> 1, iz = cz + dz;
    const int nt = el.nt, nfun = el.nfun, nfe = el.nfe;
    const int blk = (lane >> 2) & 3, i = lane >> 4, j = lane & 3;
    const int pr = 4 * quad + blk;
    if (pr >= nt * (nt + 1) / 2) return;
    int J = 0;
    while ((J + 1) * (J + 2) / 2 <= pr) ++J;
    const int I = pr - J * (J + 1) / 2;
    const int f = 4 * I + i, g = 4 * J + j;
    if (f > g || g >= nfun) return;
    const double *ma = mom + (int64_t)quad * kMomSlot + lane;
    const int pfg = I * nt + J, pgf = J * nt + I, qa = mom_quads_ae(nt);
    const double *mb = mom + (int64_t)(qa + pfg / 4) * kMomSlot + 16 * i + 4 * (pfg & 3) + j;
    const double *mc = mom + (int64_t)(qa + pgf / 4) * kMomSlot + 16 * j + 4 * (pgf & 3) + i;
    double a[3][3], a1[3][3], en[3][3];   // [kx][ky]: A and E at iz, A against 1 in z
    double ac[3][3], ad[3][3];            // A against m_cz and m_dz in z (skewed cells)
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int y = 0; y < 3; ++y) {
            const double z0 = ma[(18 * k + 3 * y) * 64], z1 = ma[(18 * k + 3 * y + 1) * 64],
                         z2 = ma[(18 * k + 3 * y + 2) * 64];
            a[k][y] = iz == 0 ? z0 : (iz == 1 ? z1 : z2);
            a1[k][y] = z0 + 2.0 * z1 + z2;
            ac[k][y] = z1 + (cz ? z2 : z0);
            ad[k][y] = z1 + (dz ? z2 : z0);
            en[k][y] = ma[(18 * k + 9 + 3 * y + iz) * 64];
        }
    double bx[2][2][3], by[2][3][2], bz[2][3][3];   // [0]: B(f, g), [1]: B(g, f)
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const double *m = t ? mc : mb;
        const int lz = t ? dz : cz;
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int y = 0; y < 3; ++y) {
                if (k < 2) bx[t][k][y] = m[(9 * k + 3 * y + iz) * 64];
                if (y < 2) by[t][k][y] = m[(18 + 6 * k + 3 * y + iz) * 64];
                bz[t][k][y] = m[(36 + 6 * k + 2 * y + lz) * 64];
            }
    }
    // x polynomials of m_c m_d and m_c in 1, xi, xi^2
    const double prod[3][3] = {{0.25, -0.5, 0.25}, {0.25, 0.0, -0.25}, {0.25, 0.5, 0.25}};
    const double lin[2][2] = {{0.5, -0.5}, {0.5, 0.5}};
    const double hz[2] = {cz ? 0.5 : -0.5, dz ? 0.5 : -0.5};
    const bool skew = kp.skew != 0;
#pragma unroll
    for (int cd = 0; cd < 16; ++cd) {
        const int cx = cd & 1, dx = (cd >> 1) & 1, cy = (cd >> 2) & 1, dy = cd >> 3, iy = cy + dy;
        const int c = cx | (cy << 1) | (cz << 2), d = dx | (dy << 1) | (dz << 2);
        const int ka = pos[c * kMaxFun + f], kb = pos[d * kMaxFun + g];
        if (ka < 0 || kb < 0) continue;
        const double *P = prod[cx + dx];
        auto xq = [&](const double (&m)[3][3], int y) { return P[0] * m[0][y] + P[1] * m[1][y] + P[2] * m[2][y]; };
        const double hx[2] = {cx ? 0.5 : -0.5, dx ? 0.5 : -0.5}, hy[2] = {cy ? 0.5 : -0.5, dy ? 0.5 : -0.5};
        const double S = xq(a, iy);
        double H = xq(en, iy);
        H += kp.G[0] * hx[0] * hx[1] * a[0][iy];
        H += kp.G[4] * hy[0] * hy[1] * (xq(a, 0) + 2.0 * xq(a, 1) + xq(a, 2));
        H += kp.G[8] * hz[0] * hz[1] * xq(a1, iy);
        if (skew) {
            // d_x M_c d_y M_d + d_y M_c d_x M_d and the other two mixed terms
            auto xl = [&](const double (&m)[3][3], int b, int y) { return lin[b][0] * m[0][y] + lin[b][1] * m[1][y]; };
            auto ly = [&](int b, const double *v) { return b ? v[1] + v[2] : v[0] + v[1]; };
            const double xd[3] = {xl(a, dx, 0), xl(a, dx, 1), xl(a, dx, 2)}, xc[3] = {xl(a, cx, 0), xl(a, cx, 1), xl(a, cx, 2)};
            H += kp.G[1] * (hx[0] * hy[1] * ly(cy, xd) + hy[0] * hx[1] * ly(dy, xc));
            H += kp.G[2] * (hx[0] * hz[1] * xl(ac, dx, iy) + hz[0] * hx[1] * xl(ad, cx, iy));
            const double vd[3] = {xq(ac, 0), xq(ac, 1), xq(ac, 2)}, vc[3] = {xq(ad, 0), xq(ad, 1), xq(ad, 2)};
            H += kp.G[5] * (hy[0] * hz[1] * ly(dy, vd) + hz[0] * hy[1] * ly(cy, vc));
        }
        H += kp.sd[0] * (hx[1] * (lin[cx][0] * bx[0][0][iy] + lin[cx][1] * bx[0][1][iy]) +
                         hx[0] * (lin[dx][0] * bx[1][0][iy] + lin[dx][1] * bx[1][1][iy]));
        H += kp.sd[1] * (hy[1] * (P[0] * by[0][0][cy] + P[1] * by[0][1][cy] + P[2] * by[0][2][cy]) +
                         hy[0] * (P[0] * by[1][0][dy] + P[1] * by[1][1][dy] + P[2] * by[1][2][dy]));
        H += kp.sd[2] * (hz[1] * xq(bz[0], iy) + hz[0] * xq(bz[1], iy));
        const int ra = nfe + ka, rb = nfe + kb;
        if (f == g && ra > rb) continue;   // its mirror image writes it
        const int64_t at = tile_at(min(ra, rb), max(ra, rb));
        out[at] = 0.5 * H;
        out[at + 256] = S;
    }
}

// Mixed entries (classical function i, enriched function (c, f)) of two
// enrichment functions f: one thread per (i, c), the moments in LDS.
template <int P>
__device__ __forceinline__ void expand_mixed(const KParams &kp, const ElemDev &el, const double *__restrict__ mom,
                                             int pair, const int16_t *__restrict__ pos, double *__restrict__ sM,
                                             double *__restrict__ out) {
    constexpr int NF = P + 2, N1 = P + 1, NFE = N1 * N1 * N1, N3 = NF * NF * NF;
    const int nt = el.nt, nf = min(2, el.nfun - 2 * pair), nfe = el.nfe;
    const double *m = mom + (int64_t)(mom_quads_ae(nt) + mom_quads_b(nt) + pair / 4) * kMomSlot;
    // sM[function][component][kz][ky][kx]
    const int f0 = 2 * (pair & 3);   // of the group's 8: row tile f0 / 4, rows f0 % 4 and the next
    for (int e = threadIdx.x; e < 5 * NF * 32; e += blockDim.x) {
        const int col = e & 15, f = (e >> 4) & 1, r = e >> 5, kz = r % NF, c = r / NF;
        if (f < nf && col < NF * NF)
            sM[(f * 5 + c) * N3 + kz * NF * NF + col] = m[(((f0 >> 2) * 5 + c) * NF + kz) * 64 + 16 * ((f0 & 3) + f) + col];
    }
    __syncthreads();
    for (int ic = threadIdx.x; ic < 8 * NFE; ic += blockDim.x) {
        const int c = ic & 7, i = ic >> 3;
        const int in[3] = {i % N1, (i / N1) % N1, i / (N1 * N1)};
        // per direction and node: N M, N' M, N M', N' M'
        double vv[2][NF], dv[2][NF], vd[2][NF], dd[2][NF];
#pragma unroll
        for (int d = 0; d < 2; ++d) {
            const int b = (c >> d) & 1;
#pragma unroll
            for (int k = 0; k < NF; ++k) {
                const double t = -1.0 + k * (2.0 / (NF - 1));
                double L[3], D[3];
                lagrange_1d(P, t, L, D);
                const double Ln = pick(in[d], L), Dn = pick(in[d], D);
                const double M = b ? 0.5 * (1.0 + t) : 0.5 * (1.0 - t), dM = b ? 0.5 : -0.5;
                vv[d][k] = Ln * M;
                dv[d][k] = Dn * M;
                vd[d][k] = Ln * dM;
                dd[d][k] = Dn * dM;
            }
        }
        const bool skew = kp.skew != 0;
        for (int f = 0; f < nf; ++f) {
            const int k = pos[c * kMaxFun + 2 * pair + f];
            if (k < 0) continue;
            const double *mf = sM + f * 5 * N3;
            double S = 0.0, H = 0.0;
#pragma unroll 1
            for (int z = 0; z < NF; ++z) {
                // z factors at this node (an array of them would be indexed at run time)
                const double t = -1.0 + z * (2.0 / (NF - 1));
                double L[3], D[3];
                lagrange_1d(P, t, L, D);
                const double Lz = pick(in[2], L), Dz = pick(in[2], D), Mz = c & 4 ? 0.5 * (1.0 + t) : 0.5 * (1.0 - t);
                const double dMz = c & 4 ? 0.5 : -0.5, vz = Lz * Mz, dvz = Dz * Mz, vdz = Lz * dMz, ddz = Dz * dMz;
                double s = 0.0, gx = 0.0, gy = 0.0, v = 0.0, bx = 0.0, by = 0.0, bz = 0.0;
                double gxy = 0.0, gxz = 0.0, gzx = 0.0, gyz = 0.0, gzy = 0.0;
#pragma unroll
                for (int y = 0; y < NF; ++y) {
                    const double *q = mf + (z * NF + y) * NF;
                    double s0 = 0.0, d0 = 0.0, v0 = 0.0, x0 = 0.0, y0 = 0.0, z0 = 0.0;
#pragma unroll
                    for (int x = 0; x < NF; ++x) {
                        s0 += vv[0][x] * q[x];
                        d0 += dd[0][x] * q[x];
                        v0 += vv[0][x] * q[N3 + x];
                        x0 += dv[0][x] * q[2 * N3 + x];
                        y0 += vv[0][x] * q[3 * N3 + x];
                        z0 += vv[0][x] * q[4 * N3 + x];
                    }
                    s += vv[1][y] * s0;
                    gx += vv[1][y] * d0;
                    gy += dd[1][y] * s0;
                    v += vv[1][y] * v0;
                    bx += vv[1][y] * x0;
                    by += dv[1][y] * y0;
                    bz += vv[1][y] * z0;
                    if (skew) {
                        double dv0 = 0.0, vd0 = 0.0;
#pragma unroll
                        for (int x = 0; x < NF; ++x) {
                            dv0 += dv[0][x] * q[x];
                            vd0 += vd[0][x] * q[x];
                        }
                        gxy += vd[1][y] * dv0 + dv[1][y] * vd0;
                        gxz += vv[1][y] * dv0;
                        gzx += vv[1][y] * vd0;
                        gyz += dv[1][y] * s0;
                        gzy += vd[1][y] * s0;
                    }
                }
                S += vz * s;
                H += vz * (kp.G[0] * gx + kp.G[4] * gy + v + kp.sd[0] * bx + kp.sd[1] * by) + kp.G[8] * ddz * s +
                     kp.sd[2] * dvz * bz;
                if (skew)
                    H += kp.G[1] * vz * gxy + kp.G[2] * (vdz * gxz + dvz * gzx) + kp.G[5] * (vdz * gyz + dvz * gzy);
            }
            const int64_t at = tile_at(i, nfe + k);
            out[at] = 0.5 * H;
            out[at + 256] = S;
        }
    }
}

// Classical entries (i <= j) of one element, the moments in LDS.
template <int P>
__device__ __forceinline__ void expand_classical(const KParams &kp, const ElemDev &el, const double *__restrict__ mom,
                                                 double *__restrict__ sM, double *__restrict__ out) {
    constexpr int NG = 2 * P + 1, N1 = P + 1, NFE = N1 * N1 * N1, N3 = NG * NG * NG, NC = (NG * NG + 15) / 16;
    const int parts = el.fchunk;
    for (int e = threadIdx.x; e < NC * NG * 32; e += blockDim.x) {   // rows 0 and 1: w, 2 V w
        const int l = e & 31, r = e >> 5, kz = r % NG, t = r / NG, col = 16 * t + (l & 15);
        if (col >= NG * NG) continue;
        double v = 0.0;
        for (int s = 0; s < parts; ++s) v += mom[(int64_t)s * kMomFFSlot + e];
        sM[(l >> 4) * N3 + kz * NG * NG + col] = v;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < NFE * (NFE + 1) / 2; e += blockDim.x) {
        int j = (int)((sqrt(8.0 * e + 1.0) - 1.0) * 0.5);
        while ((j + 1) * (j + 2) / 2 <= e) ++j;
        while (j * (j + 1) / 2 > e) --j;
        const int i = e - j * (j + 1) / 2;
        double vv[2][NG], dd[2][NG], dv[2][NG], vd[2][NG];
#pragma unroll
        for (int d = 0; d < 2; ++d) {
            const int ia = d == 0 ? i % N1 : (i / N1) % N1, ja = d == 0 ? j % N1 : (j / N1) % N1;
#pragma unroll
            for (int k = 0; k < NG; ++k) {
                double L[3], D[3];
                lagrange_1d(P, -1.0 + k * (2.0 / (NG - 1)), L, D);
                const double La = pick(ia, L), Da = pick(ia, D), Lb = pick(ja, L), Db = pick(ja, D);
                vv[d][k] = La * Lb;
                dd[d][k] = Da * Db;
                dv[d][k] = Da * Lb;
                vd[d][k] = La * Db;
            }
        }
        const bool skew = kp.skew != 0;
        double S = 0.0, H = 0.0;
#pragma unroll 1
        for (int z = 0; z < NG; ++z) {
            double L[3], D[3];
            lagrange_1d(P, -1.0 + z * (2.0 / (NG - 1)), L, D);
            const int iz = i / (N1 * N1), jz = j / (N1 * N1);
            const double vz = pick(iz, L) * pick(jz, L), ddz = pick(iz, D) * pick(jz, D);
            const double dvz = pick(iz, D) * pick(jz, L), vdz = pick(iz, L) * pick(jz, D);
            double s = 0.0, gx = 0.0, gy = 0.0, v = 0.0, gxy = 0.0, gxz = 0.0, gzx = 0.0, gyz = 0.0, gzy = 0.0;
#pragma unroll
            for (int y = 0; y < NG; ++y) {
                const double *q = sM + (z * NG + y) * NG;
                double s0 = 0.0, d0 = 0.0, v0 = 0.0, dv0 = 0.0, vd0 = 0.0;
#pragma unroll
                for (int x = 0; x < NG; ++x) {
                    s0 += vv[0][x] * q[x];
                    d0 += dd[0][x] * q[x];
                    v0 += vv[0][x] * q[N3 + x];
                    if (skew) {
                        dv0 += dv[0][x] * q[x];
                        vd0 += vd[0][x] * q[x];
                    }
                }
                s += vv[1][y] * s0;
                gx += vv[1][y] * d0;
                gy += dd[1][y] * s0;
                v += vv[1][y] * v0;
                if (skew) {
                    gxy += vd[1][y] * dv0 + dv[1][y] * vd0;
                    gxz += vv[1][y] * dv0;
                    gzx += vv[1][y] * vd0;
                    gyz += dv[1][y] * s0;
                    gzy += vd[1][y] * s0;
                }
            }
            S += vz * s;
            H += vz * (kp.G[0] * gx + kp.G[4] * gy + v) + kp.G[8] * ddz * s;
            if (skew)
                H += kp.G[1] * vz * gxy + kp.G[2] * (vdz * gxz + dvz * gzx) + kp.G[5] * (vdz * gyz + dvz * gzy);
        }
        const int64_t at = tile_at(i, j);
        out[at] = 0.5 * H;
        out[at + 256] = S;
    }
}

__global__ __launch_bounds__(256) void moment_expand_kernel(const CtxDev *__restrict__ ctxs,
                                                            const int4 *__restrict__ list, double *partial1) {
    __shared__ int16_t pos[8 * kMaxFun];   // enriched entry of (corner, function), -1: none
    __shared__ double sM[2 * 5 * 64];
    const int4 e = list[blockIdx.x];
    const CtxDev &cx = ctxs[e.w];
    const ElemDev &el = cx.elems[e.x];
    const KParams &kp = cx.kp;
    if (e.y != MOM_X_FE) {
        for (int k = threadIdx.x; k < 8 * kMaxFun; k += 256) pos[k] = -1;
        __syncthreads();
        for (int k = threadIdx.x; k < el.nloc - el.nfe; k += 256) {
            const int pk = cx.edof[el.edof_off + k];
            pos[(pk & 7) * kMaxFun + ((pk >> 3) & 255)] = (int16_t)k;
        }
        __syncthreads();
    }
    const double *mom = cx.mom + el.mom_base;
    double *out = (partial1 ? partial1 : cx.partial) + el.part_base * 512;
    if (e.y == MOM_X_ENR) {
        expand_enriched(kp, el, mom, e.z, pos, out);
    } else if (e.y == MOM_X_MIXED) {
        if (kp.p == 2) expand_mixed<2>(kp, el, mom, e.z, pos, sM, out);
        else expand_mixed<1>(kp, el, mom, e.z, pos, sM, out);
    } else {
        if (kp.p == 2) expand_classical<2>(kp, el, cx.mom + el.ff_base, sM, out);
        else expand_classical<1>(kp, el, cx.mom + el.ff_base, sM, out);
    }
}

hipError_t launch_moment_expand(const CtxDev *ctxs, const int4 *list, int n, double *partial, hipStream_t st) {
    if (n == 0) return hipSuccess;
    moment_expand_kernel<<<n, 256, 0, st>>>(ctxs, list, partial);
    return hipGetLastError();
}

}  // namespace pufe
