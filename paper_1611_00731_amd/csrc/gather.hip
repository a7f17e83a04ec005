// Assembly of H and S (eq. disceig3d, Bloch boundary conditions of eqs. bloch
// and wbpspace): every entry of the block-sparse matrices is gathered from the
// element matrices that hold it,
//   H[g_a][g_b] = sum over elements of conj(p_a) p_b H_e[a][b],
// and written once.  One wave per pair of blocks (v, w), (w, v): the matrices
// are Hermitian, so the second block is the conjugate transpose of the first.
// Where there are few blocks, several waves share the entries of each; where there
// are very many small ones, a wave takes eight blocks.
//
// Bound by writing H and S.  Scattering element by element instead needs the
// outputs zeroed, two reads and two writes of each entry per element that
// touches it, and one launch per element colour (8, or up to 27 on odd
// meshes); gathered, an entry costs one write and one 8-byte read per element
// (2.4 on average) from tiles that the caches hold, in one launch: 4.75 and
// 2.05 ms for 3.5 GB of H and S; with 64 elements the whole assembly 53.6 and
// 33.6 us.  The sums run in element order, so results do not depend on the
// launch.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "gather.hpp"

namespace pufe {

namespace {

// Local function of element slot `slot` of the vertex at corner c (-1: the
// element does not hold it): classical functions first, then the corner's
// enriched entries from cs.
__device__ __forceinline__ int local_of(int p, int nfs, int nfe, int c, int slot, int cs) {
    if (slot >= nfs) return nfe + cs + (slot - nfs);
    if (p == 1) return c;
    if (p == 2) {   // midpoint slots lie in the positive directions of the vertex
        if (slot & c) return -1;
        const int d0 = (slot & 1) + 2 * (c & 1), d1 = ((slot >> 1) & 1) + (c & 2), d2 = (slot >> 2) + ((c >> 1) & 2);
        return d0 + 3 * d1 + 9 * d2;
    }
    if (slot == 0) return c;
    const int d = (slot - 1) >> 1;
    if ((c >> d) & 1) return -1;
    const int k = (c & ((1 << d) - 1)) | ((c >> (d + 1)) << d);   // the corner's place among those with bit d clear
    return 8 + 2 * (4 * d + k) + ((slot - 1) & 1);
}

__device__ __forceinline__ int64_t entry_of(int a, int b) {
    const int lo = min(a, b), hi = max(a, b), I = lo >> 4, J = hi >> 4;
    return ((int64_t)J * (J + 1) / 2 + I) * 512 + (lo & 15) * 16 + (hi & 15);
}

__device__ __forceinline__ int64_t read_lane64(int64_t v, int lane) {
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)v, lane), hi = __builtin_amdgcn_readlane((uint32_t)(v >> 32), lane);
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

template <int DT>
struct OutType {
    typedef double2 type;
};
template <>
struct OutType<1> {
    typedef float2 type;
};
template <>
struct OutType<2> {
    typedef double type;
};
template <int DT>
__device__ __forceinline__ typename OutType<DT>::type out_value(double re, double im) {
    if constexpr (DT == 0) return make_double2(re, im);
    else if constexpr (DT == 1) return make_float2((float)re, (float)im);
    else return re;
}

}  // namespace

// Staged projector sums of a wave: the rows of v and w for 20 projector
// functions and 28 degrees of freedom, with four work groups on a compute unit.
constexpr int kGatherStage = 576;

// NL: the separable term H_ij += sum_J h_J f_J^i conj(f_J^j) is added before the
// write.  Added to the finished H it costs a read and a write of H, most of the
// blocks being coupled: 474 us for 14.5 M entries and 20 projector functions
// after 130 us of this kernel, 248 us together now.  A wave stages its block's
// rows of f in LDS, k-point by k-point; what does not fit is read through the
// caches.
// GL lanes work on a block: a wave, or eight of its lanes.
template <int DT, bool BLOCH, bool NL, int GL>
__global__ __launch_bounds__(256) void gather_kernel(const CtxDev *__restrict__ ctxs, const int4 *__restrict__ list, int n,
                                                     const double *__restrict__ partial1, void *H1, void *S1,
                                                     const KPoints kps, const double2 *__restrict__ f,
                                                     const double *__restrict__ pfun_h, int n_pfun, int64_t n_dof) {
    typedef typename OutType<DT>::type Out;
    constexpr bool WAVE = GL == 64;
    __shared__ double2 sFs[NL && WAVE ? 4 : 1][NL && WAVE ? kGatherStage : 1];
    __shared__ double2 sZ[kMaxKPerLaunch * 27];   // exp(2 pi i kappa . dn), dn = (t % 3, t / 3 % 3, t / 9) - 1
    // contributions of the blocks of eight lanes: the lanes of a block leave its loop
    // at different times, so they read each other's through LDS
    __shared__ int64_t sBase[WAVE ? 1 : 256];
    __shared__ int sCon[WAVE ? 1 : 256][3];
    const int lane = threadIdx.x & (GL - 1);
    const int at = WAVE ? __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6)) : blockIdx.x * 32 + threadIdx.x / 8;
    const bool live = at < n;
    const int4 e = list[live ? at : n - 1];
    const CtxDev &cx = ctxs[e.w & (kBlockProjected - 1)];
    const int ncon = block_count(e), nfs = cx.kp.nfs, nfe = cx.kp.nfe, p = cx.kp.p;
    // lane j holds contribution j: element tiles, corners, lattice shift and
    // the corners' enriched entries
    int64_t base = 0;
    int cc = 0, ca0 = 0, cb0 = 0, shift = 13, sa3 = 0, sb3 = 0;
    if (lane < ncon) {
        const int64_t con = cx.contr[block_first(e) + lane];
        const ElemDev &el = cx.elems[contr_elem(con)];
        cc = contr_corners(con);
        const int ca = cc >> 3, cb = cc & 7;
        base = el.part_base * 512;
        ca0 = el.cs[ca] | ((el.cs[ca + 1] - el.cs[ca]) << 16);
        cb0 = el.cs[cb] | ((el.cs[cb + 1] - el.cs[cb]) << 16);
        sa3 = (el.shifts >> (3 * ca)) & 7;
        sb3 = (el.shifts >> (3 * cb)) & 7;
        auto dn = [&](int d) { return ((sb3 >> d) & 1) - ((sa3 >> d) & 1) + 1; };
        shift = dn(0) + 3 * dn(1) + 9 * dn(2);
    }
    // a block that meets no cell boundary has phase one (and, with the
    // Bloch-periodic enrichment, the boundary phase on classical rows only).  Real
    // output of the periodic form has none at all: kappa is an integer, of any size,
    // and the cosine of a rounded 2 pi kappa is not one
    const bool mine = (BLOCH || DT != 2) && lane < ncon && (BLOCH ? (sa3 | sb3) != 0 : shift != 13);
    const bool wraps = WAVE ? __any(mine) : ((__ballot(mine) >> (threadIdx.x & 56)) & 255u) != 0;
    if (!WAVE) {
        sBase[threadIdx.x] = base;
        sCon[threadIdx.x][0] = cc | (shift << 6) | (sa3 << 11) | (sb3 << 14);
        sCon[threadIdx.x][1] = ca0;
        sCon[threadIdx.x][2] = cb0;
    }
    if (__syncthreads_or(live && wraps)) {
        for (int i = threadIdx.x; i < kps.nk * 27; i += 256) {
            const int k = i / 27, t = i - 27 * k;
            double sn, cs;
            sincos(2.0 * M_PI * (kps.kap[k][0] * (t % 3 - 1) + kps.kap[k][1] * ((t / 3) % 3 - 1) + kps.kap[k][2] * (t / 9 - 1)),
                   &sn, &cs);
            sZ[i] = make_double2(cs, sn);
        }
        __syncthreads();
    }
    if (!live) return;
    const int first = threadIdx.x & ~(GL - 1);   // contribution j of the block, in lane j or in LDS
    auto con_base = [&](int j) { return WAVE ? read_lane64(base, j) : sBase[first + j]; };
    auto con_corners = [&](int j) { return WAVE ? __builtin_amdgcn_readlane(cc, j) : sCon[first + j][0] & 63; };
    auto con_a = [&](int j) { return WAVE ? __builtin_amdgcn_readlane(ca0, j) : sCon[first + j][1]; };
    auto con_b = [&](int j) { return WAVE ? __builtin_amdgcn_readlane(cb0, j) : sCon[first + j][2]; };
    auto con_shift = [&](int j) { return WAVE ? __builtin_amdgcn_readlane(shift, j) : (sCon[first + j][0] >> 6) & 31; };
    auto con_sa = [&](int j) { return WAVE ? __builtin_amdgcn_readlane(sa3, j) : (sCon[first + j][0] >> 11) & 7; };
    auto con_sb = [&](int j) { return WAVE ? __builtin_amdgcn_readlane(sb3, j) : (sCon[first + j][0] >> 14) & 7; };
    const double *part = partial1 ? partial1 : cx.partial;
    Out *H = (Out *)(H1 ? H1 : cx.H), *S = (Out *)(H1 ? S1 : cx.S);
    const int64_t blk = block_index(e), blkT = block_mirror(e);
    const int64_t off = cx.bval_off[blk], offT = cx.bval_off[blkT], nnz = cx.nnz;
    const int64_t v = cx.brow[blk], w = cx.bcol[blk];
    const int bv = (int)(cx.dof_off[v + 1] - cx.dof_off[v]), bw = (int)(cx.dof_off[w + 1] - cx.dof_off[w]);
    const bool mirror = blk != blkT;
    const bool proj = NL && block_projected(e);
    const int dofs = bv + bw, nst = WAVE && proj && n_pfun * dofs <= kGatherStage ? n_pfun * dofs : 0;
    double2 *sF = sFs[NL && WAVE ? threadIdx.x >> 6 : 0];
    const int64_t v0 = cx.dof_off[v], w0 = cx.dof_off[w];
    for (int kn = 0; kn < (NL ? kps.nk : 1); ++kn) {
        if (NL && WAVE && nst > 0) {
            const double2 *fk = f + (int64_t)kn * n_pfun * n_dof;
            __builtin_amdgcn_wave_barrier();
            for (int i = lane; i < nst; i += 64) {
                const int J = i / dofs, d = i - J * dofs;
                sF[i] = fk[(int64_t)J * n_dof + (d < bv ? v0 + d : w0 + d - bv)];
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        for (int i = lane + GL * blockIdx.y; i < bv * bw; i += GL * gridDim.y) {
            const int sa = i / bw, sb = i - sa * bw;
            const int64_t o = off + i, oT = offT + (int64_t)sb * bv + sa;
            auto put = [&](int k, double hr, double hi, double sr, double si) {
                const int64_t b = (int64_t)k * nnz;
                if (NL && proj) {
                    double re = 0.0, im = 0.0;
                    auto add = [&](const double2 a, const double2 c, double h) {   // h a conj(c)
                        re += h * (a.x * c.x + a.y * c.y);
                        im += h * (a.y * c.x - a.x * c.y);
                    };
                    if (nst > 0) {
                        for (int J = 0; J < n_pfun; ++J) add(sF[J * dofs + sa], sF[J * dofs + bv + sb], pfun_h[J]);
                    } else {
                        const double2 *fk = f + (int64_t)k * n_pfun * n_dof;
                        for (int J = 0; J < n_pfun; ++J)
                            add(fk[(int64_t)J * n_dof + v0 + sa], fk[(int64_t)J * n_dof + w0 + sb], pfun_h[J]);
                    }
                    hr += re;
                    hi += im;
                }
                H[b + o] = out_value<DT>(hr, hi);
                if (mirror) H[b + oT] = out_value<DT>(hr, -hi);
                if (S) {
                    S[b + o] = out_value<DT>(sr, si);
                    if (mirror) S[b + oT] = out_value<DT>(sr, -si);
                }
            };
            // one element's value: hr + i hi, sr + i si before the phase
            auto value = [&](int j, double *h, double *s) -> bool {
                const int c = con_corners(j), ua = con_a(j), ub = con_b(j);
                const int a = local_of(p, nfs, nfe, c >> 3, sa, ua & 0xffff), b = local_of(p, nfs, nfe, c & 7, sb, ub & 0xffff);
                if (a < 0 || b < 0) return false;
                const double *t = part + con_base(j);
                const int64_t ab = entry_of(a, b);
                h[0] = t[ab];
                s[0] = t[ab + 256];
                if (BLOCH) {   // the imaginary rows follow the corner's real ones
                    const int ai = a >= nfe ? a + (ua >> 17) : -1, bi = b >= nfe ? b + (ub >> 17) : -1;
                    h[1] = s[1] = 0.0;
                    if (ai >= 0 && bi >= 0) {
                        const int64_t x = entry_of(ai, bi);
                        h[0] += t[x];
                        s[0] += t[x + 256];
                    }
                    if (bi >= 0) {
                        const int64_t x = entry_of(a, bi);
                        h[1] += t[x];
                        s[1] += t[x + 256];
                    }
                    if (ai >= 0) {
                        const int64_t x = entry_of(ai, b);
                        h[1] -= t[x];
                        s[1] -= t[x + 256];
                    }
                }
                return true;
            };
            if (!BLOCH && !wraps) {
                double hr = 0.0, sr = 0.0;
                for (int j = 0; j < ncon; ++j) {
                    double h[2], s[2];
                    if (value(j, h, s)) {
                        hr += h[0];
                        sr += s[0];
                    }
                }
                if (NL) put(kn, hr, 0.0, sr, 0.0);
                else
                    for (int k = 0; k < kps.nk; ++k) put(k, hr, 0.0, sr, 0.0);
                continue;
            }
            constexpr int NK = NL ? 1 : 4;   // k-points at a time
            for (int k0 = NL ? kn : 0; k0 < (NL ? kn + 1 : kps.nk); k0 += NK) {
                double hr[NK], hi[NK], sr[NK], si[NK];
#pragma unroll
                for (int u = 0; u < NK; ++u) hr[u] = hi[u] = sr[u] = si[u] = 0.0;
                for (int j = 0; j < ncon; ++j) {
                    double h[2], s[2];
                    if (!value(j, h, s)) continue;
                    int t = con_shift(j);
                    if (BLOCH) {
                        const int za = sa < nfs ? con_sa(j) : 0, zb = sb < nfs ? con_sb(j) : 0;
                        auto dn = [&](int d) { return ((zb >> d) & 1) - ((za >> d) & 1) + 1; };
                        t = dn(0) + 3 * dn(1) + 9 * dn(2);
                    }
#pragma unroll
                    for (int u = 0; u < NK; ++u) {
                        if (k0 + u >= kps.nk) break;
                        const double2 z = wraps ? sZ[(k0 + u) * 27 + t] : make_double2(1.0, 0.0);
                        hr[u] += z.x * h[0];
                        hi[u] += z.y * h[0];
                        sr[u] += z.x * s[0];
                        si[u] += z.y * s[0];
                        if (BLOCH) {
                            hr[u] -= z.y * h[1];
                            hi[u] += z.x * h[1];
                            sr[u] -= z.y * s[1];
                            si[u] += z.x * s[1];
                        }
                    }
                }
#pragma unroll
                for (int u = 0; u < NK; ++u)
                    if (k0 + u < kps.nk) put(k0 + u, hr[u], hi[u], sr[u], si[u]);
            }
        }
    }
}

hipError_t launch_gather(const CtxDev *ctxs, const int4 *list, const GatherSizes &sz, const double *partial, void *H, void *S,
                         const KPoints &kps, int out_dtype, bool bloch, const double2 *f, const double *pfun_h, int n_pfun,
                         int64_t n_dof, hipStream_t st) {
    const int n = sz.blocks - sz.small;
    // waves per block: until about 8192 are in flight (32 a CU), each with entries
    // (48 elements of 283 functions: 115 us with a wave per block, 22 with several;
    // element by element in eight launches 82)
    const int parts = n > 0 ? std::max(1, std::min((sz.max_entries + 63) / 64, 8192 / n)) : 1;
    auto go = [&](auto *k, auto *ks) {
        if (n > 0)
            k<<<dim3((n + 3) / 4, parts), 256, 0, st>>>(ctxs, list, n, partial, H, S, kps, f, pfun_h, n_pfun, n_dof);
        if (sz.small > 0)
            ks<<<(sz.small + 31) / 32, 256, 0, st>>>(ctxs, list + n, sz.small, partial, H, S, kps, f, pfun_h, n_pfun, n_dof);
        return hipGetLastError();
    };
    auto type = [&](auto bl, auto nl) {
        constexpr bool B = decltype(bl)::value, N = decltype(nl)::value;
        if (out_dtype == 0) return go(gather_kernel<0, B, N, 64>, gather_kernel<0, B, N, 8>);
        if (out_dtype == 1) return go(gather_kernel<1, B, N, 64>, gather_kernel<1, B, N, 8>);
        return go(gather_kernel<2, B, N, 64>, gather_kernel<2, B, N, 8>);
    };
    if (bloch) return f ? type(std::true_type(), std::true_type()) : type(std::true_type(), std::false_type());
    return f ? type(std::false_type(), std::true_type()) : type(std::false_type(), std::false_type());
}

}  // namespace pufe
