// Device-side table layouts shared by the host planner and the HIP kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pufe {

constexpr int kMaxFun = 64;       // enrichment functions on one element
constexpr int kMaxGroups = 32;    // (atom, descriptor) groups on one element
constexpr int kMaxNloc = 512;     // functions on one element
constexpr int kTile = 16;         // MFMA tile edge
constexpr int kBlockTiles = 4;    // tiles per row/column block of a work item
constexpr int kMaxGauss = 12;
constexpr int kMaxLevel = 8;
constexpr int kMaxRowChunks = 64; // enriched-row chunks of one partial work item
constexpr int kMaxProjCols = 64;  // projector columns reaching one element
constexpr int kBlockProjected = 1 << 26;   // assembly list entry: projectors couple the block
constexpr int kMaxPGroups = 32;   // projector-image groups reaching one element
// dynamic LDS a kernel may request: the 160 KiB of a CU minus room for the
// small static __shared__ variables some kernels also declare
constexpr size_t kMaxDynLds = 159 * 1024;

// One element: geometry index, function counts, table offsets and the BSR
// addresses of its 8x8 corner-vertex blocks.
struct ElemDev {
    int32_t nloc, nfe, nfun, ngrp;
    int32_t grp_off, edof_off;
    int32_t ijk[3];
    int32_t shifts;      // lattice shift bits of corner c at bits 3c..3c+2 (bit d = direction d)
    int32_t nchunk;      // K-chunks of the contraction
    int64_t leaf_off, leaf_end;
    int64_t part_base;   // first partial tile-pair slot
    int64_t blk[64];     // value offset of BSR block (vertex of corner ca, vertex of corner cb) at ca*8+cb
    int32_t bw[8];       // width of the block column of corner c (b_w of its vertex)
    int32_t pg_off, npg; // projector-image groups reaching the element
    int32_t ncol;        // projector columns (sum of 2l+1 over the groups)
    int32_t pf_nchunk;   // K-chunks of its projector coefficients (0: none)
    int64_t pf_base;     // first double of its projector-coefficient slots, F[chunk][col][npad]
    // moment form (FP64 contraction): K-chunks (0: the element runs the direct
    // kernels), 4-row tiles of its enrichment functions, first double of its
    // moment slots [chunk][task][kMomSlot], K-chunks of its classical part and
    // the first double of theirs [chunk][kMomFFSlot]
    int32_t mchunk, nt, fchunk;
    int64_t mom_base, ff_base;
    int32_t cs[9];       // first enriched entry of each corner, and their number
};

// Projector descriptor of one atom image that reaches an element: the 2l+1
// columns col0 .. col0 + 2l of the element's projector coefficients, the
// projector functions J0 .. J0 + 2l, the image centre and its lattice shift.
struct PGroupDev {
    double c[3];
    double a, rc;
    int32_t l, col0, J0, n[3];
};

// A nonlocal work item: one element, one range of its octree leaves, one row
// block of its local functions (tiles R0 .. R0 + nR - 1).
struct NlItemDev {
    int32_t elem, chunk, R0, nR;
    int64_t leaf_b, leaf_e;
};

// (atom, descriptor) group: 2l+1 functions with one radial part and the list
// of lattice images whose cutoff sphere reaches the element.  A tabulated
// radial (nspl > 0 intervals of width rc / nspl, a = nspl / rc) is the cubic
// on interval j = floor(a r) with coefficients spl[spl_off + 4 j + 0..3] in
// powers of tau = a r - j.
struct GroupDev {
    int32_t atom, desc, l, fbase, img_off, nimg, nspl, spl_off;
    double a, rc;   // a: Gaussian exponent (analytic) or intervals per bohr (tabulated)
};

// Serendipity elements (fe_order 3): the k-th (k = 0..3) corner whose bit d
// is clear, where edge 4 d + k along direction d starts.
static inline __host__ __device__ int serendipity_edge_corner(int d, int k) {
    const int low = k & ((1 << d) - 1);
    return low | ((k >> d) << (d + 1));
}

// Enriched local function: corner | element-function << 3 | vertex slot << 11
static inline __host__ __device__ int32_t edof_pack(int corner, int f, int slot) {
    return corner | (f << 3) | (slot << 11);
}

// Contribution of an element to a block of the assembly: its corners cv and cw are
// the block's vertices.  Assembly list entry of a block: the blocks (v, w) and
// (w, v) and its first contribution (32 bits unsigned each), and in w the problem,
// whether projectors couple the block, and the number of contributions (at most 8).
static inline __host__ __device__ int64_t contr_pack(int64_t elem, int cv, int cw) { return elem << 6 | cv << 3 | cw; }
static inline __host__ __device__ int64_t contr_elem(int64_t c) { return c >> 6; }
static inline __host__ __device__ int contr_corners(int64_t c) { return (int)(c & 63); }
static inline __host__ __device__ int4 block_pack(int64_t b, int64_t mirror, int64_t first, int n, bool projected) {
    int4 e;
    e.x = (int)(uint32_t)b;
    e.y = (int)(uint32_t)mirror;
    e.z = (int)(uint32_t)first;
    e.w = n << 27 | (projected ? kBlockProjected : 0);
    return e;
}
static inline __host__ __device__ int64_t block_index(const int4 &e) { return (int64_t)(uint32_t)e.x; }
static inline __host__ __device__ int64_t block_mirror(const int4 &e) { return (int64_t)(uint32_t)e.y; }
static inline __host__ __device__ int64_t block_first(const int4 &e) { return (int64_t)(uint32_t)e.z; }
static inline __host__ __device__ bool block_projected(const int4 &e) { return (e.w & kBlockProjected) != 0; }
static inline __host__ __device__ int block_count(const int4 &e) { return e.w >> 27; }

// A contraction work item: one element, one row block and one column block of
// 16x16 tiles, one range of octree leaves (a K-chunk).
struct ItemDev {
    int32_t elem, I0, nI, J0, nJ, chunk;
    int64_t leaf_b, leaf_e;
    int32_t ctx;         // problem of a batched launch (0 otherwise)
};

// A work item of the moment form: one element, one range of octree leaves and
// the wave tasks wave_task[tab & 0xffffff ..] (one per wave of the work group;
// planes per stage at bits 24..27, stage buffers at 28..29).  Items of the
// classical part have no tasks.
struct MomItemDev {
    int32_t elem, chunk, tab, ctx;
    int64_t leaf_b, leaf_e;
};

// Wave tasks of the moment form: role | index << 8 | second index << 20.  An
// element's moment slots are its energy quads, its gradient quads and its
// mixed groups, in that order; the index is the quad of 4x4 tile pairs or the
// group of 8 functions.
enum {
    MOM_IDLE = 0,
    MOM_E = 1,      // E of every x power and A of x^2
    MOM_BXY = 2,    // B_x and B_y
    MOM_A = 3,      // A of x^0 and x^1 (energy quad: index)
    MOM_BZ = 4,     // B_z (gradient quad: second index)
    MOM_A_BZ = 5,   // both
    MOM_F = 6       // mixed
};
constexpr int kMomSlot = 54 * 64;   // doubles of one task's moments
constexpr int kMomFFSlot = 320;     // doubles of the classical moments of one leaf range
static inline __host__ __device__ int mom_quads_ae(int nt) { return (nt * (nt + 1) / 2 + 3) / 4; }
static inline __host__ __device__ int mom_quads_b(int nt) { return (nt * nt + 3) / 4; }
static inline __host__ __device__ int mom_groups_f(int nt) { return (nt + 1) / 2; }
static inline __host__ __device__ int mom_slots(int nt) { return mom_quads_ae(nt) + mom_quads_b(nt) + mom_groups_f(nt); }

// Per-launch constants of the mesh and the rule.
struct KParams {
    double E[9];      // row d: a_d / n_d (element edge vector)
    double Jt[9];     // grad_x[c] = sum_d Jt[3c+d] dphi/dxi_d
    double jac;       // det of the reference-to-element map
    double gx[kMaxGauss], gw[kMaxGauss];   // base rule (n points)
    double rx[kMaxGauss], rw[kMaxGauss];   // reference rule of the error mode (nref points)
    int32_t n, n3, p, nfe, nfs, nref;
    int32_t mesh[3];
    // reference metric G = Jt^T Jt and its inverse, the scale of the stored
    // gradients against reference derivatives, and whether the cell is skewed
    double G[9], Gi[9], sd[3];
    int32_t skew;
    const double *spl;   // coefficients of the tabulated radials (device)
    // Bloch-periodic enrichment: the weight of every image entry at the
    // k-point of the launch, cos or sin(2 pi kappa.n) (null: periodic, all 1)
    const double *wimg;
};

// Tables and buffers of one problem, for launches that cover several problems
// (one per lattice constant of a sweep).
struct CtxDev {
    KParams kp;
    const ElemDev *elems;
    const GroupDev *groups;
    const double *img;
    const int32_t *edof;
    const uint32_t *leaves;
    const double *V;
    double *partial;
    double *mom;         // moment slots
    // block layout and the elements of every block (assembly)
    const int64_t *contr;
    const int32_t *brow, *bcol;
    const int64_t *bval_off, *dof_off;
    void *H, *S;
    int64_t nnz;
};

// Octree cell of the error-driven rule builder: element, leaf code, and the
// bit mask of the element's enrichment functions still tested on it.
struct CellDev {
    uint64_t mask;
    int32_t elem;
    uint32_t code;
    int32_t open;   // 1 while the cell may still split
    int32_t pad;
};

// Leaf code: level in bits 27..30, cell coordinates in 9-bit fields.
static inline __host__ __device__ uint32_t leaf_pack(int lev, int c1, int c2, int c3) {
    return (uint32_t)c1 | ((uint32_t)c2 << 9) | ((uint32_t)c3 << 18) | ((uint32_t)lev << 27);
}

}  // namespace pufe
