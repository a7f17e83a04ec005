// C ABI of the PUFE assembly library (declared in include/pufe.h).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "../../include/pufe.h"
#include "aq_error.hpp"
#include "adjoint.hpp"
#include "backward.hpp"
#include "bloch.hpp"
#include "forms.hpp"
#include "gather.hpp"
#include "kernels.hpp"
#include "moments.hpp"
#include "nonlocal.hpp"
#include "plan.hpp"
#include "scf.hpp"

using namespace pufe;

namespace {

template <class T>
struct DevBuf {
    T *p = nullptr;
    size_t n = 0;
    DevBuf() = default;
    DevBuf(const DevBuf &) = delete;
    DevBuf &operator=(const DevBuf &) = delete;
    ~DevBuf() { release(); }
    void release() {
        if (p) (void)hipFree(p);
        p = nullptr;
        n = 0;
    }
    hipError_t alloc(size_t count) {
        release();
        if (count == 0) count = 1;
        hipError_t e = hipMalloc((void **)&p, count * sizeof(T));
        if (e == hipSuccess) n = count;
        else p = nullptr;
        return e;
    }
    // upload, with no buffer at all for an empty list (which no launch reads)
    hipError_t upload_list(const std::vector<T> &v, hipStream_t st) {
        if (!v.empty()) return upload(v, st);
        release();
        return hipSuccess;
    }
    hipError_t upload(const std::vector<T> &v, hipStream_t st) {
        hipError_t e = alloc(v.size());
        if (e != hipSuccess || v.empty()) return e;
        e = hipMemcpyAsync(p, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice, st);
        if (e != hipSuccess) return e;
        return hipStreamSynchronize(st);
    }
};

}  // namespace

struct pufe_ctx {
    int device = 0;
    std::string err;
    bool have_problem = false, have_setup = false;
    // what pufe_setup makes for the problem is there; without have_setup the rule and its
    // plan are not (a call that replaces them failed midway), pufe_set_rule may give them
    bool have_tables = false;
    Problem prob;
    Plan plan;
    int64_t n_leaves = 0, n_qp = 0;
    std::vector<int64_t> leaf_off_h;
    std::vector<ItemDev> items, items_split;
    // wide work items: the row and column blocks of elements of more than
    // kWholeMaxTiles tiles, for the 8-wave kernel (wide_tiles = 0: none, those
    // elements go to the narrow kernel)
    std::vector<ItemDev> items_wide;
    int wide_tiles = kWideTiles, max_rows_wide = 16, max_item_leaves_wide = 1;
    size_t lds_wide = 0;
    size_t lds = 0;
    int max_rows = 16, max_rows_split = 16, max_item_leaves_split = 1;
    int64_t part_slots = 0;
    double tune_items = 4096.0;
    int tune_block = kBlockTiles;
    bool tuned = false;             // item plan and stage length chosen by pufe_tune
    int contract_q = 24;            // points per LDS stage of the FP64 contraction (16, 24 or 32)
    int max_item_leaves = 1;
    // bumped whenever the device tables or work items are rebuilt (problem,
    // setup, tuner): a batch created earlier refuses to run on a newer plan
    uint64_t plan_gen = 0;
    DevBuf<ElemDev> d_elems;
    DevBuf<GroupDev> d_groups;
    DevBuf<double> d_img, d_pos, d_partial;
    DevBuf<double> d_spl;           // coefficients of the tabulated radials
    DevBuf<int32_t> d_edof, d_leaf_elem, d_brow, d_bcol;
    DevBuf<int64_t> d_contr;
    DevBuf<int4> d_blocks;
    std::vector<int2> reduce;       // (element, tile pair) of every element with several K-chunks
    std::vector<int2> reduce_f64;   // those of the elements on the direct FP64 kernels
    DevBuf<int2> d_reduce, d_reduce_f64;
    // moment form (FP64): items of the 4- and 8-wave work groups with their
    // costs, the wave tasks they point into, chunk sums and expansion lists
    // (index 2: the items of the classical part)
    std::vector<MomItemDev> mom_items[3];
    std::vector<double> mom_cost[3];
    std::vector<int32_t> mom_tasks;
    std::vector<int4> mom_reduce, mom_expand;
    size_t mom_lds[3] = {0, 0, 0};
    int64_t mom_doubles = 0;
    DevBuf<MomItemDev> d_mom_items[3];
    DevBuf<int32_t> d_mom_tasks;
    DevBuf<int4> d_mom_reduce, d_mom_expand;
    DevBuf<double> d_mom;
    DevBuf<CtxDev> d_self;          // this problem's tables, for the kernels that take a list of problems; [1] with
                                    // the allocation-free entry's moment slots
    DevBuf<double> d_mom_na;        // these slots, where its workspace has no room for them
    // the moment forms' device memory: the caller's limit (negative: none), and
    // whether the forward plan has given the form up for lack of it
    int64_t mom_limit = -1;
    bool mom_off = false;
    double planned_items = 0.0;     // what plan_items last planned for
    int planned_block = 0;
    DevBuf<uint32_t> d_leaves;
    DevBuf<int64_t> d_leaf_count, d_leaf_off, d_bval_off, d_dof_off;
    DevBuf<ItemDev> d_items, d_items_split, d_items_wide;
    // adjoint
    // the adjoint's blocks, its choice of form, its direct kernels' items
    bool have_bw = false, have_adj = false, have_bw_direct = false;
    std::vector<ItemDev> bw_items, bw_items_wide;   // elements of <= 80 functions, and the rest
    size_t bw_lds = 0, bw_lds_wide = 0;
    // FP64 adjoint in moment form: items by 4 and 8 waves, or none
    std::vector<MomItemDev> adj_items[2];
    size_t adj_lds[2] = {0, 0};
    DevBuf<MomItemDev> d_adj_items[2];
    std::vector<int4> adj_fold;
    DevBuf<int4> d_adj_fold;
    DevBuf<int64_t> d_adj_base, d_adj_ptr, d_adj_slots;
    DevBuf<double> d_adj_lam, d_adj_Qt, d_adj_f;
    DevBuf<ItemDev> d_bw_items, d_bw_items_wide;
    DevBuf<int64_t> d_pt_off, d_atom_ptr, d_atom_slots;
    DevBuf<double> d_Pt, d_fP, d_fQ;
    // separable nonlocal term
    std::vector<NlItemDev> nl_items;
    std::vector<int32_t> nl_elems;
    int64_t nl_doubles = 0;
    size_t nl_lds = 0;
    int nl_planes = 0;              // planes per stage of the projectors' moment form, 0: direct
    DevBuf<NlItemDev> d_nl_items;
    DevBuf<PGroupDev> d_pgroups;
    DevBuf<double> d_Fp, d_pfun_h;
    DevBuf<int64_t> d_dof_el_off;
    DevBuf<int2> d_dof_el;
    DevBuf<int32_t> d_nl_elems;
    DevBuf<double2> d_nlf;
    // Bloch-periodic enrichment: image shifts and kinds, the per-k image
    // weights, the partner table of the enriched entries
    DevBuf<int32_t> d_img_nk, d_bpart;
    DevBuf<double> d_wimg;
    // self-consistent field pieces: per-element load sums, the classical FE
    // blocks of the stiffness matrix, the FE integrals m_i, CG workspace
    DevBuf<double> d_fe_be, d_Kfe, d_mfe, d_fe_ones, d_cg, d_dot;
    DevBuf<CgState> d_cg_state;
    DevBuf<int64_t> d_brow_ptr;
    bool have_poisson = false;
    double m_sum = 0.0;
    // timing
    bool timing = false;
    std::vector<std::pair<hipEvent_t, hipEvent_t>> ev[5];
    ~pufe_ctx() { clear_events(); }
    void clear_events() {
        for (auto &v : ev) {
            for (auto &pr : v) {
                (void)hipEventDestroy(pr.first);
                (void)hipEventDestroy(pr.second);
            }
            v.clear();
        }
    }
};

// Bracket the launches enqueued between begin() and end() with events when
// timing is on.
struct TimedRegion {
    pufe_ctx *c;
    int slot;
    hipStream_t st;
    hipEvent_t a = nullptr, b = nullptr;
    TimedRegion(pufe_ctx *c_, int s, hipStream_t st_) : c(c_), slot(s), st(st_) {
        if (!c->timing || slot < 0) return;
        if (hipEventCreate(&a) != hipSuccess || hipEventCreate(&b) != hipSuccess) { a = b = nullptr; return; }
        (void)hipEventRecord(a, st);
    }
    ~TimedRegion() {
        if (!a) return;
        (void)hipEventRecord(b, st);
        c->ev[slot].push_back({a, b});
    }
};

static int fail(pufe_ctx *c, int code, const std::string &msg) {
    if (c) c->err = msg;
    return code;
}

static int hipfail(pufe_ctx *c, hipError_t e, const char *where) {
    int code = (e == hipErrorOutOfMemory) ? PUFE_ERR_OOM : PUFE_ERR_HIP;
    return fail(c, code, std::string(where) + ": " + hipGetErrorString(e));
}

// The problem's device tables, without the buffers of a call.
static CtxDev tables_of(const pufe_ctx *c) {
    CtxDev d{};
    d.kp = c->plan.kp;
    d.elems = c->d_elems.p;
    d.groups = c->d_groups.p;
    d.img = c->d_img.p;
    d.edof = c->d_edof.p;
    d.leaves = c->d_leaves.p;
    d.partial = c->d_partial.p;
    d.mom = c->d_mom.p;
    d.contr = c->d_contr.p;
    d.brow = c->d_brow.p;
    d.bcol = c->d_bcol.p;
    d.bval_off = c->d_bval_off.p;
    d.dof_off = c->d_dof_off.p;
    d.nnz = c->plan.nnz;
    return d;
}

// Workspace of the allocation-free entry: the partial tiles, behind the room
// that its size limit counts for a phase table.
static constexpr size_t kNoallocTiles = (sizeof(double2) * kMaxKPerLaunch * 27 + 255) / 256 * 256;
static size_t noalloc_bytes(const pufe_ctx *c) { return kNoallocTiles + (size_t)c->part_slots * 512 * sizeof(double); }

#define CHECK_HIP(ctx, x, where)                          \
    do {                                                  \
        hipError_t e_ = (x);                              \
        if (e_ != hipSuccess) return hipfail(ctx, e_, where); \
    } while (0)

extern "C" {

const char *pufe_error_string(int code) {
    switch (code) {
        case PUFE_OK: return "ok";
        case PUFE_ERR_INVALID_ARG: return "invalid argument";
        case PUFE_ERR_UNSUPPORTED: return "unsupported";
        case PUFE_ERR_OOM: return "out of device memory";
        case PUFE_ERR_HIP: return "HIP runtime error";
        case PUFE_ERR_STATE: return "call out of order";
        default: return "unknown error";
    }
}

const char *pufe_last_error_message(const pufe_ctx *ctx) {
    if (!ctx) return "no context";
    return ctx->err.c_str();
}

int pufe_create(pufe_ctx **out, int device) {
    if (!out) return PUFE_ERR_INVALID_ARG;
    if (device < 0) return PUFE_ERR_INVALID_ARG;
    pufe_ctx *c = new (std::nothrow) pufe_ctx();
    if (!c) return PUFE_ERR_OOM;
    c->device = device;
    *out = c;
    return PUFE_OK;
}

int pufe_destroy(pufe_ctx *ctx) {
    if (!ctx) return PUFE_ERR_INVALID_ARG;
    if (ctx->d_leaf_off.p) (void)hipSetDevice(ctx->device);   // it has device buffers
    delete ctx;
    return PUFE_OK;
}

int pufe_set_problem(pufe_ctx *ctx, const double lattice[9], const int mesh[3], int fe_order, int n_atoms,
                     const double *pos, const int *species, int n_enr, const pufe_enrichment *enr,
                     const pufe_quad *quad) {
    if (!ctx) return PUFE_ERR_INVALID_ARG;
    if (!lattice || !mesh || !quad || n_atoms < 0 || n_enr < 0 || (n_atoms > 0 && (!pos || !species)) ||
        (n_enr > 0 && !enr))
        return fail(ctx, PUFE_ERR_INVALID_ARG, "null pointer or negative count");
    Problem pr;
    std::memcpy(pr.lat, lattice, sizeof pr.lat);
    std::memcpy(pr.mesh, mesh, sizeof pr.mesh);
    pr.p = fe_order;
    pr.pos.assign(pos, pos + 3 * (size_t)n_atoms);
    pr.species.assign(species, species + n_atoms);
    pr.enr.assign(enr, enr + n_enr);
    pr.radial.assign(n_enr, {});
    for (int k = 0; k < n_enr; ++k) {   // keep a copy of the samples, never the caller's pointer
        if (enr[k].radial_kind == 1) {
            if (!enr[k].radial || enr[k].n_radial < 0 || enr[k].n_radial > 4096)
                return fail(ctx, PUFE_ERR_INVALID_ARG, "a tabulated radial needs 4..4096 samples");
            pr.radial[k].assign(enr[k].radial, enr[k].radial + enr[k].n_radial);
        }
        pr.enr[k].radial = nullptr;
        pr.enr[k].n_radial = (int)pr.radial[k].size();
    }
    pr.quad = *quad;
    for (double v : pr.pos)
        if (!std::isfinite(v)) return fail(ctx, PUFE_ERR_INVALID_ARG, "non-finite atom position");
    Plan pl;
    std::string err;
    int rc = build_plan(pr, pl, err);
    if (rc != PUFE_OK) return fail(ctx, rc, err);
    ctx->prob = std::move(pr);
    ctx->plan = std::move(pl);
    ctx->have_problem = true;
    ctx->have_setup = ctx->have_tables = false;
    ctx->have_bw = ctx->have_adj = ctx->have_bw_direct = false;
    ctx->n_leaves = ctx->n_qp = 0;
    ++ctx->plan_gen;
    return PUFE_OK;
}

int pufe_set_projectors(pufe_ctx *ctx, int n, const pufe_projector *proj) {
    if (!ctx) return PUFE_ERR_INVALID_ARG;
    if (!ctx->have_problem) return fail(ctx, PUFE_ERR_STATE, "pufe_set_problem must come first");
    if (ctx->have_tables) return fail(ctx, PUFE_ERR_STATE, "projectors are set before pufe_setup");
    if (n < 0 || (n > 0 && !proj)) return fail(ctx, PUFE_ERR_INVALID_ARG, "null pointer or negative count");
    Problem pr = ctx->prob;
    pr.proj.assign(proj, proj + n);
    Plan pl;
    std::string err;
    int rc = build_plan(pr, pl, err);
    if (rc != PUFE_OK) return fail(ctx, rc, err);
    ctx->prob = std::move(pr);
    ctx->plan = std::move(pl);
    ++ctx->plan_gen;
    return PUFE_OK;
}

int pufe_set_enrichment_phase(pufe_ctx *ctx, int form) {
    if (!ctx) return PUFE_ERR_INVALID_ARG;
    if (!ctx->have_problem) return fail(ctx, PUFE_ERR_STATE, "pufe_set_problem must come first");
    if (ctx->have_tables) return fail(ctx, PUFE_ERR_STATE, "the enrichment form is set before pufe_setup");
    if (form != PUFE_ENR_PERIODIC && form != PUFE_ENR_BLOCH)
        return fail(ctx, PUFE_ERR_INVALID_ARG, "unknown enrichment form");
    Problem pr = ctx->prob;
    pr.enr_phase = form;
    Plan pl;
    std::string err;
    int rc = build_plan(pr, pl, err);
    if (rc != PUFE_OK) return fail(ctx, rc, err);
    ctx->prob = std::move(pr);
    ctx->plan = std::move(pl);
    ++ctx->plan_gen;
    return PUFE_OK;
}

// Split each element's contraction into K-chunks (ranges of leaves) of about
// equal MFMA work; the chunking fixes the layout of the partial tiles and does
// not depend on how the tile pairs of a chunk are grouped into work items.  It is
// that of the split precisions for every element; in FP64 an element in moment form
// writes its first slot only.
static void plan_chunks(pufe_ctx *c, double target_items) {
    Plan &pl = c->plan;
    const int n3 = pl.kp.n3;
    double total = 0;
    for (const ElemDev &el : pl.elems) {
        const int T = (el.nloc + 15) / 16;
        total += (double)T * (T + 1) / 2 * n3 * (el.leaf_end - el.leaf_off);
    }
    const double target = std::max(total / target_items, 1.0);
    int64_t base = 0;
    for (ElemDev &el : pl.elems) {
        const int T = (el.nloc + 15) / 16;
        const int64_t P = (int64_t)T * (T + 1) / 2, nleaf = el.leaf_end - el.leaf_off;
        int64_t nch = (int64_t)std::llround((double)nleaf * n3 * P / target);
        nch = std::max<int64_t>(1, std::min<int64_t>(nch, nleaf));
        el.nchunk = (int32_t)nch;
        el.part_base = base;
        base += nch * P;
    }
    c->part_slots = base;
    c->reduce.clear();
    for (int64_t e = 0; e < pl.nel; ++e) {
        const ElemDev &el = pl.elems[e];
        const int T = (el.nloc + 15) / 16;
        if (el.nchunk > 1)
            for (int p = 0; p < T * (T + 1) / 2; ++p) c->reduce.push_back(make_int2((int)e, p));
    }
    c->reduce_f64.clear();
    for (const int2 &r : c->reduce)
        if (pl.elems[r.x].mchunk == 0) c->reduce_f64.push_back(r);
}

// ---- moment form

// SIMD cycles per quadrature point of the wave tasks of an element (MFMA 17,
// FP64 VALU 6, as measured beside each other on two waves per SIMD): the x
// sums per line of n points, the y and z sums per line and per plane; fill:
// the enrichment functions, once per work group.
struct MomCost {
    double e, a, bxy, bz, f, ff, fill;
};
static MomCost mom_cost_of(const Plan &pl, const ElemDev &el) {
    const int n = pl.kp.n;
    const double k = std::ceil(n / 4.0) / n, line = 6.0 / n, plane = 6.0 / (n * n);
    MomCost m;
    m.e = k * (13 * 17 + 9 * 6) + 12 * line + 36 * plane;
    m.a = k * (2 * 17 + 6) + 6 * line + 18 * plane;
    m.bxy = k * (5 * 17 + 2 * 6) + 12 * line + 36 * plane;
    m.bz = k * (3 * 17 + 2 * 6) + 9 * line + 18 * plane;
    m.f = (10 * 17 + 4 * 6) / 4.0 + 40 * plane;
    m.ff = (2 * 17 + 4 * 6) / 4.0;
    m.fill = 0.0;
    for (int g = 0; g < el.ngrp; ++g) m.fill += (70 + 14 * (2 * pl.groups[el.grp_off + g].l + 1)) * 6.0 / 64.0;
    return m;
}
static double mom_cost_total(const MomCost &m, int nt, int items) {
    return mom_quads_ae(nt) * (m.e + m.a) + mom_quads_b(nt) * (m.bxy + m.bz) + mom_groups_f(nt) * m.f + items * m.fill;
}

// Waves per work group of the enriched part: elements of up to 12 functions
// take 4-wave groups, two per CU, the others 8-wave groups with twice the
// tasks to each evaluation of the enrichment functions.
static int mom_waves(int nt) { return nt <= 3 ? 4 : 8; }

// Wave tasks of an element of nt row tiles in nw-wave work groups, appended to
// `out`; returns the work groups per K-chunk.  The overlap moments of x^0
// and x^1 and the B_z moments (18 sums each) share a wave.  Tasks go, longest first, to the
// least loaded SIMD (waves w and w + 4 of a work group); 4-wave groups come in
// four rotations (4 entries each), so that two groups on one CU put their
// longest task on different SIMDs.
static int mom_wave_tasks(int nt, int nw, const MomCost &m, std::vector<int32_t> &out) {
    std::vector<std::pair<double, int32_t>> tasks;
    const int qa = mom_quads_ae(nt), qb = mom_quads_b(nt);
    for (int i = 0; i < qa; ++i) tasks.push_back({m.e, MOM_E | (i << 8)});
    for (int i = 0; i < qb; ++i) tasks.push_back({m.bxy, MOM_BXY | (i << 8)});
    for (int i = 0; i < mom_groups_f(nt); ++i) tasks.push_back({m.f, MOM_F | (i << 8)});
    for (int i = 0; i < std::max(qa, qb); ++i)   // qa <= qb for every nt
        tasks.push_back(i < qa ? std::make_pair(m.a + m.bz, (int32_t)(MOM_A_BZ | (i << 8) | (i << 20)))
                               : std::make_pair(m.bz, (int32_t)(MOM_BZ | (i << 20))));
    std::stable_sort(tasks.begin(), tasks.end(),
                     [](const std::pair<double, int32_t> &a, const std::pair<double, int32_t> &b) { return a.first > b.first; });
    const int items = ((int)tasks.size() + nw - 1) / nw, cap = nw / 4, bins = 4 * items;
    std::vector<double> load(bins, 0.0);
    std::vector<int> used(bins, 0);
    std::vector<int32_t> t((size_t)nw * items, MOM_IDLE);
    for (const auto &k : tasks) {
        int best = -1;
        for (int b = 0; b < bins; ++b)
            if (used[b] < cap && (best < 0 || load[b] < load[best])) best = b;
        t[(size_t)nw * (best / 4) + best % 4 + 4 * used[best]] = k.second;
        load[best] += k.first;
        ++used[best];
    }
    for (int i = 0; i < items; ++i)
        for (int r = 0; r < (nw == 4 ? 4 : 1); ++r)
            for (int w = 0; w < nw; ++w) out.push_back(t[(size_t)nw * i + (w + r) % nw]);
    return items;
}

// Which elements run in moment form, their K-chunks, slots and work items.
static void plan_moments(pufe_ctx *c) {
    Plan &pl = c->plan;
    const int n = pl.kp.n, p = pl.kp.p;
    for (int k = 0; k < 3; ++k) {
        c->mom_items[k].clear();
        c->mom_cost[k].clear();
        c->mom_lds[k] = 0;
    }
    c->mom_tasks.clear();
    c->mom_reduce.clear();
    c->mom_expand.clear();
    c->mom_doubles = 0;
    for (ElemDev &el : pl.elems) {
        el.mchunk = el.fchunk = 0;
        el.mom_base = el.ff_base = 0;
        el.nt = (el.nfun + 3) / 4;
    }
    if (c->mom_off || p > 2) return;   // the serendipity functions stay with the direct kernels
    int nimg = 0;
    for (const ElemDev &el : pl.elems)
        if (el.ngrp > 0) {
            const GroupDev &g = pl.groups[el.grp_off + el.ngrp - 1];
            nimg = std::max(nimg, g.img_off + g.nimg - pl.groups[el.grp_off].img_off);
        }
    // per number of row tiles: first wave task, work groups per chunk, stage
    struct Kind {
        int tab = -1, items = 0;
        MomStage st{0, 0, 0};
    };
    std::vector<Kind> kinds(kMaxFun / 4 + 1);
    FormModel model;
    model.el.resize(pl.nel);
    model.n3 = pl.kp.n3;
    model.nfun = pl.max_nfun;
    model.nimg = pl.max_img;
    const bool general = !pl.spl.empty() || pl.bloch;
    model.moment[0] *= pl.kp.skew ? 1.30 : (general ? 1.08 : 1.0);
    model.moment[1] *= pl.kp.skew ? 1.73 : (general ? 1.08 : 1.0);
    std::vector<char> able(pl.nel, 0), none(pl.nel, 0);
    double work = 0.0;
    for (int64_t e = 0; e < pl.nel; ++e) {
        const ElemDev &el = pl.elems[e];
        const MomCost m = mom_cost_of(pl, el);
        Kind &kd = kinds[el.nt];
        if (el.nt > 0 && kd.tab < 0) {
            kd.st = mom_stage(el.nt, nimg, n, p, mom_waves(el.nt));
            kd.tab = (int)c->mom_tasks.size();
            kd.items = mom_wave_tasks(el.nt, mom_waves(el.nt), m, c->mom_tasks);
        }
        able[e] = el.nt == 0 || kd.st.planes > 0;
        FormElem &f = model.el[e];
        f.leaves = (double)(el.leaf_end - el.leaf_off);
        f.pts = f.leaves * pl.kp.n3;
        f.fill = m.fill;
        f.per_point = el.nt > 0 ? mom_cost_total(m, el.nt, kd.items) : 0.0;
        f.ff = m.ff;
        f.nloc = el.nloc;
        f.nt = el.nt;
        f.nfun = el.nfun;
        f.tiles = (el.nloc + 15) / 16;
        f.pairs = 0.5 * f.tiles * (f.tiles + 1.0);
        f.items = kd.items;
        f.stages = kd.st.planes > 0 ? (n + kd.st.planes - 1) / kd.st.planes : 0;
        f.buffers = kd.st.buffers;
        work += f.pairs * f.pts;
    }
    for (FormElem &f : model.el)   // the default K-chunks of the direct kernels, whatever the tuner has chosen
        f.chunks = std::max(1.0, std::min(f.leaves, std::round(f.pairs * f.pts * 4096.0 / std::max(work, 4096.0))));
    // every element that can, those whose own work is less that way, or none:
    // the fastest by the model, the direct kernels unless another is faster by 6 %
    // (measured over the 360 problems: no choice but four costs more than 2 % over
    // the direct kernels, the worst 13 %; without that margin eleven and 32 %)
    std::vector<char> some(pl.nel, 0);
    const double d = model.dur(able);
    for (int64_t e = 0; e < pl.nel; ++e) some[e] = able[e] && model.cheaper(model.el[e], d);
    const std::vector<char> *best = &none;
    double t = 0.94 * model.time(none);
    for (const std::vector<char> *m : {&able, &some}) {
        if (std::find(m->begin(), m->end(), (char)1) == m->end()) continue;
        const double tm = model.time(*m);
        if (tm < t) {
            t = tm;
            best = m;
        }
    }
    if (best == &none) {
        c->mom_tasks.clear();
        return;
    }
    std::vector<double> cost(pl.nel, 0.0);
    double total = 0.0, fe_cost = 0.0;
    for (int64_t e = 0; e < pl.nel; ++e) {
        if (!(*best)[e]) continue;
        const FormElem &f = model.el[e];
        pl.elems[e].mchunk = 1;
        fe_cost = f.ff;
        cost[e] = f.per_point * f.pts;
        total += cost[e] + f.ff * f.pts;
    }
    // chunks: about four rounds of work groups over the chip, none shorter
    // than 40,000 cycles (the start of a work group and its moments' stores)
    const double dur = std::max(total / (1024.0 * 4.0), 40000.0);
    for (int64_t e = 0; e < pl.nel; ++e) {
        ElemDev &el = pl.elems[e];
        if (el.mchunk == 0) continue;
        const Kind &kd = kinds[el.nt];
        const int w = mom_waves(el.nt) == 4 ? 0 : 1, slots = mom_slots(el.nt), nw = w ? 8 : 4;
        const int64_t nleaf = el.leaf_end - el.leaf_off;
        auto chunks = [&](double co) {
            return std::max<int64_t>(1, std::min<int64_t>(nleaf, (int64_t)std::ceil(co / dur)));
        };
        auto add = [&](int list, int64_t ch, int64_t nch, int tab, double co) {
            MomItemDev it{};
            it.elem = (int32_t)e;
            it.chunk = (int32_t)ch;
            it.leaf_b = el.leaf_off + ch * nleaf / nch;
            it.leaf_e = el.leaf_off + (ch + 1) * nleaf / nch;
            it.tab = tab;
            c->mom_items[list].push_back(it);
            c->mom_cost[list].push_back(co / nch);
        };
        if (el.nt > 0) {
            const double item = cost[e] / kd.items / (w ? 4.0 : 2.0);
            const int64_t nch = chunks(item);
            el.mchunk = (int32_t)nch;
            el.mom_base = c->mom_doubles;
            c->mom_doubles += nch * slots * (int64_t)kMomSlot;
            c->mom_lds[w] = std::max(c->mom_lds[w], kd.st.lds);
            for (int64_t ch = 0; ch < nch; ++ch)
                for (int i = 0; i < kd.items; ++i) {
                    const int k = (int)c->mom_items[w].size();
                    const int off = w ? nw * i : 4 * (4 * i + ((k ^ (k >> 3) ^ (k >> 5) ^ (k >> 8)) & 3));
                    add(w, ch, nch, (kd.tab + off) | (kd.st.planes << 24) | (kd.st.buffers << 28), item);
                }
            if (nch > 1) {
                const int qe = mom_quads_ae(el.nt) + mom_quads_b(el.nt);
                for (int s = 0; s < slots; ++s) c->mom_reduce.push_back(make_int4((int)e, s, (s < qe ? 54 : 40) * 64, 0));
            }
        }
        // the classical part: a few leaves per wave (each leaf is a chain of
        // planes, bound by latency)
        const double fe = fe_cost * pl.kp.n3 * (double)nleaf / 2.0;
        el.fchunk = (int32_t)((nleaf + 15) / 16);
        el.ff_base = c->mom_doubles;
        c->mom_doubles += el.fchunk * (int64_t)kMomFFSlot;
        for (int64_t ch = 0; ch < el.fchunk; ++ch) add(2, ch, el.fchunk, 0, fe);
        for (int q = 0; q < mom_quads_ae(el.nt); ++q) c->mom_expand.push_back(make_int4((int)e, MOM_X_ENR, q, 0));
        for (int q = 0; 2 * q < el.nfun; ++q) c->mom_expand.push_back(make_int4((int)e, MOM_X_MIXED, q, 0));
        c->mom_expand.push_back(make_int4((int)e, MOM_X_FE, 0, 0));
    }
    for (int w = 0; w < 3; ++w) {   // longest first
        std::vector<size_t> order(c->mom_items[w].size());
        for (size_t i = 0; i < order.size(); ++i) order[i] = i;
        std::stable_sort(order.begin(), order.end(), [&](size_t a, size_t b) { return c->mom_cost[w][a] > c->mom_cost[w][b]; });
        std::vector<MomItemDev> it;
        std::vector<double> co;
        for (size_t i : order) {
            it.push_back(c->mom_items[w][i]);
            co.push_back(c->mom_cost[w][i]);
        }
        c->mom_items[w].swap(it);
        c->mom_cost[w].swap(co);
    }
}

static int upload_moments(pufe_ctx *ctx, hipStream_t st);

// Whether a moment form may take `doubles` of device memory: within the caller's
// limit, and at most half of what is free, so that a problem whose tables fit with
// the direct kernels keeps room for its caller's matrices.
static bool moments_fit(const pufe_ctx *c, int64_t doubles) {
    const uint64_t bytes = (uint64_t)doubles * sizeof(double);
    if (c->mom_limit >= 0) return bytes <= (uint64_t)c->mom_limit;
    size_t avail = 0, total = 0;
    if (hipMemGetInfo(&avail, &total) != hipSuccess) {
        (void)hipGetLastError();
        return true;
    }
    return bytes <= avail / 2;
}

// Work items (row block x column block of 16x16 tiles x K-chunk), largest
// MFMA work first.  sel: 0 every element (the split kernels); the elements on
// the direct FP64 kernels: 1 those of at most kWholeMaxTiles tiles, 2 the
// others, 3 all.
static std::vector<ItemDev> make_items(const pufe_ctx *c, int block_tiles, int *max_rows, int *max_leaves,
                                       int sel = 0) {
    const Plan &pl = c->plan;
    std::vector<ItemDev> items;
    std::vector<double> cost;
    for (int64_t e = 0; e < pl.nel; ++e) {
        const ElemDev &el = pl.elems[e];
        const int T = (el.nloc + 15) / 16;
        if ((sel == 1 && T > kWholeMaxTiles) || (sel == 2 && T <= kWholeMaxTiles) || (sel > 0 && el.mchunk > 0)) continue;
        // up to 5 tiles fit one diagonal block (15 tile pairs over 4 waves)
        const int bt = (T <= 5 && block_tiles >= 4) ? T : block_tiles;
        const int nb = (T + bt - 1) / bt;
        const int64_t nleaf = el.leaf_end - el.leaf_off, nch = el.nchunk;
        for (int64_t ch = 0; ch < nch; ++ch) {
            const int64_t lb = el.leaf_off + ch * nleaf / nch, le = el.leaf_off + (ch + 1) * nleaf / nch;
            for (int bj = 0; bj < nb; ++bj)
                for (int bi = 0; bi <= bj; ++bi) {
                    ItemDev it{};
                    it.elem = (int32_t)e;
                    it.I0 = bi * bt;
                    it.nI = std::min(bt, T - it.I0);
                    it.J0 = bj * bt;
                    it.nJ = std::min(bt, T - it.J0);
                    it.chunk = (int32_t)ch;
                    it.leaf_b = lb;
                    it.leaf_e = le;
                    const int pairs = bi == bj ? it.nI * (it.nI + 1) / 2 : it.nI * it.nJ;
                    items.push_back(it);
                    cost.push_back((double)pairs * (le - lb));
                }
        }
    }
    std::vector<size_t> order(items.size());
    for (size_t i = 0; i < order.size(); ++i) order[i] = i;
    std::stable_sort(order.begin(), order.end(), [&](size_t a, size_t b) { return cost[a] > cost[b]; });
    std::vector<ItemDev> sorted;
    sorted.reserve(order.size());
    int rows = 16, leaves = 1;
    for (size_t i : order) {
        sorted.push_back(items[i]);
        rows = std::max(rows, 16 * (items[i].I0 == items[i].J0 ? items[i].nI : items[i].nI + items[i].nJ));
        leaves = std::max(leaves, (int)(items[i].leaf_e - items[i].leaf_b));
    }
    *max_rows = rows;
    if (max_leaves) *max_leaves = leaves;
    return sorted;
}

static void plan_items(pufe_ctx *c, double target_items, int block_tiles, bool moments = true) {
    c->mom_off = !moments;
    c->planned_items = target_items;
    c->planned_block = block_tiles;
    plan_moments(c);
    plan_chunks(c, target_items);
    const int nfun = std::max(c->plan.max_nfun, 1);
    const int n3 = c->plan.kp.n3;
    // wide items first: tile blocks of wide_tiles (fewer if the stage does
    // not fit in LDS); without them every element goes to the narrow kernel
    c->items_wide.clear();
    bool wide = false;
    for (int b = c->wide_tiles; b >= 2; --b) {
        c->items_wide = make_items(c, b, &c->max_rows_wide, &c->max_item_leaves_wide, 2);
        c->lds_wide = contract_wide_lds_bytes(c->max_rows_wide, nfun, c->plan.max_img, c->max_item_leaves_wide, n3);
        if (c->lds_wide <= kMaxDynLds) {
            wide = true;
            break;
        }
    }
    if (!wide) c->items_wide.clear();
    // the FP64 stage double-buffers the rows of an item: use the largest
    // tile block (and stage length) whose buffers fit in LDS
    for (int b = block_tiles; b >= 1; --b) {
        c->items = make_items(c, b, &c->max_rows, &c->max_item_leaves, wide ? 1 : 3);
        c->lds = contract_lds_bytes(c->contract_q, c->max_rows, nfun, c->plan.max_img, c->max_item_leaves, n3);
        if (c->lds > kMaxDynLds && c->contract_q > 16) {   // shorter stages before smaller blocks
            c->contract_q = 16;
            c->lds = contract_lds_bytes(16, c->max_rows, nfun, c->plan.max_img, c->max_item_leaves, n3);
        }
        if (c->lds <= kMaxDynLds) break;
    }
    // the split stage keeps bf16 limbs of every row: use the largest tile
    // block whose three-limb stage fits in LDS
    for (int b = block_tiles; b >= 1; --b) {
        c->items_split = make_items(c, b, &c->max_rows_split, &c->max_item_leaves_split);
        if (split_lds_bytes(3, c->max_rows_split, nfun, c->plan.max_img, c->max_item_leaves_split, n3) <= kMaxDynLds)
            break;
    }
    // nonlocal work items: the contraction's K-chunks of every element a
    // projector image reaches, cut into row blocks of at most 16 tile pairs
    // (row tiles x projector column tiles); one coefficient slot per chunk
    c->nl_items.clear();
    c->nl_elems.clear();
    c->nl_doubles = 0;
    int max_npad = 16, max_leaves = 1;
    // moment form on tensor-product elements whose rows all fit in LDS
    size_t mom_lds = 0;
    c->nl_planes = c->plan.kp.p <= 2 ? nl_moment_planes(c->plan.kp.n) : 0;
    if (c->nl_planes > 0) {
        for (const ElemDev &el : c->plan.elems)
            if (el.npg > 0)
                mom_lds = std::max(mom_lds, nl_moment_lds(el.nfun, el.ncol, c->plan.max_img, c->plan.kp.n, c->nl_planes));
        if (mom_lds > kMaxDynLds) c->nl_planes = 0;
    }
    for (int64_t e = 0; e < c->plan.nel; ++e) {
        ElemDev &el = c->plan.elems[e];
        el.pf_nchunk = 0;
        el.pf_base = 0;
        if (el.npg == 0) continue;
        const int T = (el.nloc + 15) / 16, TC = (el.ncol + 15) / 16;
        const int rows = c->nl_planes > 0 ? nl_moment_tasks(el.nfun, el.ncol) : T;
        const int RB = c->nl_planes > 0 ? kNlMomentTasks : std::max(1, 16 / TC);
        const int64_t nleaf = el.leaf_end - el.leaf_off, nch = el.nchunk;
        el.pf_nchunk = (int32_t)nch;
        el.pf_base = c->nl_doubles;
        c->nl_doubles += nch * (int64_t)(16 * TC) * (16 * T);
        c->nl_elems.push_back((int32_t)e);
        max_npad = std::max(max_npad, 16 * T);
        for (int64_t ch = 0; ch < nch; ++ch)
            for (int R0 = 0; R0 < rows; R0 += RB) {
                NlItemDev it{};
                it.elem = (int32_t)e;
                it.chunk = (int32_t)ch;
                it.R0 = R0;
                it.nR = std::min(RB, rows - R0);
                it.leaf_b = el.leaf_off + ch * nleaf / nch;
                it.leaf_e = el.leaf_off + (ch + 1) * nleaf / nch;
                max_leaves = std::max(max_leaves, (int)(it.leaf_e - it.leaf_b));
                c->nl_items.push_back(it);
            }
    }
    c->nl_lds = nl_lds_bytes(max_npad, std::max(c->plan.max_ncol, 1), nfun, c->plan.max_img, max_leaves, n3);
    // what the direct form could not hold stays refused
    if (c->nl_planes > 0 && c->nl_lds <= kMaxDynLds) c->nl_lds = mom_lds;
}

// Projector coefficients of every element a projector reaches.
static hipError_t run_projectors(pufe_ctx *c, const KParams &kp, hipStream_t st) {
    const int n = (int)c->nl_items.size();
    hipError_t e;
    if (c->nl_planes > 0)
        e = launch_nl_moments(kp, n, c->d_nl_items.p, c->d_elems.p, c->d_groups.p, c->d_img.p, c->d_edof.p, c->d_leaves.p,
                              c->d_pgroups.p, c->nl_planes, c->d_Fp.p, c->nl_lds, st);
    else
        e = launch_nl_f(c->plan.max_l, kp, n, c->d_nl_items.p, c->d_elems.p, c->d_groups.p, c->d_img.p, c->d_edof.p,
                        c->d_leaves.p, c->d_pgroups.p, c->d_Fp.p, c->nl_lds, st);
    if (e != hipSuccess) return e;
    return launch_nl_reduce(c->d_elems.p, c->d_nl_elems.p, (int)c->nl_elems.size(), c->d_Fp.p, st);
}

static int upload_items(pufe_ctx *ctx, hipStream_t st);

// Device tables and buffers of the nonlocal term for the current plan.
static int upload_nonlocal(pufe_ctx *ctx, hipStream_t st) {
    const Plan &pl = ctx->plan;
    if (pl.n_pfun == 0) return PUFE_OK;
    if (ctx->nl_lds > kMaxDynLds) return fail(ctx, PUFE_ERR_UNSUPPORTED, "nonlocal stage does not fit in LDS");
    CHECK_HIP(ctx, ctx->d_nl_items.upload(ctx->nl_items, st), "upload nonlocal items");
    CHECK_HIP(ctx, ctx->d_nl_elems.upload(ctx->nl_elems, st), "upload nonlocal elements");
    CHECK_HIP(ctx, ctx->d_pgroups.upload(pl.pgroups, st), "upload projector groups");
    CHECK_HIP(ctx, ctx->d_pfun_h.upload(pl.pfun_h, st), "upload projector weights");
    CHECK_HIP(ctx, ctx->d_dof_el_off.upload(pl.dof_el_off, st), "upload DOF map");
    CHECK_HIP(ctx, ctx->d_dof_el.upload(pl.dof_el, st), "upload DOF map");
    CHECK_HIP(ctx, ctx->d_Fp.alloc((size_t)std::max<int64_t>(ctx->nl_doubles, 1)), "alloc projector coefficients");
    CHECK_HIP(ctx, ctx->d_nlf.alloc((size_t)kMaxKPerLaunch * pl.n_pfun * pl.dof_off[pl.nv]), "alloc projector sums");
    return PUFE_OK;
}

static int place_moments(pufe_ctx *ctx, hipStream_t st);

int pufe_set_moment_limit(pufe_ctx *ctx, int64_t bytes) {
    if (!ctx) return PUFE_ERR_INVALID_ARG;
    if (!ctx->have_problem) return fail(ctx, PUFE_ERR_STATE, "pufe_set_problem must come first");
    if (ctx->have_tables) return fail(ctx, PUFE_ERR_STATE, "the moment forms' limit is set before pufe_setup");
    ctx->mom_limit = bytes < 0 ? -1 : bytes;
    return PUFE_OK;
}

int pufe_setup(pufe_ctx *ctx, void *stream) {
    if (!ctx) return PUFE_ERR_INVALID_ARG;
    if (!ctx->have_problem) return fail(ctx, PUFE_ERR_STATE, "pufe_set_problem must come first");
    hipStream_t st = (hipStream_t)stream;
    CHECK_HIP(ctx, hipSetDevice(ctx->device), "hipSetDevice");
    ctx->have_setup = ctx->have_tables = false;   // until all of it has succeeded
    ++ctx->plan_gen;   // a batch's graph must not replay over what is replaced, also if this fails
    {
        hipError_t ea = init_contract_attributes();
        if (ea == hipSuccess) ea = init_moment_attributes();
        if (ea == hipSuccess) ea = init_split_attributes();
        if (ea == hipSuccess) ea = init_backward_attributes();
        if (ea == hipSuccess) ea = init_adjoint_attributes();
        if (ea == hipSuccess) ea = init_nonlocal_attributes();
        if (ea != hipSuccess) {
            (void)hipGetLastError();   // do not leave the error for the caller's next HIP call
            return hipfail(ctx, ea, "kernel attributes");
        }
    }
    Plan &pl = ctx->plan;
    const int64_t nel = pl.nel;
    const int n_atoms = (int)ctx->prob.species.size();
    CHECK_HIP(ctx, ctx->d_pos.upload(ctx->prob.pos, st), "upload positions");
    CHECK_HIP(ctx, ctx->d_spl.upload(pl.spl, st), "upload radial tables");
    pl.kp.spl = ctx->d_spl.p;
    CHECK_HIP(ctx, ctx->d_leaf_count.alloc(nel + 1), "alloc leaf counts");
    CHECK_HIP(ctx, ctx->d_leaf_off.alloc(nel + 1), "alloc leaf offsets");
    const double L[3] = {pl.lat[0], pl.lat[4], pl.lat[8]};
    const pufe_quad &q = ctx->prob.quad;
    ctx->leaf_off_h.assign(nel + 1, 0);
    if (q.mode == PUFE_QUAD_GEOM) {
        // count leaves, scan, emit (one octree walk per element, twice)
        CHECK_HIP(ctx, launch_aq_geom(pl.kp, nel, ctx->d_pos.p, n_atoms, L, q.max_level, q.dist, ctx->d_leaf_count.p,
                                      nullptr, nullptr, nullptr, st), "adaptive quadrature (count)");
        CHECK_HIP(ctx, launch_scan(ctx->d_leaf_count.p, nel, ctx->d_leaf_off.p, st), "scan");
        CHECK_HIP(ctx, hipMemcpyAsync(ctx->leaf_off_h.data(), ctx->d_leaf_off.p, sizeof(int64_t) * (nel + 1),
                                      hipMemcpyDeviceToHost, st), "download leaf offsets");
        CHECK_HIP(ctx, hipStreamSynchronize(st), "sync");
        ctx->n_leaves = ctx->leaf_off_h[nel];
        CHECK_HIP(ctx, ctx->d_leaves.alloc(ctx->n_leaves), "alloc leaves");
        CHECK_HIP(ctx, ctx->d_leaf_elem.alloc(ctx->n_leaves), "alloc leaf elements");
        CHECK_HIP(ctx, launch_aq_geom(pl.kp, nel, ctx->d_pos.p, n_atoms, L, q.max_level, q.dist, nullptr,
                                      ctx->d_leaf_off.p, ctx->d_leaves.p, ctx->d_leaf_elem.p, st),
                  "adaptive quadrature (emit)");
    } else {
        // error-driven rule: the element tables are needed first
        DevBuf<ElemDev> elems;
        CHECK_HIP(ctx, elems.upload(pl.elems, st), "upload elements");
        CHECK_HIP(ctx, ctx->d_groups.upload(pl.groups, st), "upload groups");
        CHECK_HIP(ctx, ctx->d_img.upload(pl.img_cur, st), "upload images");
        DevBuf<CellDev> cur, next;
        DevBuf<int64_t> cnt, off;
        DevBuf<uint64_t> nmask;
        CHECK_HIP(ctx, cur.alloc(nel), "alloc cells");
        CHECK_HIP(ctx, launch_aq_error_init(nel, elems.p, cur.p, st), "rule roots");
        int64_t n = nel;
        for (int lev = 0; lev < q.max_level; ++lev) {
            CHECK_HIP(ctx, cnt.alloc(n + 1), "alloc counts");
            CHECK_HIP(ctx, off.alloc(n + 1), "alloc offsets");
            CHECK_HIP(ctx, nmask.alloc(n + 1), "alloc masks");
            CHECK_HIP(ctx, launch_aq_error_test(pl.kp, elems.p, ctx->d_groups.p, ctx->d_img.p, cur.p, n, q.max_level,
                                                q.tol, cnt.p, nmask.p, st), "rule test");
            CHECK_HIP(ctx, launch_scan(cnt.p, n, off.p, st), "scan");
            int64_t total = 0;
            CHECK_HIP(ctx, hipMemcpyAsync(&total, off.p + n, sizeof(int64_t), hipMemcpyDeviceToHost, st), "download");
            CHECK_HIP(ctx, hipStreamSynchronize(st), "sync");
            if (total == n) break;   // no cell split at this level
            CHECK_HIP(ctx, next.alloc(total), "alloc cells");
            CHECK_HIP(ctx, launch_aq_error_expand(n, cur.p, off.p, nmask.p, next.p, st), "rule expand");
            std::swap(cur.p, next.p);
            std::swap(cur.n, next.n);
            n = total;
        }
        ctx->n_leaves = n;
        CHECK_HIP(ctx, ctx->d_leaves.alloc(n), "alloc leaves");
        CHECK_HIP(ctx, ctx->d_leaf_elem.alloc(n), "alloc leaf elements");
        CHECK_HIP(ctx, launch_aq_error_finish(n, cur.p, ctx->d_leaves.p, ctx->d_leaf_elem.p, ctx->d_leaf_count.p, st),
                  "rule leaves");
        CHECK_HIP(ctx, launch_scan(ctx->d_leaf_count.p, nel, ctx->d_leaf_off.p, st), "scan");
        CHECK_HIP(ctx, hipMemcpyAsync(ctx->leaf_off_h.data(), ctx->d_leaf_off.p, sizeof(int64_t) * (nel + 1),
                                      hipMemcpyDeviceToHost, st), "download leaf offsets");
        CHECK_HIP(ctx, hipStreamSynchronize(st), "sync");
    }
    ctx->n_qp = ctx->n_leaves * pl.kp.n3;
    for (int64_t e = 0; e < nel; ++e) {
        pl.elems[e].leaf_off = ctx->leaf_off_h[e];
        pl.elems[e].leaf_end = ctx->leaf_off_h[e + 1];
    }
    plan_items(ctx, ctx->tune_items, ctx->tune_block);
    if (ctx->lds > kMaxDynLds)
        return fail(ctx, PUFE_ERR_UNSUPPORTED, "contraction stage does not fit in LDS");
    CHECK_HIP(ctx, ctx->d_elems.upload(pl.elems, st), "upload elements");
    CHECK_HIP(ctx, ctx->d_groups.upload(pl.groups, st), "upload groups");
    CHECK_HIP(ctx, ctx->d_img.upload(pl.img_cur, st), "upload images");
    CHECK_HIP(ctx, ctx->d_edof.upload(pl.edof, st), "upload enriched functions");
    if (pl.bloch) {
        CHECK_HIP(ctx, ctx->d_img_nk.upload(pl.img_nk, st), "upload image shifts");
        CHECK_HIP(ctx, ctx->d_bpart.upload(pl.bpart, st), "upload enriched partners");
        CHECK_HIP(ctx, ctx->d_wimg.alloc(pl.img_nk.size() / 4), "alloc image weights");
    }
    CHECK_HIP(ctx, ctx->d_items.upload_list(ctx->items, st), "upload work items");
    CHECK_HIP(ctx, ctx->d_items_wide.upload_list(ctx->items_wide, st), "upload work items");
    CHECK_HIP(ctx, ctx->d_items_split.upload_list(ctx->items_split, st), "upload work items");
    // tables of the self-consistent field pieces and of the adjoint belong to the
    // previous plan (and its rule: a caller's, if pufe_set_rule gave one)
    ctx->d_dof_el_off.release();
    ctx->d_dof_el.release();
    ctx->d_fe_be.release();
    ctx->have_poisson = false;
    ctx->have_bw = ctx->have_adj = ctx->have_bw_direct = false;
    {
        int rc = upload_nonlocal(ctx, st);
        if (rc != PUFE_OK) return rc;
    }
    CHECK_HIP(ctx, ctx->d_contr.upload(pl.contr, st), "upload assembly lists");
    CHECK_HIP(ctx, ctx->d_blocks.upload(pl.blocks, st), "upload assembly lists");
    CHECK_HIP(ctx, ctx->d_reduce.upload_list(ctx->reduce, st), "upload chunk reduction list");
    CHECK_HIP(ctx, ctx->d_reduce_f64.upload_list(ctx->reduce_f64, st), "upload chunk reduction list");
    CHECK_HIP(ctx, ctx->d_brow.upload(pl.brow, st), "upload layout");
    CHECK_HIP(ctx, ctx->d_bcol.upload(pl.bcol, st), "upload layout");
    CHECK_HIP(ctx, ctx->d_bval_off.upload(pl.bval_off, st), "upload layout");
    CHECK_HIP(ctx, ctx->d_dof_off.upload(pl.dof_off, st), "upload layout");
    CHECK_HIP(ctx, ctx->d_partial.alloc((size_t)ctx->part_slots * 512), "alloc partial tiles");
    {
        int rc = place_moments(ctx, st);
        if (rc != PUFE_OK) return rc;
    }
    {
        // the allocation-free entry's workspace: its device address is looked
        // up once per device, here at set-up
        double *ws = nullptr;
        CHECK_HIP(ctx, scratch_address(ctx->device, &ws), "workspace address");
    }
    CHECK_HIP(ctx, hipStreamSynchronize(st), "sync");
    ctx->have_setup = ctx->have_tables = true;
    ++ctx->plan_gen;
    return PUFE_OK;
}

int pufe_set_rule(pufe_ctx *ctx, int64_t n_leaves, const int32_t *level, const int32_t *ijk,
                  const int64_t *elem_leaf_offset, void *stream) {
    if (!ctx) return PUFE_ERR_INVALID_ARG;
    if (!ctx->have_tables) return fail(ctx, PUFE_ERR_STATE, "pufe_setup must come first");
    Plan &pl = ctx->plan;
    const int64_t nel = pl.nel;
    if (n_leaves < nel || !level || !ijk || !elem_leaf_offset)
        return fail(ctx, PUFE_ERR_INVALID_ARG, "null pointer or fewer leaves than elements");
    if (elem_leaf_offset[0] != 0 || elem_leaf_offset[nel] != n_leaves)
        return fail(ctx, PUFE_ERR_INVALID_ARG, "leaf offsets must run from 0 to n_leaves");
    std::vector<uint32_t> codes(n_leaves);
    std::vector<int32_t> lelem(n_leaves);
    for (int64_t e = 0; e < nel; ++e) {
        const int64_t b = elem_leaf_offset[e], en = elem_leaf_offset[e + 1];
        if (en <= b) return fail(ctx, PUFE_ERR_INVALID_ARG, "every element needs at least one leaf");
        // the leaves of an element tile its reference cube: their volumes,
        // in units of the finest cell, add up to the whole
        int64_t vol = 0;
        for (int64_t k = b; k < en; ++k) {
            const int lev = level[k];
            if (lev < 0 || lev > kMaxLevel) return fail(ctx, PUFE_ERR_INVALID_ARG, "leaf level outside 0..8");
            for (int d = 0; d < 3; ++d)
                if (ijk[3 * k + d] < 0 || ijk[3 * k + d] >= (1 << lev))
                    return fail(ctx, PUFE_ERR_INVALID_ARG, "leaf coordinate outside its level's range");
            vol += (int64_t)1 << (3 * (kMaxLevel - lev));
            codes[k] = leaf_pack(lev, ijk[3 * k], ijk[3 * k + 1], ijk[3 * k + 2]);
            lelem[k] = (int32_t)e;
        }
        if (vol != (int64_t)1 << (3 * kMaxLevel))
            return fail(ctx, PUFE_ERR_INVALID_ARG, "the leaves of an element do not cover its cell once");
    }
    hipStream_t st = (hipStream_t)stream;
    CHECK_HIP(ctx, hipSetDevice(ctx->device), "hipSetDevice");
    CHECK_HIP(ctx, hipStreamSynchronize(st), "sync");
    // from here on the tables are the new rule's in part: a failure leaves a context
    // without a rule, not one whose launches (a batch's graph either) read freed or
    // short lists
    ctx->have_setup = false;
    ++ctx->plan_gen;
    CHECK_HIP(ctx, ctx->d_leaves.alloc(n_leaves), "alloc leaves");
    CHECK_HIP(ctx, ctx->d_leaf_elem.alloc(n_leaves), "alloc leaf elements");
    CHECK_HIP(ctx, hipMemcpy(ctx->d_leaves.p, codes.data(), sizeof(uint32_t) * n_leaves, hipMemcpyHostToDevice),
              "upload leaves");
    CHECK_HIP(ctx, hipMemcpy(ctx->d_leaf_elem.p, lelem.data(), sizeof(int32_t) * n_leaves, hipMemcpyHostToDevice),
              "upload leaf elements");
    ctx->leaf_off_h.assign(elem_leaf_offset, elem_leaf_offset + nel + 1);
    CHECK_HIP(ctx, hipMemcpy(ctx->d_leaf_off.p, ctx->leaf_off_h.data(), sizeof(int64_t) * (nel + 1),
                             hipMemcpyHostToDevice), "upload leaf offsets");
    ctx->n_leaves = n_leaves;
    ctx->n_qp = n_leaves * pl.kp.n3;
    for (int64_t e = 0; e < nel; ++e) {
        pl.elems[e].leaf_off = ctx->leaf_off_h[e];
        pl.elems[e].leaf_end = ctx->leaf_off_h[e + 1];
    }
    plan_items(ctx, ctx->tune_items, ctx->tune_block);
    if (ctx->lds > kMaxDynLds) return fail(ctx, PUFE_ERR_UNSUPPORTED, "contraction stage does not fit in LDS");
    const int rc = upload_items(ctx, nullptr);
    ctx->have_setup = rc == PUFE_OK;
    return rc;
}

int pufe_query(pufe_ctx *ctx, pufe_sizes *out) {
    if (!ctx || !out) return PUFE_ERR_INVALID_ARG;
    if (!ctx->have_problem) return fail(ctx, PUFE_ERR_STATE, "no problem defined");
    const Plan &pl = ctx->plan;
    std::memset(out, 0, sizeof *out);
    out->n_elem = pl.nel;
    out->n_vertex = pl.nv;
    out->n_dof = pl.dof_off[pl.nv];
    out->n_fe_dof = pl.nv * pl.nfs;
    out->n_enr_dof = out->n_dof - out->n_fe_dof;
    out->nnzb = (int64_t)pl.bcol.size();
    out->nnz = pl.nnz;
    out->n_qp = ctx->n_qp;
    out->n_leaves = ctx->n_leaves;
    out->max_nloc = pl.max_nloc;
    out->n_colors = pl.n_colors;
    out->n_atoms = (int32_t)ctx->prob.species.size();
    out->n_fe_slots = pl.nfs;
    return PUFE_OK;
}

int pufe_get_layout(pufe_ctx *ctx, int64_t *dof_offset, int64_t *brow_ptr, int32_t *bcol, int64_t *bval_offset) {
    if (!ctx) return PUFE_ERR_INVALID_ARG;
    if (!ctx->have_problem) return fail(ctx, PUFE_ERR_STATE, "no problem defined");
    const Plan &pl = ctx->plan;
    if (dof_offset) std::memcpy(dof_offset, pl.dof_off.data(), sizeof(int64_t) * pl.dof_off.size());
    if (brow_ptr) std::memcpy(brow_ptr, pl.brow_ptr.data(), sizeof(int64_t) * pl.brow_ptr.size());
    if (bcol) std::memcpy(bcol, pl.bcol.data(), sizeof(int32_t) * pl.bcol.size());
    if (bval_offset) std::memcpy(bval_offset, pl.bval_off.data(), sizeof(int64_t) * pl.bval_off.size());
    return PUFE_OK;
}

int pufe_get_quadrature(pufe_ctx *ctx, double *d_xyz, double *d_w, int64_t *d_elem_qp_offset, void *stream) {
    if (!ctx) return PUFE_ERR_INVALID_ARG;
    if (!ctx->have_setup) return fail(ctx, PUFE_ERR_STATE, "pufe_setup must come first");
    hipStream_t st = (hipStream_t)stream;
    CHECK_HIP(ctx, hipSetDevice(ctx->device), "hipSetDevice");
    if (d_xyz || d_w)
        CHECK_HIP(ctx, launch_qp_export(ctx->plan.kp, ctx->n_leaves, ctx->d_leaves.p, ctx->d_leaf_elem.p, d_xyz, d_w, st),
                  "quadrature export");
    if (d_elem_qp_offset)
        CHECK_HIP(ctx, launch_elem_qp_offset(ctx->plan.kp, ctx->plan.nel, ctx->d_leaf_off.p, d_elem_qp_offset, st),
                  "quadrature offsets");
    return PUFE_OK;
}

int pufe_get_forms(pufe_ctx *ctx, int32_t *elem_moment, int32_t *adjoint_moment) {
    if (!ctx) return PUFE_ERR_INVALID_ARG;
    if (!ctx->have_setup) return fail(ctx, PUFE_ERR_STATE, "pufe_setup must come first");
    if (elem_moment)
        for (int64_t e = 0; e < ctx->plan.nel; ++e) elem_moment[e] = ctx->plan.elems[e].mchunk > 0;
    if (adjoint_moment) *adjoint_moment = ctx->have_adj && !ctx->adj_fold.empty();
    return PUFE_OK;
}

int pufe_get_leaves(pufe_ctx *ctx, int32_t *level, int32_t *ijk, int64_t *elem_leaf_offset) {
    if (!ctx) return PUFE_ERR_INVALID_ARG;
    if (!ctx->have_setup) return fail(ctx, PUFE_ERR_STATE, "pufe_setup must come first");
    CHECK_HIP(ctx, hipSetDevice(ctx->device), "hipSetDevice");
    std::vector<uint32_t> codes(std::max<int64_t>(ctx->n_leaves, 1));
    CHECK_HIP(ctx, hipMemcpy(codes.data(), ctx->d_leaves.p, sizeof(uint32_t) * ctx->n_leaves, hipMemcpyDeviceToHost),
              "download leaves");
    for (int64_t i = 0; i < ctx->n_leaves; ++i) {
        uint32_t c = codes[i];
        if (level) level[i] = (int32_t)(c >> 27);
        if (ijk) {
            ijk[3 * i] = (int32_t)(c & 511u);
            ijk[3 * i + 1] = (int32_t)((c >> 9) & 511u);
            ijk[3 * i + 2] = (int32_t)((c >> 18) & 511u);
        }
    }
    if (elem_leaf_offset) std::memcpy(elem_leaf_offset, ctx->leaf_off_h.data(), sizeof(int64_t) * ctx->leaf_off_h.size());
    return PUFE_OK;
}

// Problems with tabulated radials, serendipity elements or the Bloch-periodic
// enrichment run the general variant of the contraction kernels; the others a
// variant compiled for analytic radials and Lagrange elements only (fewer
// live registers).
static bool general_variant(const Plan &pl) { return !pl.spl.empty() || pl.kp.p == 3 || pl.bloch; }

// The element contraction and the K-chunk sum into `partial` (the context's
// partial-tile buffer, or the fixed workspace of the allocation-free entry);
// wimg: image weights of the Bloch-periodic enrichment at one k-point (null
// for the periodic form).
static int run_contraction(pufe_ctx *ctx, const double *d_V, int precision, hipStream_t st, double *partial,
                           bool timed = true, const double *wimg = nullptr) {
    const CtxDev *self = ctx->d_self.p + (partial == ctx->d_partial.p ? 0 : 1);
    const bool saved = ctx->timing;
    ctx->timing = saved && timed;
    struct Restore {
        pufe_ctx *c;
        bool v;
        ~Restore() { c->timing = v; }
    } restore{ctx, saved};
    const Plan &pl = ctx->plan;
    KParams kp = pl.kp;
    kp.wimg = wimg;
    if (precision == PUFE_PREC_BF16X3 || precision == PUFE_PREC_BF16X6) {
        const int nl = precision == PUFE_PREC_BF16X3 ? 2 : 3;
        const size_t lds = split_lds_bytes(nl, ctx->max_rows_split, std::max(pl.max_nfun, 1), pl.max_img,
                                           ctx->max_item_leaves_split, pl.kp.n3);
        if (lds > kMaxDynLds) return fail(ctx, PUFE_ERR_UNSUPPORTED, "split stage does not fit in LDS");
        {
            TimedRegion tr(ctx, 0, st);
            CHECK_HIP(ctx, launch_contract_split(nl, pl.max_l, general_variant(pl), kp, (int)ctx->items_split.size(), ctx->d_items_split.p,
                                                 ctx->d_elems.p, ctx->d_groups.p, ctx->d_img.p, ctx->d_edof.p,
                                                 ctx->d_leaves.p, d_V, partial, lds, st),
                      "split contraction");
        }
    } else {
        TimedRegion tr(ctx, 0, st);
        // wide items first: they are the longest
        CHECK_HIP(ctx, launch_contract_wide(pl.max_l, general_variant(pl), kp, (int)ctx->items_wide.size(), ctx->d_items_wide.p,
                                            ctx->d_elems.p, ctx->d_groups.p, ctx->d_img.p, ctx->d_edof.p,
                                            ctx->d_leaves.p, d_V, partial, ctx->lds_wide, st),
                  "contraction (wide items)");
        CHECK_HIP(ctx, launch_contract_f64(ctx->contract_q, pl.max_l, general_variant(pl), kp, (int)ctx->items.size(), ctx->d_items.p,
                                           ctx->d_elems.p, ctx->d_groups.p, ctx->d_img.p, ctx->d_edof.p,
                                           ctx->d_leaves.p, d_V, partial, ctx->lds, st),
                  "contraction");
        CHECK_HIP(ctx, launch_classical_moments(self, ctx->d_mom_items[2].p, (int)ctx->mom_items[2].size(), d_V, st),
                  "contraction (classical moments)");
        for (int w = 1; w >= 0; --w)
            CHECK_HIP(ctx, launch_moments(w ? 8 : 4, pl.kp.n, pl.max_l, general_variant(pl), pl.kp.skew != 0, self, ctx->d_mom_items[w].p,
                                          (int)ctx->mom_items[w].size(), ctx->d_mom_tasks.p, d_V, wimg, ctx->mom_lds[w], st),
                      "contraction (moments)");
    }
    TimedRegion tr(ctx, 3, st);
    if (precision == PUFE_PREC_FP64) {
        CHECK_HIP(ctx, launch_chunk_reduce(ctx->d_elems.p, ctx->d_reduce_f64.p, (int)ctx->reduce_f64.size(), partial, st),
                  "K-chunk reduction");
        CHECK_HIP(ctx, launch_moment_reduce(self, ctx->d_mom_reduce.p, (int)ctx->mom_reduce.size(), st),
                  "K-chunk reduction (moments)");
        CHECK_HIP(ctx, launch_moment_expand(self, ctx->d_mom_expand.p, (int)ctx->mom_expand.size(), partial, st),
                  "element matrices from moments");
        return PUFE_OK;
    }
    CHECK_HIP(ctx, launch_chunk_reduce(ctx->d_elems.p, ctx->d_reduce.p, (int)ctx->reduce.size(), partial, st),
              "K-chunk reduction");
    return PUFE_OK;
}

// Argument checks shared by pufe_assemble and pufe_assemble_noalloc.
static int check_assemble_args(pufe_ctx *ctx, const double *d_V, const double *kpts, int n_k, int precision,
                               int out_dtype, void *d_H) {
    if (!ctx) return PUFE_ERR_INVALID_ARG;
    if (!ctx->have_setup) return fail(ctx, PUFE_ERR_STATE, "pufe_setup must come first");
    if (!d_V || !kpts || n_k < 1 || !d_H) return fail(ctx, PUFE_ERR_INVALID_ARG, "null pointer or n_k < 1");
    if (precision < PUFE_PREC_FP64 || precision > PUFE_PREC_BF16X6)
        return fail(ctx, PUFE_ERR_INVALID_ARG, "unknown precision");
    if (out_dtype < PUFE_OUT_C128 || out_dtype > PUFE_OUT_F64_GAMMA)
        return fail(ctx, PUFE_ERR_INVALID_ARG, "unknown output dtype");
    for (int k = 0; k < n_k; ++k) {
        for (int d = 0; d < 3; ++d)
            if (!std::isfinite(kpts[3 * k + d])) return fail(ctx, PUFE_ERR_INVALID_ARG, "non-finite k-point");
        if (out_dtype == PUFE_OUT_F64_GAMMA &&
            (std::fmod(kpts[3 * k], 1.0) != 0.0 || std::fmod(kpts[3 * k + 1], 1.0) != 0.0 ||
             std::fmod(kpts[3 * k + 2], 1.0) != 0.0))
            return fail(ctx, PUFE_ERR_INVALID_ARG, "real output needs every k-point at Gamma");
    }
    return PUFE_OK;
}

// Assembly with the Bloch-periodic enrichment: for every k-point the image
// weights, the contraction of the real and imaginary rows, the K-chunk sum,
// the projector coefficients of those rows (with projectors), the assembly of
// that k-point's output and the separable term.
static int assemble_bloch(pufe_ctx *ctx, const double *d_V, const double *kpts, int n_k, int precision,
                          int out_dtype, void *d_H, void *d_S, hipStream_t st, bool nonlocal) {
    const Plan &pl = ctx->plan;
    const int64_t per = out_dtype == PUFE_OUT_F64_GAMMA ? pl.nnz : 2 * pl.nnz;
    const size_t esz = out_dtype == PUFE_OUT_C64 ? sizeof(float) : sizeof(double);
    const int64_t nimg = (int64_t)(pl.img_nk.size() / 4);
    for (int k0 = 0; k0 < n_k; k0 += kMaxKPerLaunch) {
        KPoints kps;
        std::memset(&kps, 0, sizeof kps);
        kps.nk = std::min(kMaxKPerLaunch, n_k - k0);
        for (int k = 0; k < kps.nk; ++k)
            for (int d = 0; d < 3; ++d) kps.kap[k][d] = kpts[3 * (k0 + k) + d];
        for (int k = 0; k < kps.nk; ++k) {
            CHECK_HIP(ctx, launch_image_weights(ctx->d_img_nk.p, nimg, kps.kap[k], ctx->d_wimg.p, st),
                      "image weights");
            int rc = run_contraction(ctx, d_V, precision, st, ctx->d_partial.p, true, ctx->d_wimg.p);
            if (rc != PUFE_OK) return rc;
            const bool with_nl = nonlocal && pl.n_pfun > 0;
            if (with_nl) {
                // projector coefficients of this k-point's rows
                TimedRegion tn(ctx, 4, st);
                KParams kp = pl.kp;
                kp.wimg = ctx->d_wimg.p;
                CHECK_HIP(ctx, run_projectors(ctx, kp, st), "projector coefficients");
            }
            TimedRegion tr(ctx, 1, st);
            char *H = (char *)d_H + (size_t)(k0 + k) * per * esz;
            char *S = d_S ? (char *)d_S + (size_t)(k0 + k) * per * esz : nullptr;
            KPoints one;
            std::memset(&one, 0, sizeof one);
            one.nk = 1;
            for (int d = 0; d < 3; ++d) one.kap[0][d] = kps.kap[k][d];
            const int64_t ndof = pl.dof_off[pl.nv];
            if (with_nl)
                CHECK_HIP(ctx, launch_nl_gather(pl.kp, ctx->d_elems.p, ctx->d_pgroups.p, ctx->d_edof.p, ctx->d_bpart.p,
                                                ctx->d_dof_el_off.p, ctx->d_dof_el.p, ctx->d_Fp.p, one, pl.n_pfun,
                                                ndof, ctx->d_nlf.p, st),
                          "projector sums");
            CHECK_HIP(ctx, launch_gather(ctx->d_self.p, ctx->d_blocks.p, pl.gather, ctx->d_partial.p, H, S, one,
                                         out_dtype, true, with_nl ? ctx->d_nlf.p : nullptr, ctx->d_pfun_h.p, pl.n_pfun,
                                         ndof, st),
                      "assembly");
        }
    }
    return PUFE_OK;
}

// Contraction, K-chunk sum and assembly of H and S, with the partial tiles in
// the given buffer.
static int assemble_impl(pufe_ctx *ctx, const double *d_V, const double *kpts, int n_k, int precision, int out_dtype,
                         void *d_H, void *d_S, hipStream_t st, double *partial, bool timed, bool nonlocal = true) {
    if (ctx->plan.bloch) return assemble_bloch(ctx, d_V, kpts, n_k, precision, out_dtype, d_H, d_S, st, nonlocal);
    int rc = run_contraction(ctx, d_V, precision, st, partial, timed);
    if (rc != PUFE_OK) return rc;
    const Plan &pl = ctx->plan;
    const bool with_nl = nonlocal && pl.n_pfun > 0;
    if (with_nl) {
        // projector coefficients of every element a projector image reaches
        TimedRegion tn(ctx, timed ? 4 : -1, st);
        CHECK_HIP(ctx, run_projectors(ctx, pl.kp, st), "projector coefficients");
    }
    TimedRegion tr(ctx, timed ? 1 : -1, st);
    const int64_t per = out_dtype == PUFE_OUT_F64_GAMMA ? pl.nnz : 2 * pl.nnz;
    const bool f32 = out_dtype == PUFE_OUT_C64;
    const size_t esz = f32 ? sizeof(float) : sizeof(double);
    for (int k0 = 0; k0 < n_k; k0 += kMaxKPerLaunch) {
        KPoints kps;
        std::memset(&kps, 0, sizeof kps);
        kps.nk = std::min(kMaxKPerLaunch, n_k - k0);
        for (int k = 0; k < kps.nk; ++k)
            for (int d = 0; d < 3; ++d) kps.kap[k][d] = kpts[3 * (k0 + k) + d];
        char *H = (char *)d_H + (size_t)k0 * per * esz;
        char *S = d_S ? (char *)d_S + (size_t)k0 * per * esz : nullptr;
        const int64_t ndof = pl.dof_off[pl.nv];
        if (with_nl)
            CHECK_HIP(ctx, launch_nl_gather(pl.kp, ctx->d_elems.p, ctx->d_pgroups.p, ctx->d_edof.p, nullptr,
                                            ctx->d_dof_el_off.p, ctx->d_dof_el.p, ctx->d_Fp.p, kps, pl.n_pfun, ndof,
                                            ctx->d_nlf.p, st),
                      "projector sums");
        CHECK_HIP(ctx, launch_gather(ctx->d_self.p, ctx->d_blocks.p, pl.gather, partial, H, S, kps, out_dtype,
                                     false, with_nl ? ctx->d_nlf.p : nullptr, ctx->d_pfun_h.p, pl.n_pfun, ndof, st),
                  "assembly");
    }
    return PUFE_OK;
}

int pufe_assemble(pufe_ctx *ctx, const double *d_V, const double *kpts, int n_k, int precision, int out_dtype,
                  void *d_H, void *d_S, void *stream) {
    int rc = check_assemble_args(ctx, d_V, kpts, n_k, precision, out_dtype, d_H);
    if (rc != PUFE_OK) return rc;
    hipStream_t st = (hipStream_t)stream;
    CHECK_HIP(ctx, hipSetDevice(ctx->device), "hipSetDevice");
    return assemble_impl(ctx, d_V, kpts, n_k, precision, out_dtype, d_H, d_S, st, ctx->d_partial.p, true);
}

int pufe_assemble_noalloc(pufe_ctx *ctx, const double *d_V, const double *kpts, int n_k, int precision, int out_dtype,
                          void *d_H, void *d_S, void *stream) {
    int rc = check_assemble_args(ctx, d_V, kpts, n_k, precision, out_dtype, d_H);
    if (rc != PUFE_OK) return rc;
    if (ctx->plan.n_pfun > 0)
        return fail(ctx, PUFE_ERR_UNSUPPORTED,
                    "pufe_assemble_noalloc: the nonlocal term keeps its coefficients in context buffers; use pufe_assemble");
    if (ctx->plan.bloch)
        return fail(ctx, PUFE_ERR_UNSUPPORTED,
                    "pufe_assemble_noalloc: the Bloch-periodic enrichment keeps its image weights in context buffers; "
                    "use pufe_assemble");
    const size_t need = noalloc_bytes(ctx);
    if (need > kScratchBytes)
        return fail(ctx, PUFE_ERR_UNSUPPORTED,
                    "pufe_assemble_noalloc: this problem's partial tiles need " + std::to_string(need) +
                        " bytes of workspace, more than the fixed " + std::to_string(kScratchBytes) +
                        " bytes; use pufe_assemble");
    hipStream_t st = (hipStream_t)stream;
    CHECK_HIP(ctx, hipSetDevice(ctx->device), "hipSetDevice");
    double *ws = nullptr;
    CHECK_HIP(ctx, scratch_address(ctx->device, &ws), "workspace address");
    return assemble_impl(ctx, d_V, kpts, n_k, precision, out_dtype, d_H, d_S, st,
                         ws + kNoallocTiles / sizeof(double), false);
}

int pufe_element_matrices(pufe_ctx *ctx, int64_t elem, const double *d_V, int precision, double *d_He,
                          double *d_Se, int32_t *nloc, void *stream) {
    if (!ctx) return PUFE_ERR_INVALID_ARG;
    if (!ctx->have_setup) return fail(ctx, PUFE_ERR_STATE, "pufe_setup must come first");
    if (!d_V || !d_He || !d_Se || elem < 0 || elem >= ctx->plan.nel)
        return fail(ctx, PUFE_ERR_INVALID_ARG, "bad element or null pointer");
    if (ctx->plan.bloch)
        return fail(ctx, PUFE_ERR_UNSUPPORTED, "element matrices of the Bloch-periodic enrichment are complex and per "
                                               "k-point; use pufe_assemble");
    hipStream_t st = (hipStream_t)stream;
    CHECK_HIP(ctx, hipSetDevice(ctx->device), "hipSetDevice");
    int rc = run_contraction(ctx, d_V, precision, st, ctx->d_partial.p);
    if (rc != PUFE_OK) return rc;
    CHECK_HIP(ctx, launch_elem_matrices(ctx->d_elems.p, elem, ctx->d_partial.p, d_He, d_Se, ctx->plan.elems[elem].nloc, st),
              "element matrices");
    if (nloc) *nloc = ctx->plan.elems[elem].nloc;
    return PUFE_OK;
}

// ------------------------------------------------ self-consistent field pieces

static bool dev_scalar(pufe_ctx *ctx, const double *d, double *h, hipStream_t st) {
    return hipMemcpyAsync(h, d, sizeof(double), hipMemcpyDeviceToHost, st) == hipSuccess &&
           hipStreamSynchronize(st) == hipSuccess;
}

// The (element, local function) pairs of every DOF and the per-element load
// sums, for the classical FE space's load vector.
static int ensure_fe_map(pufe_ctx *ctx, hipStream_t st) {
    const Plan &pl = ctx->plan;
    if (!ctx->d_dof_el_off.p) CHECK_HIP(ctx, ctx->d_dof_el_off.upload(pl.dof_el_off, st), "upload DOF map");
    if (!ctx->d_dof_el.p) CHECK_HIP(ctx, ctx->d_dof_el.upload(pl.dof_el, st), "upload DOF map");
    if (!ctx->d_fe_be.p) CHECK_HIP(ctx, ctx->d_fe_be.alloc((size_t)pl.nel * 32), "alloc load sums");
    return PUFE_OK;
}

static int fe_load_impl(pufe_ctx *ctx, const double *d_f, double *d_b, hipStream_t st) {
    const Plan &pl = ctx->plan;
    CHECK_HIP(ctx, launch_fe_load(pl.kp, ctx->d_elems.p, pl.nel, ctx->d_leaves.p, d_f, ctx->d_fe_be.p, pl.nv, pl.nfs,
                                  ctx->d_dof_off.p, ctx->d_dof_el_off.p, ctx->d_dof_el.p, d_b, st),
              "FE load vector");
    return PUFE_OK;
}

int pufe_fe_load(pufe_ctx *ctx, const double *d_f, double *d_b, void *stream) {
    if (!ctx) return PUFE_ERR_INVALID_ARG;
    if (!ctx->have_setup) return fail(ctx, PUFE_ERR_STATE, "pufe_setup must come first");
    if (!d_f || !d_b) return fail(ctx, PUFE_ERR_INVALID_ARG, "null pointer");
    hipStream_t st = (hipStream_t)stream;
    CHECK_HIP(ctx, hipSetDevice(ctx->device), "hipSetDevice");
    int rc = ensure_fe_map(ctx, st);
    if (rc != PUFE_OK) return rc;
    return fe_load_impl(ctx, d_f, d_b, st);
}

int pufe_fe_eval(pufe_ctx *ctx, const double *d_u, double *d_out, void *stream) {
    if (!ctx) return PUFE_ERR_INVALID_ARG;
    if (!ctx->have_setup) return fail(ctx, PUFE_ERR_STATE, "pufe_setup must come first");
    if (!d_u || !d_out) return fail(ctx, PUFE_ERR_INVALID_ARG, "null pointer");
    hipStream_t st = (hipStream_t)stream;
    CHECK_HIP(ctx, hipSetDevice(ctx->device), "hipSetDevice");
    CHECK_HIP(ctx, launch_fe_eval(ctx->plan.kp, ctx->d_elems.p, ctx->d_edof.p, ctx->d_leaves.p, ctx->d_leaf_elem.p,
                                  ctx->n_qp, d_u, d_out, st),
              "FE evaluation");
    return PUFE_OK;
}

// The Poisson operator of the classical FE space: K = 2 H restricted to the
// FE rows and columns of an assembly at Gamma with V = 0 (the kinetic term
// 1/2 int grad phi_i . grad phi_j of eq. disceig3d), without the separable
// term; and m_i = int phi_i.
static int build_poisson(pufe_ctx *ctx, hipStream_t st) {
    const Plan &pl = ctx->plan;
    const int64_t nfe = pl.nv * pl.nfs, nnzb = (int64_t)pl.bcol.size();
    {
        DevBuf<double> zeroV, Hfull;
        CHECK_HIP(ctx, zeroV.alloc((size_t)std::max<int64_t>(ctx->n_qp, 1)), "alloc zero potential");
        CHECK_HIP(ctx, launch_fill_zero(zeroV.p, ctx->n_qp, st), "zero potential");
        CHECK_HIP(ctx, Hfull.alloc((size_t)pl.nnz), "alloc kinetic matrix");
        const double gamma[3] = {0.0, 0.0, 0.0};
        int rc = assemble_impl(ctx, zeroV.p, gamma, 1, PUFE_PREC_FP64, PUFE_OUT_F64_GAMMA, Hfull.p, nullptr, st,
                               ctx->d_partial.p, false, false);
        if (rc != PUFE_OK) return rc;
        CHECK_HIP(ctx, ctx->d_Kfe.alloc((size_t)(nnzb * pl.nfs * pl.nfs)), "alloc FE stiffness");
        CHECK_HIP(ctx, launch_fe_blocks(nnzb, pl.nfs, ctx->d_bcol.p, ctx->d_bval_off.p, ctx->d_dof_off.p, Hfull.p, 2.0,
                                        ctx->d_Kfe.p, st),
                  "FE stiffness blocks");
        CHECK_HIP(ctx, hipStreamSynchronize(st), "sync");
    }
    CHECK_HIP(ctx, ctx->d_brow_ptr.upload(pl.brow_ptr, st), "upload block rows");
    CHECK_HIP(ctx, ctx->d_mfe.alloc((size_t)nfe), "alloc FE integrals");
    CHECK_HIP(ctx, ctx->d_fe_ones.alloc((size_t)std::max<int64_t>(nfe, ctx->n_qp)), "alloc ones");
    {
        std::vector<double> ones((size_t)std::max<int64_t>(nfe, ctx->n_qp), 1.0);
        CHECK_HIP(ctx, ctx->d_fe_ones.upload(ones, st), "upload ones");
    }
    int rc = fe_load_impl(ctx, ctx->d_fe_ones.p, ctx->d_mfe.p, st);
    if (rc != PUFE_OK) return rc;
    CHECK_HIP(ctx, ctx->d_cg.alloc((size_t)(6 * nfe)), "alloc CG workspace");
    CHECK_HIP(ctx, ctx->d_dot.alloc((size_t)(dot_partial_slots() + 1 + cg_partial_slots(pl.nv))), "alloc dot workspace");
    CHECK_HIP(ctx, ctx->d_cg_state.alloc(1), "alloc CG state");
    double *out = ctx->d_dot.p + dot_partial_slots();
    CHECK_HIP(ctx, launch_dot(nfe, ctx->d_mfe.p, ctx->d_fe_ones.p, ctx->d_dot.p, out, st), "dot");
    if (!dev_scalar(ctx, out, &ctx->m_sum, st)) return fail(ctx, PUFE_ERR_HIP, "read FE integral sum");
    ctx->have_poisson = true;
    return PUFE_OK;
}

int pufe_hartree(pufe_ctx *ctx, const double *d_n, double *d_vh, double *d_v, double tol, int max_iter,
                 int *iters, double *resid, void *stream) {
    if (!ctx) return PUFE_ERR_INVALID_ARG;
    if (!ctx->have_setup) return fail(ctx, PUFE_ERR_STATE, "pufe_setup must come first");
    if (!d_n || !d_vh) return fail(ctx, PUFE_ERR_INVALID_ARG, "null pointer");
    if (!(tol > 0.0) || max_iter < 1) return fail(ctx, PUFE_ERR_INVALID_ARG, "need tol > 0 and max_iter >= 1");
    hipStream_t st = (hipStream_t)stream;
    CHECK_HIP(ctx, hipSetDevice(ctx->device), "hipSetDevice");
    int rc = ensure_fe_map(ctx, st);
    if (rc != PUFE_OK) return rc;
    if (!ctx->have_poisson) {
        rc = build_poisson(ctx, st);
        if (rc != PUFE_OK) return rc;
    }
    const Plan &pl = ctx->plan;
    const int64_t n = pl.nv * pl.nfs;
    double *b = ctx->d_cg.p, *x = b + 5 * n;
    double *dots = ctx->d_dot.p;   // block partials of sum b and sum m x
    CgSolve cg{pl.nv, pl.nfs, ctx->d_brow_ptr.p, ctx->d_bcol.p, ctx->d_Kfe.p, b + n, b + 2 * n, b + 3 * n, b + 4 * n, x,
               dots + dot_partial_slots() + 1, ctx->d_cg_state.p};
    // right-hand side 4 pi (b - nbar m), nbar = int n / int 1 (the neutralising
    // background); conjugate gradients on K x = r from x = 0 (K is singular
    // with the constants as its kernel; r is orthogonal to them)
    rc = fe_load_impl(ctx, d_n, b, st);
    if (rc != PUFE_OK) return rc;
    CHECK_HIP(ctx, launch_dot_partials(n, b, ctx->d_fe_ones.p, dots, st), "dot");
    CHECK_HIP(ctx, launch_cg_start(cg, b, ctx->d_mfe.p, dots, ctx->m_sum, st), "right-hand side");
    CgState state{};
    for (int it = 0; it <= max_iter;) {
        // launches past the end of the solve do nothing: a batch is long
        // enough to hide the look at its outcome, short enough to waste little
        const int end = std::min(it + 16, max_iter);
        for (; it < end; ++it) CHECK_HIP(ctx, launch_cg_iteration(cg, it, tol, false, st), "CG iteration");
        CHECK_HIP(ctx, launch_cg_iteration(cg, it, tol, it == max_iter, st), "CG iteration");
        ++it;
        CHECK_HIP(ctx, hipMemcpyAsync(&state, ctx->d_cg_state.p, sizeof state, hipMemcpyDeviceToHost, st), "CG state");
        CHECK_HIP(ctx, hipStreamSynchronize(st), "CG state");
        if (state.done || state.ended) break;
    }
    const int it = state.it;
    const double rel = state.rel;
    // zero mean: int V_H = sum_i x_i m_i = 0
    CHECK_HIP(ctx, launch_dot_partials(n, ctx->d_mfe.p, x, dots, st), "dot");
    CHECK_HIP(ctx, launch_cg_mean(cg, dots, ctx->m_sum, d_v, st), "zero mean");
    CHECK_HIP(ctx, launch_fe_eval(pl.kp, ctx->d_elems.p, ctx->d_edof.p, ctx->d_leaves.p, ctx->d_leaf_elem.p,
                                  ctx->n_qp, x, d_vh, st),
              "Hartree potential at the points");
    if (iters) *iters = it;
    if (resid) *resid = rel;
    return PUFE_OK;
}

int pufe_lda_xc(int64_t n, const double *d_rho, double *d_vxc, double *d_exc, void *stream) {
    if (n < 0 || (n > 0 && (!d_rho || !d_vxc))) return PUFE_ERR_INVALID_ARG;
    hipError_t e = launch_lda_xc(n, d_rho, d_vxc, d_exc, (hipStream_t)stream);
    return e == hipSuccess ? PUFE_OK : PUFE_ERR_HIP;
}

// Plan the adjoint: one work item per (element, K-chunk of the forward
// partition), the padded Ps blocks, and for each atom the list of per-item
// group partial forces in a fixed order.
static int plan_adjoint_moments(pufe_ctx *c, int64_t pt_doubles, hipStream_t st);

static int plan_backward(pufe_ctx *c, bool split, hipStream_t st) {
    Plan &pl = c->plan;
    int max_npad = 16, max_nfun = 1, max_nenr = 1, max_nfun_wide = 1;
    std::vector<int64_t> pt_off(pl.nel + 1, 0);
    // an element runs the block-resident kernel when it has at most 80
    // functions and the launch's stage (sized by the largest Ps, row count and
    // enrichment table of its elements) still fits in LDS with it: elements
    // are taken in order of their own stage size; the others run the wide
    // kernel
    const int nimg = std::max(pl.max_img, 1);
    std::vector<char> wide(pl.nel, 1);
    {
        std::vector<std::pair<size_t, int64_t>> order;
        for (int64_t e = 0; e < pl.nel; ++e) {
            const ElemDev &el = pl.elems[e];
            if (el.nloc <= kBackwardMaxNloc)
                order.push_back({backward_lds_bytes(16 * ((el.nloc + 15) / 16), el.nloc - el.nfe, el.nfun, nimg), e});
        }
        std::stable_sort(order.begin(), order.end());
        int np = 16, ne = 1, nf = 1;
        for (const auto &o : order) {
            const ElemDev &el = pl.elems[o.second];
            const int np2 = std::max(np, 16 * ((el.nloc + 15) / 16)), ne2 = std::max(ne, el.nloc - el.nfe);
            const int nf2 = std::max(nf, el.nfun);
            if (backward_lds_bytes(np2, ne2, nf2, nimg) > kMaxDynLds) continue;
            np = np2, ne = ne2, nf = nf2;
            wide[o.second] = 0;
        }
    }
    for (int64_t e = 0; e < pl.nel; ++e) {
        const ElemDev &el = pl.elems[e];
        const int npad = 16 * ((el.nloc + 15) / 16);
        if (wide[e]) {
            if (el.nloc - el.nfe > kBackwardWideMaxEnr)
                return fail(c, PUFE_ERR_UNSUPPORTED, "the adjoint kernels hold at most " +
                                                         std::to_string(kBackwardWideMaxEnr) +
                                                         " enriched functions on one element");
            max_nfun_wide = std::max(max_nfun_wide, el.nfun);
        } else {
            max_npad = std::max(max_npad, npad);
            max_nfun = std::max(max_nfun, el.nfun);
            max_nenr = std::max(max_nenr, el.nloc - el.nfe);
        }
        pt_off[e + 1] = pt_off[e] + (int64_t)npad * npad;
    }
    c->bw_lds = backward_lds_bytes(max_npad, max_nenr, max_nfun, nimg);
    c->bw_lds_wide = backward_wide_lds_bytes(max_nfun_wide, nimg);
    if (c->bw_lds > kMaxDynLds || c->bw_lds_wide > kMaxDynLds)
        return fail(c, PUFE_ERR_UNSUPPORTED, "adjoint stage does not fit in LDS");
    c->bw_items.clear();
    c->bw_items_wide.clear();
    const int mg = std::max(pl.max_ngrp, 1);
    // items of elements up to 80 functions first, then the wide ones; the
    // partial-force slots follow that order
    for (int pass = 0; pass < 2; ++pass)
        for (int64_t e = 0; e < pl.nel; ++e) {
            const ElemDev &el = pl.elems[e];
            if ((wide[e] != 0) != (pass == 1)) continue;
            // twice the forward's K-chunks (at most one per leaf): the adjoint's
            // stages cost more, and finer items balance the refined elements
            int64_t nleaf = el.leaf_end - el.leaf_off, nch = std::min<int64_t>(2 * el.nchunk, nleaf);
            for (int64_t ch = 0; ch < nch; ++ch) {
                ItemDev it{};
                it.elem = (int32_t)e;
                it.chunk = (int32_t)ch;
                it.leaf_b = el.leaf_off + ch * nleaf / nch;
                it.leaf_e = el.leaf_off + (ch + 1) * nleaf / nch;
                (pass == 0 ? c->bw_items : c->bw_items_wide).push_back(it);
            }
        }
    if (!c->have_bw) {
        CHECK_HIP(c, c->d_pt_off.upload(pt_off, st), "upload adjoint offsets");
        CHECK_HIP(c, c->d_Pt.alloc((size_t)pt_off[pl.nel]), "alloc adjoint blocks");
        c->have_bw = true;
    }
    // with the moment form, the direct kernels serve the split precisions only
    if (!split && !c->have_adj) {
        const int rc = plan_adjoint_moments(c, pt_off[pl.nel], st);
        if (rc != PUFE_OK) return rc;
        c->have_adj = true;
    }
    if (!split && !c->adj_fold.empty()) return PUFE_OK;
    if (c->have_bw_direct) return PUFE_OK;
    std::vector<std::vector<int64_t>> slots(c->prob.species.size());
    const int64_t nn = (int64_t)c->bw_items.size(), ntot = nn + (int64_t)c->bw_items_wide.size();
    for (int64_t idx = 0; idx < ntot; ++idx) {
        const ItemDev &it = idx < nn ? c->bw_items[idx] : c->bw_items_wide[idx - nn];
        const ElemDev &el = pl.elems[it.elem];
        for (int g = 0; g < el.ngrp; ++g) slots[pl.groups[el.grp_off + g].atom].push_back(idx * mg + g);
    }
    std::vector<int64_t> aptr(slots.size() + 1, 0), aslots;
    for (size_t A = 0; A < slots.size(); ++A) {
        aslots.insert(aslots.end(), slots[A].begin(), slots[A].end());
        aptr[A + 1] = (int64_t)aslots.size();
    }
    CHECK_HIP(c, c->d_bw_items.upload_list(c->bw_items, st), "upload adjoint items");
    CHECK_HIP(c, c->d_bw_items_wide.upload_list(c->bw_items_wide, st), "upload adjoint items");
    CHECK_HIP(c, c->d_atom_ptr.upload(aptr, st), "upload atom lists");
    CHECK_HIP(c, c->d_atom_slots.upload(aslots, st), "upload atom lists");
    CHECK_HIP(c, c->d_fP.alloc((size_t)ntot * mg * 3), "alloc partial forces");
    CHECK_HIP(c, c->d_fQ.alloc((size_t)ntot * mg * 3), "alloc partial forces");
    c->have_bw_direct = true;
    return PUFE_OK;
}

// Moment form of the FP64 adjoint: all elements or none, also where its memory does
// not fit (the direct kernels then serve FP64 too).
static int plan_adjoint_moments(pufe_ctx *c, int64_t pt_doubles, hipStream_t st) {
    Plan &pl = c->plan;
    const int n = pl.kp.n, p = pl.kp.p, mg = std::max(pl.max_ngrp, 1);
    auto drop = [&] {
        for (int w = 0; w < 2; ++w) {
            c->adj_items[w].clear();
            c->adj_lds[w] = 0;
            c->d_adj_items[w].release();
        }
        c->adj_fold.clear();
        c->d_adj_fold.release();
        c->d_adj_base.release();
        c->d_adj_ptr.release();
        c->d_adj_slots.release();
        c->d_adj_lam.release();
        c->d_adj_Qt.release();
        c->d_adj_f.release();
    };
    drop();
    // the fold knows neither the serendipity functions' polynomials nor, on sheared
    // cells, the metric's mixed terms: both stay with the direct kernels
    if (p > 2 || pl.kp.skew) return PUFE_OK;
    std::vector<AdjStage> stages(pl.nel);
    std::vector<double> cost(pl.nel);
    double total = 0.0;
    for (int64_t e = 0; e < pl.nel; ++e) {
        const ElemDev &el = pl.elems[e];
        int nimg = 0;
        if (el.ngrp > 0) {
            const GroupDev &g = pl.groups[el.grp_off + el.ngrp - 1];
            nimg = g.img_off + g.nimg - pl.groups[el.grp_off].img_off;
        }
        stages[e] = adj_stage((el.nfun + 3) / 4, nimg, n, p);
        if (stages[e].waves == 0) return PUFE_OK;
        cost[e] = (double)(el.leaf_end - el.leaf_off) * (adj_tasks((el.nfun + 3) / 4) + 0.5 * el.ngrp + 1.0);
        total += cost[e];
    }
    // four items per resident group of four waves (512), six per group of eight
    // (256): the shortest of 2, 3, 4, 6 and 8 on elements of one and two row tiles
    // and of eight and eleven, by 7 % and 10 % over the next coarser cut
    const double dur[2] = {total / 2048.0, total / 1536.0};
    std::vector<int64_t> order(pl.nel), base(pl.nel + 1, 0);
    for (int64_t e = 0; e < pl.nel; ++e) {
        order[e] = e;
        const int nt = (pl.elems[e].nfun + 3) / 4;
        base[e + 1] = base[e] + adj_doubles(nt, p);
        for (int q = 0; 4 * q < mom_quads_b(nt); ++q) c->adj_fold.push_back(make_int4((int)e, ADJ_PAIRS, q, 0));
        for (int t = 0; t < ((nt + 3) & ~3); ++t) c->adj_fold.push_back(make_int4((int)e, ADJ_MIXED, t, 0));
        c->adj_fold.push_back(make_int4((int)e, ADJ_CLASSICAL, 0, 0));
    }
    std::stable_sort(order.begin(), order.end(), [&](int64_t a, int64_t b) { return cost[a] > cost[b]; });
    // an element's items go to one XCD (work groups are dealt round the eight),
    // next to each other: they read the same coefficients
    std::vector<MomItemDev> queue[2][8];
    double load[2][8] = {};
    for (int64_t e : order) {
        const ElemDev &el = pl.elems[e];
        const AdjStage &s = stages[e];
        const int w = s.waves == 4 ? 0 : 1;
        c->adj_lds[w] = std::max(c->adj_lds[w], s.lds);
        int x = 0;
        for (int k = 1; k < 8; ++k)
            if (load[w][k] < load[w][x]) x = k;
        load[w][x] += cost[e];
        const int64_t nst = (el.leaf_end - el.leaf_off) * (s.planes > 0 ? (n + s.planes - 1) / s.planes
                                                                        : n * ((n + s.lines - 1) / s.lines));
        const int64_t nch = std::max<int64_t>(1, std::min<int64_t>(nst, (int64_t)std::ceil(cost[e] / dur[w])));
        for (int64_t ch = 0; ch < nch; ++ch) {
            MomItemDev it{};
            it.elem = (int32_t)e;
            it.leaf_b = ch * nst / nch;
            it.leaf_e = (ch + 1) * nst / nch;
            it.tab = s.planes | (s.lines << 8);
            queue[w][x].push_back(it);
        }
    }
    std::vector<std::vector<int64_t>> slots(c->prob.species.size());
    int32_t slot = 0;
    for (int w = 0; w < 2; ++w) {
        size_t longest = 0;
        for (int x = 0; x < 8; ++x) longest = std::max(longest, queue[w][x].size());
        for (size_t k = 0; k < longest; ++k)
            for (int x = 0; x < 8; ++x)
                if (k < queue[w][x].size()) {
                    MomItemDev it = queue[w][x][k];
                    it.chunk = slot;
                    c->adj_items[w].push_back(it);
                    const ElemDev &el = pl.elems[it.elem];
                    for (int g = 0; g < el.ngrp; ++g)
                        slots[pl.groups[el.grp_off + g].atom].push_back((int64_t)slot * mg + g);
                    ++slot;
                }
    }
    std::vector<int64_t> aptr(slots.size() + 1, 0), aslots;
    for (size_t A = 0; A < slots.size(); ++A) {
        aslots.insert(aslots.end(), slots[A].begin(), slots[A].end());
        aptr[A + 1] = (int64_t)aslots.size();
    }
    const int64_t forces = (int64_t)slot * mg * 3;
    hipError_t e = moments_fit(c, base[pl.nel] + pt_doubles + forces) ? hipSuccess : hipErrorOutOfMemory;
    if (e == hipSuccess) e = c->d_adj_lam.alloc((size_t)base[pl.nel]);
    if (e == hipSuccess) e = c->d_adj_Qt.alloc((size_t)pt_doubles);
    if (e == hipSuccess) e = c->d_adj_f.alloc((size_t)forces);
    for (int w = 0; w < 2; ++w)
        if (e == hipSuccess) e = c->d_adj_items[w].upload_list(c->adj_items[w], st);
    if (e == hipSuccess) e = c->d_adj_fold.upload(c->adj_fold, st);
    if (e == hipSuccess) e = c->d_adj_base.upload(base, st);
    if (e == hipSuccess) e = c->d_adj_ptr.upload(aptr, st);
    if (e == hipSuccess) e = c->d_adj_slots.upload(aslots, st);
    if (e == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        drop();
        return PUFE_OK;
    }
    CHECK_HIP(c, e, "adjoint tables");
    return PUFE_OK;
}

int pufe_assemble_backward(pufe_ctx *ctx, const double *d_V, const double kpt[3], const void *d_P, const void *d_Q,
                           int precision, double *d_dLdV, double *d_dLdR, void *stream) {
    if (!ctx) return PUFE_ERR_INVALID_ARG;
    if (!ctx->have_setup) return fail(ctx, PUFE_ERR_STATE, "pufe_setup must come first");
    if (!d_V || !kpt) return fail(ctx, PUFE_ERR_INVALID_ARG, "null V or k-point");
    if (precision < PUFE_PREC_FP64 || precision > PUFE_PREC_BF16X6)
        return fail(ctx, PUFE_ERR_INVALID_ARG, "unknown precision");
    const int nl = precision == PUFE_PREC_BF16X3 ? 2 : (precision == PUFE_PREC_BF16X6 ? 3 : 0);
    for (int d = 0; d < 3; ++d)
        if (!std::isfinite(kpt[d])) return fail(ctx, PUFE_ERR_INVALID_ARG, "non-finite k-point");
    if (ctx->plan.bloch)
        return fail(ctx, PUFE_ERR_UNSUPPORTED, "the adjoint of the Bloch-periodic enrichment is not supported");
    hipStream_t st = (hipStream_t)stream;
    CHECK_HIP(ctx, hipSetDevice(ctx->device), "hipSetDevice");
    if (!ctx->have_bw || (nl == 0 && !ctx->have_adj) || ((nl != 0 || ctx->adj_fold.empty()) && !ctx->have_bw_direct)) {
        int rc = plan_backward(ctx, nl != 0, st);
        if (rc != PUFE_OK) return rc;
    }
    const Plan &pl = ctx->plan;
    const int nwide = (int)ctx->bw_items_wide.size();
    if (nl != 0 && nwide > 0)
        return fail(ctx, PUFE_ERR_UNSUPPORTED,
                    "the split-precision adjoint holds elements of at most " + std::to_string(kBackwardMaxNloc) +
                        " functions (use FP64)");
    TimedRegion tr(ctx, 2, st);
    const int mg = std::max(pl.max_ngrp, 1);
    const int nit = (int)ctx->bw_items.size();
    if (nl == 0 && !ctx->adj_fold.empty()) {   // P and Q in one pass
        if (d_P || d_Q) {
            CHECK_HIP(ctx, launch_gather_adjoint(pl.kp, pl.nel, pl.max_nloc, ctx->d_elems.p, ctx->d_edof.p,
                                                 ctx->d_pt_off.p, (const double *)d_P, (const double *)d_Q, kpt,
                                                 ctx->d_Pt.p, ctx->d_adj_Qt.p, st), "gather P and Q");
            CHECK_HIP(ctx, launch_adjoint_fold(ctx->d_self.p, ctx->d_adj_fold.p, (int)ctx->adj_fold.size(),
                                               ctx->d_pt_off.p, d_P ? ctx->d_Pt.p : nullptr,
                                               d_Q ? ctx->d_adj_Qt.p : nullptr, ctx->d_adj_base.p, ctx->d_adj_lam.p, st),
                      "adjoint coefficients");
            for (int w = 1; w >= 0; --w)
                CHECK_HIP(ctx, launch_adjoint_moments(w ? 8 : 4, ctx->d_self.p, ctx->d_adj_items[w].p,
                                                      (int)ctx->adj_items[w].size(), ctx->d_adj_base.p,
                                                      ctx->d_adj_lam.p, d_V, d_P ? d_dLdV : nullptr, ctx->d_adj_f.p, mg,
                                                      ctx->adj_lds[w], st), "adjoint");
        }
        if (!d_P && d_dLdV) CHECK_HIP(ctx, launch_fill_zero(d_dLdV, ctx->n_qp, st), "zero dLdV");
        if (d_dLdR)
            CHECK_HIP(ctx, launch_force_reduce((int)ctx->prob.species.size(), ctx->d_adj_ptr.p, ctx->d_adj_slots.p,
                                               d_P || d_Q ? ctx->d_adj_f.p : nullptr, nullptr, d_dLdR, st),
                      "force reduction");
        return PUFE_OK;
    }
    const size_t wide_slots = (size_t)nit * mg * 3;   // the wide items' partial forces follow the others
    if (d_P) {
        CHECK_HIP(ctx, launch_gather_adjoint(pl.kp, pl.nel, pl.max_nloc, ctx->d_elems.p, ctx->d_edof.p, ctx->d_pt_off.p,
                                             (const double *)d_P, nullptr, kpt, ctx->d_Pt.p, nullptr, st), "gather P");
        CHECK_HIP(ctx, launch_backward(pl.kp, false, nl, nit, ctx->d_bw_items.p, ctx->d_elems.p, ctx->d_groups.p,
                                       ctx->d_img.p, ctx->d_edof.p, ctx->d_leaves.p, d_V, ctx->d_pt_off.p,
                                       ctx->d_Pt.p, d_dLdV, ctx->d_fP.p, mg, ctx->bw_lds, st), "adjoint (P)");
        CHECK_HIP(ctx, launch_backward_wide(pl.kp, false, nwide, ctx->d_bw_items_wide.p, ctx->d_elems.p,
                                            ctx->d_groups.p, ctx->d_img.p, ctx->d_edof.p, ctx->d_leaves.p, d_V,
                                            ctx->d_pt_off.p, ctx->d_Pt.p, d_dLdV, ctx->d_fP.p + wide_slots, mg,
                                            ctx->bw_lds_wide, st), "adjoint (P, wide elements)");
    } else if (d_dLdV) {
        CHECK_HIP(ctx, launch_fill_zero(d_dLdV, ctx->n_qp, st), "zero dLdV");
    }
    if (d_Q) {
        CHECK_HIP(ctx, launch_gather_adjoint(pl.kp, pl.nel, pl.max_nloc, ctx->d_elems.p, ctx->d_edof.p, ctx->d_pt_off.p,
                                             nullptr, (const double *)d_Q, kpt, nullptr, ctx->d_Pt.p, st), "gather Q");
        CHECK_HIP(ctx, launch_backward(pl.kp, true, nl, nit, ctx->d_bw_items.p, ctx->d_elems.p, ctx->d_groups.p,
                                       ctx->d_img.p, ctx->d_edof.p, ctx->d_leaves.p, d_V, ctx->d_pt_off.p,
                                       ctx->d_Pt.p, nullptr, ctx->d_fQ.p, mg, ctx->bw_lds, st), "adjoint (Q)");
        CHECK_HIP(ctx, launch_backward_wide(pl.kp, true, nwide, ctx->d_bw_items_wide.p, ctx->d_elems.p,
                                            ctx->d_groups.p, ctx->d_img.p, ctx->d_edof.p, ctx->d_leaves.p, d_V,
                                            ctx->d_pt_off.p, ctx->d_Pt.p, nullptr, ctx->d_fQ.p + wide_slots, mg,
                                            ctx->bw_lds_wide, st), "adjoint (Q, wide elements)");
    }
    if (d_dLdR)
        CHECK_HIP(ctx, launch_force_reduce((int)ctx->prob.species.size(), ctx->d_atom_ptr.p, ctx->d_atom_slots.p,
                                           d_P ? ctx->d_fP.p : nullptr, d_Q ? ctx->d_fQ.p : nullptr, d_dLdR, st),
                  "force reduction");
    return PUFE_OK;
}

int pufe_set_positions(pufe_ctx *ctx, const double *pos) {
    if (!ctx || !pos) return PUFE_ERR_INVALID_ARG;
    if (!ctx->have_problem) return fail(ctx, PUFE_ERR_STATE, "no problem defined");
    Plan &pl = ctx->plan;
    const size_t na = ctx->prob.species.size();
    for (size_t A = 0; A < na; ++A) {
        double d2 = 0;
        for (int c = 0; c < 3; ++c) {
            if (!std::isfinite(pos[3 * A + c])) return fail(ctx, PUFE_ERR_INVALID_ARG, "non-finite position");
            double d = pos[3 * A + c] - ctx->prob.pos[3 * A + c];
            d2 += d * d;
        }
        if (std::sqrt(d2) > kImageMargin)
            return fail(ctx, PUFE_ERR_INVALID_ARG, "an enrichment centre moved farther than the image margin");
    }
    // shift every image centre of a group by its atom's displacement
    for (const ElemDev &el : pl.elems)
        for (int g = 0; g < el.ngrp; ++g) {
            const GroupDev &G = pl.groups[el.grp_off + g];
            for (int k = 0; k < G.nimg; ++k)
                for (int c = 0; c < 3; ++c)
                    pl.img_cur[3 * (G.img_off + k) + c] = pl.img[3 * (G.img_off + k) + c] +
                                                          (pos[3 * G.atom + c] - ctx->prob.pos[3 * G.atom + c]);
        }
    if (ctx->have_setup) {
        CHECK_HIP(ctx, hipSetDevice(ctx->device), "hipSetDevice");
        CHECK_HIP(ctx, hipMemcpy(ctx->d_img.p, pl.img_cur.data(), sizeof(double) * pl.img_cur.size(),
                                 hipMemcpyHostToDevice), "upload image centres");
    }
    return PUFE_OK;
}

int pufe_bsr_to_dense(pufe_ctx *ctx, const void *d_bsr, int dtype, double *d_dense, void *stream) {
    if (!ctx) return PUFE_ERR_INVALID_ARG;
    if (!ctx->have_setup) return fail(ctx, PUFE_ERR_STATE, "pufe_setup must come first");
    if (!d_bsr || !d_dense) return fail(ctx, PUFE_ERR_INVALID_ARG, "null pointer");
    if (dtype != PUFE_OUT_C128 && dtype != PUFE_OUT_F64_GAMMA)
        return fail(ctx, PUFE_ERR_INVALID_ARG, "dense expansion takes C128 or F64_GAMMA values");
    hipStream_t st = (hipStream_t)stream;
    CHECK_HIP(ctx, hipSetDevice(ctx->device), "hipSetDevice");
    const Plan &pl = ctx->plan;
    int64_t n = pl.dof_off[pl.nv];
    CHECK_HIP(ctx, launch_fill_zero(d_dense, 2 * n * n, st), "zero dense");
    CHECK_HIP(ctx, launch_bsr_to_dense((int64_t)pl.bcol.size(), ctx->d_brow.p, ctx->d_bcol.p, ctx->d_bval_off.p,
                                       ctx->d_dof_off.p, d_bsr, dtype == PUFE_OUT_C128 ? 0 : 1, n, d_dense, st),
              "bsr to dense");
    return PUFE_OK;
}

int pufe_enable_timing(pufe_ctx *ctx, int on) {
    if (!ctx) return PUFE_ERR_INVALID_ARG;
    ctx->timing = on != 0;
    return PUFE_OK;
}

int pufe_kernel_times(pufe_ctx *ctx, double *out_ms, int64_t *counts, int reset) {
    if (!ctx) return PUFE_ERR_INVALID_ARG;
    for (int k = 0; k < 5; ++k) {
        double ms = 0.0;
        for (auto &pr : ctx->ev[k]) {
            CHECK_HIP(ctx, hipEventSynchronize(pr.second), "event sync");
            float t = 0.f;
            CHECK_HIP(ctx, hipEventElapsedTime(&t, pr.first, pr.second), "event time");
            ms += t;
        }
        if (out_ms) out_ms[k] = ms;
        if (counts) counts[k] = (int64_t)ctx->ev[k].size();
    }
    if (reset) ctx->clear_events();
    return PUFE_OK;
}

// Device tables and slots of the moment form for the current plan, and the
// problem's own entry of a list of problems (the other tables are in place).
static int upload_moments(pufe_ctx *ctx, hipStream_t st) {
    for (int w = 0; w < 3; ++w)
        CHECK_HIP(ctx, ctx->d_mom_items[w].upload_list(ctx->mom_items[w], st), "upload work items");
    CHECK_HIP(ctx, ctx->d_mom_tasks.upload_list(ctx->mom_tasks, st), "upload wave tasks");
    CHECK_HIP(ctx, ctx->d_mom_reduce.upload_list(ctx->mom_reduce, st), "upload chunk reduction list");
    CHECK_HIP(ctx, ctx->d_mom_expand.upload_list(ctx->mom_expand, st), "upload expansion list");
    ctx->d_mom.release();
    ctx->d_mom_na.release();
    if (ctx->mom_doubles > 0) {
        if (!moments_fit(ctx, ctx->mom_doubles)) return PUFE_ERR_OOM;
        CHECK_HIP(ctx, ctx->d_mom.alloc((size_t)ctx->mom_doubles), "alloc moments");
    }
    std::vector<CtxDev> self(2, tables_of(ctx));
    // the allocation-free entry may overlap pufe_assemble on another stream: its
    // moments lie behind its partial tiles or in slots of their own
    const size_t tiles = noalloc_bytes(ctx);
    if (ctx->mom_doubles > 0 && tiles <= kScratchBytes) {
        if (tiles + (size_t)ctx->mom_doubles * sizeof(double) <= kScratchBytes) {
            double *ws = nullptr;
            CHECK_HIP(ctx, scratch_address(ctx->device, &ws), "workspace address");
            self[1].mom = ws + tiles / sizeof(double);
        } else {
            if (!moments_fit(ctx, ctx->mom_doubles)) return PUFE_ERR_OOM;
            CHECK_HIP(ctx, ctx->d_mom_na.alloc((size_t)ctx->mom_doubles), "alloc moments");
            self[1].mom = ctx->d_mom_na.p;
        }
    }
    CHECK_HIP(ctx, ctx->d_self.upload(self, st), "upload tables");
    return PUFE_OK;
}

// The moment form's tables and slots, after the other tables of the plan; where
// there is no memory for them, a plan of direct kernels alone (the partial tiles,
// the split kernels' items and the projectors' stay as they are).
static int place_moments(pufe_ctx *ctx, hipStream_t st) {
    int rc = upload_moments(ctx, st);
    if (rc != PUFE_ERR_OOM || ctx->mom_doubles == 0) return rc;
    (void)hipGetLastError();
    plan_items(ctx, ctx->planned_items, ctx->planned_block, false);
    if (ctx->lds > kMaxDynLds) return fail(ctx, PUFE_ERR_UNSUPPORTED, "contraction stage does not fit in LDS");
    CHECK_HIP(ctx, ctx->d_elems.upload(ctx->plan.elems, st), "upload elements");
    CHECK_HIP(ctx, ctx->d_items.upload_list(ctx->items, st), "upload work items");
    CHECK_HIP(ctx, ctx->d_items_wide.upload_list(ctx->items_wide, st), "upload work items");
    CHECK_HIP(ctx, ctx->d_reduce_f64.upload_list(ctx->reduce_f64, st), "upload chunk reduction list");
    return upload_moments(ctx, st);
}

// Upload the element table, work items and partial buffer of the current plan.
static int upload_items(pufe_ctx *ctx, hipStream_t st) {
    ++ctx->plan_gen;
    ctx->have_bw = ctx->have_adj = ctx->have_bw_direct = false;
    ctx->have_poisson = false;
    CHECK_HIP(ctx, ctx->d_elems.upload(ctx->plan.elems, st), "upload elements");
    CHECK_HIP(ctx, ctx->d_items.upload_list(ctx->items, st), "upload work items");
    CHECK_HIP(ctx, ctx->d_items_wide.upload_list(ctx->items_wide, st), "upload work items");
    CHECK_HIP(ctx, ctx->d_items_split.upload_list(ctx->items_split, st), "upload work items");
    CHECK_HIP(ctx, ctx->d_reduce.upload_list(ctx->reduce, st), "upload chunk reduction list");
    CHECK_HIP(ctx, ctx->d_reduce_f64.upload_list(ctx->reduce_f64, st), "upload chunk reduction list");
    CHECK_HIP(ctx, ctx->d_partial.alloc((size_t)ctx->part_slots * 512), "alloc partial tiles");
    {
        int rc = upload_nonlocal(ctx, st);
        if (rc == PUFE_OK) rc = place_moments(ctx, st);
        if (rc != PUFE_OK) return rc;
    }
    return PUFE_OK;
}

int pufe_tune(pufe_ctx *ctx, int precision, const char *cache_path) {
    if (!ctx) return PUFE_ERR_INVALID_ARG;
    if (!ctx->have_setup) return fail(ctx, PUFE_ERR_STATE, "pufe_setup must come first");
    if (precision < PUFE_PREC_FP64 || precision > PUFE_PREC_BF16X6)
        return fail(ctx, PUFE_ERR_INVALID_ARG, "unknown precision");
    CHECK_HIP(ctx, hipSetDevice(ctx->device), "hipSetDevice");
    const Plan &pl = ctx->plan;
    int64_t sum_nloc = 0;
    for (const ElemDev &el : pl.elems) sum_nloc += el.nloc;
    char key[256];
    hipDeviceProp_t prop;
    CHECK_HIP(ctx, hipGetDeviceProperties(&prop, ctx->device), "device properties");
    std::snprintf(key, sizeof key, "%s|prec%d|nel%lld|leaves%lld|n3_%d|nloc%lld|maxnloc%d", prop.gcnArchName, precision,
                  (long long)pl.nel, (long long)ctx->n_leaves, pl.kp.n3, (long long)sum_nloc, pl.max_nloc);
    // cached choice?
    std::string text;
    if (cache_path) {
        if (FILE *f = std::fopen(cache_path, "rb")) {
            char buf[4096];
            size_t r;
            while ((r = std::fread(buf, 1, sizeof buf, f)) > 0) text.append(buf, r);
            std::fclose(f);
        }
        std::string pat = std::string("\"") + key + "\": {\"items\": ";
        size_t at = text.find(pat);
        if (at != std::string::npos) {
            double items = 0;
            int block = 0, qv = 0, wide = kWideTiles;
            const int nf = std::sscanf(text.c_str() + at + pat.size(), "%lf, \"block\": %d, \"q\": %d, \"wide\": %d",
                                       &items, &block, &qv, &wide);
            if (nf >= 3 && items > 0 && block >= 1 && block <= kBlockTiles && contract_q_supported(qv) &&
                (wide == 0 || (wide >= 2 && wide <= kWideTiles))) {
                ctx->tune_items = items;
                ctx->tune_block = block;
                ctx->contract_q = qv;
                ctx->wide_tiles = wide;
                ctx->tuned = true;
                plan_items(ctx, items, block);
                const int rc = upload_items(ctx, nullptr);
                ctx->have_setup = rc == PUFE_OK;
                return rc;
            }
        }
    }
    DevBuf<double> V;
    CHECK_HIP(ctx, V.alloc(std::max<int64_t>(ctx->n_qp, 1)), "alloc timing input");
    CHECK_HIP(ctx, hipMemset(V.p, 0, sizeof(double) * V.n), "zero timing input");
    hipEvent_t a, b;
    CHECK_HIP(ctx, hipEventCreate(&a), "event");
    CHECK_HIP(ctx, hipEventCreate(&b), "event");
    const bool saved = ctx->timing;
    ctx->timing = false;
    // Coordinate descent from the current choice: the item count first, then
    // the tile block, then the stage length, each candidate timed once after
    // a warm-up run (a problem of a few hundred milliseconds per assembly is
    // tuned in seconds rather than minutes).
    double best = 1e300, best_items = ctx->tune_items;
    int best_block = ctx->tune_block, best_q = ctx->contract_q, best_wide = ctx->wide_tiles;
    struct Tried {
        double items;
        int block, q, wide;
    };
    std::vector<Tried> tried;
    auto trial = [&](double items, int block, int qv, int wide) -> int {
        for (auto &t : tried)
            if (t.items == items && t.block == block && t.q == qv && t.wide == wide) return PUFE_OK;
        tried.push_back({items, block, qv, wide});
        ctx->contract_q = qv;
        ctx->wide_tiles = wide;
        plan_items(ctx, items, block);
        if (ctx->lds > kMaxDynLds || ctx->contract_q != qv) return PUFE_OK;   // does not fit: skip
        int rc = upload_items(ctx, nullptr);
        if (rc != PUFE_OK) return rc;
        rc = run_contraction(ctx, V.p, precision, nullptr, ctx->d_partial.p);   // warm-up
        if (rc != PUFE_OK) return rc;
        CHECK_HIP(ctx, hipEventRecord(a, nullptr), "event");
        rc = run_contraction(ctx, V.p, precision, nullptr, ctx->d_partial.p);
        if (rc != PUFE_OK) return rc;
        CHECK_HIP(ctx, hipEventRecord(b, nullptr), "event");
        CHECK_HIP(ctx, hipEventSynchronize(b), "event");
        float ms = 0;
        CHECK_HIP(ctx, hipEventElapsedTime(&ms, a, b), "event");
        if (ms < best) {
            best = ms;
            best_items = items;
            best_block = block;
            best_q = qv;
            best_wide = wide;
        }
        return PUFE_OK;
    };
    int trc = PUFE_OK;
    // with every element in moment form all candidates would time the same FP64
    // launches, and chance would set the K-chunks (the size of the partial tiles,
    // the order of the projectors' sums): the current choice stays
    const bool choice = precision != PUFE_PREC_FP64 || !ctx->items.empty() || !ctx->items_wide.empty();
    const int start_block = ctx->tune_block, start_q = ctx->contract_q, start_wide = ctx->wide_tiles;
    if (!choice) trc = trial(best_items, start_block, start_q, start_wide);
    for (double items : {1024.0, 2048.0, 4096.0, 8192.0, 16384.0})
        if (choice && trc == PUFE_OK) trc = trial(items, start_block, start_q, start_wide);
    for (int block = 2; choice && block <= kBlockTiles && trc == PUFE_OK; ++block)
        trc = trial(best_items, block, start_q, start_wide);
    for (int qv : {16, 24, 32})
        if (choice && trc == PUFE_OK) trc = trial(best_items, best_block, qv, start_wide);
    if (choice && pl.max_nloc > 16 * kWholeMaxTiles)   // elements for the wide kernel
        for (int wide : {kWideTiles, kWideTiles - 1, 0})
            if (trc == PUFE_OK) trc = trial(best_items, best_block, best_q, wide);
    (void)hipEventDestroy(a);
    (void)hipEventDestroy(b);
    if (trc != PUFE_OK) {
        ctx->timing = saved;
        ctx->have_setup = false;   // the plan of a trial, in part
        return trc;
    }
    ctx->timing = saved;
    ctx->tune_items = best_items;
    ctx->tune_block = best_block;
    ctx->contract_q = best_q;
    ctx->wide_tiles = best_wide;
    ctx->tuned = true;
    plan_items(ctx, best_items, best_block);
    int rc = upload_items(ctx, nullptr);
    ctx->have_setup = rc == PUFE_OK;
    if (rc != PUFE_OK) return rc;
    if (cache_path) {
        // append or insert the entry into a flat JSON object
        char entry[512];
        std::snprintf(entry, sizeof entry, "\"%s\": {\"items\": %.0f, \"block\": %d, \"q\": %d, \"wide\": %d, \"ms\": %.4f}",
                      key, best_items, best_block, best_q, best_wide, best);
        size_t close = text.rfind('}');
        std::string out;
        if (close == std::string::npos || text.find('{') == std::string::npos)
            out = std::string("{\n  ") + entry + "\n}\n";
        else {
            std::string head = text.substr(0, close);
            while (!head.empty() && (head.back() == '\n' || head.back() == ' ')) head.pop_back();
            out = head + (head.back() == '{' ? "\n  " : ",\n  ") + entry + "\n}\n";
        }
        if (FILE *f = std::fopen(cache_path, "wb")) {
            std::fwrite(out.data(), 1, out.size(), f);
            std::fclose(f);
        }
    }
    return PUFE_OK;
}

// stage lengths of the batch's FP64 classes, longest first; each has a class
// of problems sharing a CU two work groups at a time and one of the rest
static const int kBatchQ[3] = {32, 24, 16};
constexpr int kBatchClasses = 6;

struct pufe_batch {
    std::vector<pufe_ctx *> ctxs;
    std::vector<uint64_t> gens;             // plan generation of each context at creation
    int device = 0;
    std::vector<ItemDev> items, items_split;
    std::vector<int4> blocks;               // assembly list of all problems (gather.hpp)
    GatherSizes gather;
    // FP64 items in up to kBatchClasses classes, each a persistent launch of
    // its own (items [item_off[c], item_off[c + 1])): per stage length, the
    // problems whose combined stage fits two work groups per CU, then the rest
    size_t lds_f64[kBatchClasses] = {}, lds_split[2] = {0, 0};
    int max_l = 0, q[kBatchClasses] = {};
    bool gen = false;                       // some problem needs the general kernel variant
    int grid_f64[kBatchClasses] = {}, grid_split[2] = {0, 0};
    int64_t item_off[kBatchClasses + 1] = {};
    // wide items of all problems (8-wave persistent launch)
    std::vector<ItemDev> items_wide;
    size_t lds_wide = 0;
    int grid_wide = 0;
    DevBuf<CtxDev> d_ctxs;
    DevBuf<ItemDev> d_items, d_items_split, d_items_wide;
    DevBuf<int4> d_blocks;
    // (problem, element, tile pair) of multi-chunk elements: all, and those on the direct FP64 kernels
    std::vector<int4> reduce, reduce_f64;
    DevBuf<int4> d_reduce, d_reduce_f64;
    // moment form: items of all problems by work group width (index / 3: 4 or 8
    // waves) and x steps of the rule (index % 3: 1..3); index 6: classical part
    std::vector<MomItemDev> mom_items[7];
    bool skew = false;                      // some cell is skewed
    std::vector<int32_t> mom_tasks;
    std::vector<int4> mom_reduce, mom_expand;
    size_t mom_lds[7] = {};
    DevBuf<MomItemDev> d_mom_items[7];
    DevBuf<int32_t> d_mom_tasks;
    DevBuf<int4> d_mom_reduce, d_mom_expand;
    DevBuf<int> d_counter;
    hipStream_t cap = nullptr;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    std::vector<uintptr_t> key;
    std::string err;
    ~pufe_batch() {
        if (exec) (void)hipGraphExecDestroy(exec);
        if (graph) (void)hipGraphDestroy(graph);
        if (cap) (void)hipStreamDestroy(cap);
    }
};

static int bfail(pufe_batch *b, int code, const std::string &msg) {
    if (b) b->err = msg;
    return code;
}

#define CHECK_HIP_B(b, x, where)                                                               \
    do {                                                                                       \
        hipError_t e_ = (x);                                                                   \
        if (e_ != hipSuccess)                                                                  \
            return bfail(b, e_ == hipErrorOutOfMemory ? PUFE_ERR_OOM : PUFE_ERR_HIP,            \
                         std::string(where) + ": " + hipGetErrorString(e_));                   \
    } while (0)

static double item_cost(const ItemDev &it, int n3) {
    const int pairs = it.I0 == it.J0 ? it.nI * (it.nI + 1) / 2 : it.nI * it.nJ;
    return (double)pairs * (double)(it.leaf_e - it.leaf_b) * n3;
}

int pufe_batch_create(pufe_batch **out, pufe_ctx *const *ctxs, int n) {
    if (!out || !ctxs || n < 1) return PUFE_ERR_INVALID_ARG;
    pufe_batch *b = new (std::nothrow) pufe_batch();
    if (!b) return PUFE_ERR_OOM;
    for (int i = 0; i < n; ++i) {
        if (!ctxs[i] || !ctxs[i]->have_setup || ctxs[i]->device != ctxs[0]->device) {
            delete b;
            return PUFE_ERR_STATE;
        }
        if (ctxs[i]->plan.n_pfun > 0 || ctxs[i]->plan.bloch) {   // no nonlocal or per-k launches in the batch graph
            delete b;
            return PUFE_ERR_UNSUPPORTED;
        }
        b->ctxs.push_back(ctxs[i]);
        b->gens.push_back(ctxs[i]->plan_gen);
    }
    b->device = ctxs[0]->device;
    if (hipSetDevice(b->device) != hipSuccess) { delete b; return PUFE_ERR_HIP; }
    int max_rows_split = 16, max_nfun = 1, max_img = 0, max_leaves_split = 1, max_n3 = 1;
    // FP64 classes.  Each problem keeps its own stage length (the one pufe_tune
    // chose, else the library default); the problems of one length, in order of
    // their own stage size, join that length's first class while the class's
    // combined stage still fits two work groups per CU, the others its second.
    std::vector<int> cls(n, 0);
    for (int qi = 0; qi < 3; ++qi) {
        const int qv = kBatchQ[qi];
        std::vector<std::pair<size_t, int>> by_lds;
        for (int i = 0; i < n; ++i) {
            const pufe_ctx *c = ctxs[i];
            const int qc = contract_q_supported(c->contract_q) ? c->contract_q : 24;
            if (qc != qv) continue;
            by_lds.push_back({contract_lds_bytes(qv, c->max_rows, std::max(c->plan.max_nfun, 1), c->plan.max_img,
                                                 c->max_item_leaves, c->plan.kp.n3), i});
        }
        std::stable_sort(by_lds.begin(), by_lds.end());
        int r = 16, f = 1, im = 0, lv = 1, n3 = 1;
        for (const auto &pr : by_lds) {
            const pufe_ctx *c = ctxs[pr.second];
            const int r2 = std::max(r, c->max_rows), f2 = std::max(f, c->plan.max_nfun), im2 = std::max(im, c->plan.max_img);
            const int lv2 = std::max(lv, c->max_item_leaves), n32 = std::max(n3, c->plan.kp.n3);
            cls[pr.second] = 2 * qi + 1;
            if (persistent_blocks_per_cu(contract_lds_bytes(qv, r2, f2, im2, lv2, n32)) < 2) continue;
            r = r2, f = f2, im = im2, lv = lv2, n3 = n32;
            cls[pr.second] = 2 * qi;
        }
    }
    for (int pass = 0; pass < kBatchClasses + 2; ++pass) {
        // passes 0 .. kBatchClasses-1: FP64 items of each class; then the
        // split items and the wide FP64 items
        const int split_pass = kBatchClasses, wide_pass = kBatchClasses + 1;
        std::vector<std::pair<double, size_t>> order;
        std::vector<ItemDev> all;
        for (int i = 0; i < n; ++i) {
            pufe_ctx *c = ctxs[i];
            if (pass < split_pass && cls[i] != pass) continue;
            for (const ItemDev &it0 : pass < split_pass ? c->items : (pass == split_pass ? c->items_split : c->items_wide)) {
                ItemDev it = it0;
                it.ctx = i;
                order.push_back({item_cost(it, c->plan.kp.n3), all.size()});
                all.push_back(it);
            }
        }
        std::stable_sort(order.begin(), order.end(),
                         [](const std::pair<double, size_t> &a, const std::pair<double, size_t> &c) { return a.first > c.first; });
        std::vector<ItemDev> &dst = pass < split_pass ? b->items : (pass == split_pass ? b->items_split : b->items_wide);
        for (auto &o : order) dst.push_back(all[o.second]);
        if (pass < split_pass) b->item_off[pass + 1] = (int64_t)b->items.size();
    }
    int cr[kBatchClasses], cf[kBatchClasses], ci[kBatchClasses], cl[kBatchClasses], cn3[kBatchClasses];
    bool all_tuned[kBatchClasses];
    for (int k = 0; k < kBatchClasses; ++k) cr[k] = 16, cf[k] = 1, ci[k] = 0, cl[k] = 1, cn3[k] = 1, all_tuned[k] = true;
    for (int i = 0; i < n; ++i) {
        pufe_ctx *c = ctxs[i];
        const int k = cls[i];
        cr[k] = std::max(cr[k], c->max_rows);
        cf[k] = std::max(cf[k], c->plan.max_nfun);
        ci[k] = std::max(ci[k], c->plan.max_img);
        cl[k] = std::max(cl[k], c->max_item_leaves);
        cn3[k] = std::max(cn3[k], c->plan.kp.n3);
        all_tuned[k] = all_tuned[k] && c->tuned;
        max_rows_split = std::max(max_rows_split, c->max_rows_split);
        max_nfun = std::max(max_nfun, c->plan.max_nfun);
        max_img = std::max(max_img, c->plan.max_img);
        max_leaves_split = std::max(max_leaves_split, c->max_item_leaves_split);
        max_n3 = std::max(max_n3, c->plan.kp.n3);
        b->max_l = std::max(b->max_l, c->plan.max_l);
        b->gen = b->gen || general_variant(c->plan);
        if (!c->items_wide.empty()) b->lds_wide = std::max(b->lds_wide, c->lds_wide);
        for (const int2 &r : c->reduce) b->reduce.push_back(make_int4(i, r.x, r.y, 0));
        for (const int2 &r : c->reduce_f64) b->reduce_f64.push_back(make_int4(i, r.x, r.y, 0));
        for (int4 r : c->mom_reduce) {
            r.w = i;
            b->mom_reduce.push_back(r);
        }
        for (int4 r : c->mom_expand) {
            r.w = i;
            b->mom_expand.push_back(r);
        }
    }
    // assembly list: the small blocks of the problems that list them apart go last
    for (int part = 0; part < 2; ++part)
        for (int i = 0; i < n; ++i) {
            const Plan &pl = ctxs[i]->plan;
            const size_t cut = pl.blocks.size() - pl.gather.small;
            for (size_t k = part ? cut : 0; k < (part ? pl.blocks.size() : cut); ++k) {
                b->blocks.push_back(pl.blocks[k]);
                b->blocks.back().w |= i;
            }
        }
    b->gather.blocks = (int)b->blocks.size();
    for (int i = 0; i < n; ++i) {
        b->gather.small += ctxs[i]->plan.gather.small;
        b->gather.max_entries = std::max(b->gather.max_entries, ctxs[i]->plan.gather.max_entries);
    }
    // moment items of all problems, longest first, over the joined wave tasks
    for (int i = 0; i < n; ++i) b->skew = b->skew || ctxs[i]->plan.kp.skew != 0;
    for (int w = 0; w < 7; ++w) {
        std::vector<std::pair<double, MomItemDev>> all;
        int base = 0;
        for (int i = 0; i < n; ++i) {
            pufe_ctx *c = ctxs[i];
            if (w == 6 || (c->plan.kp.n + 3) / 4 == w % 3 + 1) {
                for (size_t k = 0; k < c->mom_items[w / 3].size(); ++k) {
                    MomItemDev it = c->mom_items[w / 3][k];
                    it.ctx = i;
                    it.tab += base;
                    all.push_back({c->mom_cost[w / 3][k], it});
                }
                b->mom_lds[w] = std::max(b->mom_lds[w], c->mom_lds[w / 3]);
            }
            if (w == 0) b->mom_tasks.insert(b->mom_tasks.end(), c->mom_tasks.begin(), c->mom_tasks.end());
            base += (int)c->mom_tasks.size();
        }
        std::stable_sort(all.begin(), all.end(),
                         [](const std::pair<double, MomItemDev> &a, const std::pair<double, MomItemDev> &c) { return a.first > c.first; });
        for (auto &a : all) b->mom_items[w].push_back(a.second);
    }
    int ncu = 0;
    if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, b->device) != hipSuccess || ncu < 1) ncu = 256;
    // a first class runs at its stage length, two work groups per CU.  A
    // second class keeps its length when every member was tuned (the tuner
    // timed that length against its LDS occupancy) or when two work groups
    // still share a CU; otherwise it runs 16-point stages, two per CU.
    for (int k = 0; k < kBatchClasses; ++k) {
        const int qv = kBatchQ[k / 2];
        b->q[k] = qv;
        b->lds_f64[k] = contract_lds_bytes(qv, cr[k], cf[k], ci[k], cl[k], cn3[k]);
        const bool keep = all_tuned[k] && b->lds_f64[k] <= kMaxDynLds;
        if ((k & 1) && qv > 16 && !keep && persistent_blocks_per_cu(b->lds_f64[k]) < 2) {
            b->q[k] = 16;
            b->lds_f64[k] = contract_lds_bytes(16, cr[k], cf[k], ci[k], cl[k], cn3[k]);
        }
        b->grid_f64[k] = ncu * std::max(persistent_blocks_per_cu(b->lds_f64[k]), 1);
    }
    for (int k = 0; k < 2; ++k) {
        b->lds_split[k] = split_lds_bytes(k + 2, max_rows_split, max_nfun, max_img, max_leaves_split, max_n3);
        b->grid_split[k] = ncu * persistent_blocks_per_cu(b->lds_split[k]);
    }
    // the wide items' stage: each problem's own fits, and one wide work group
    // per CU; the largest stage of the problems serves all of them
    {
        int rw = 16, lw = 1;
        for (int i = 0; i < n; ++i)
            if (!ctxs[i]->items_wide.empty()) {
                rw = std::max(rw, ctxs[i]->max_rows_wide);
                lw = std::max(lw, ctxs[i]->max_item_leaves_wide);
            }
        if (!b->items_wide.empty()) b->lds_wide = contract_wide_lds_bytes(rw, max_nfun, max_img, lw, max_n3);
        b->grid_wide = ncu;
    }
    hipStream_t st = nullptr;
    if (b->d_items.upload(b->items, st) != hipSuccess || b->d_items_split.upload(b->items_split, st) != hipSuccess ||
        b->d_items_wide.upload(b->items_wide, st) != hipSuccess ||
        b->d_blocks.upload(b->blocks, st) != hipSuccess || b->d_reduce.upload(b->reduce, st) != hipSuccess ||
        b->d_reduce_f64.upload(b->reduce_f64, st) != hipSuccess ||
        b->d_mom_items[0].upload(b->mom_items[0], st) != hipSuccess ||
        b->d_mom_items[1].upload(b->mom_items[1], st) != hipSuccess ||
        b->d_mom_items[2].upload(b->mom_items[2], st) != hipSuccess ||
        b->d_mom_items[3].upload(b->mom_items[3], st) != hipSuccess ||
        b->d_mom_items[4].upload(b->mom_items[4], st) != hipSuccess ||
        b->d_mom_items[5].upload(b->mom_items[5], st) != hipSuccess ||
        b->d_mom_items[6].upload(b->mom_items[6], st) != hipSuccess ||
        b->d_mom_tasks.upload(b->mom_tasks, st) != hipSuccess || b->d_mom_reduce.upload(b->mom_reduce, st) != hipSuccess ||
        b->d_mom_expand.upload(b->mom_expand, st) != hipSuccess ||
        b->d_counter.alloc(1) != hipSuccess || b->d_ctxs.alloc(n) != hipSuccess ||
        hipStreamCreateWithFlags(&b->cap, hipStreamNonBlocking) != hipSuccess) {
        delete b;
        return PUFE_ERR_OOM;
    }
    *out = b;
    return PUFE_OK;
}

int pufe_batch_destroy(pufe_batch *b) {
    if (!b) return PUFE_ERR_INVALID_ARG;
    (void)hipSetDevice(b->device);
    delete b;
    return PUFE_OK;
}

int pufe_batch_assemble(pufe_batch *b, const double *const *d_V, const double *kpts, int n_k, int precision,
                        int out_dtype, void *const *d_H, void *const *d_S, void *stream) {
    if (!b) return PUFE_ERR_INVALID_ARG;
    const int n = (int)b->ctxs.size();
    if (!d_V || !d_H || !kpts || n_k < 1 || n_k > kMaxKPerLaunch)
        return bfail(b, PUFE_ERR_INVALID_ARG, "null pointer or n_k outside 1..16");
    if (precision < PUFE_PREC_FP64 || precision > PUFE_PREC_BF16X6 || out_dtype < PUFE_OUT_C128 ||
        out_dtype > PUFE_OUT_F64_GAMMA)
        return bfail(b, PUFE_ERR_INVALID_ARG, "unknown precision or dtype");
    for (int i = 0; i < n; ++i)
        if (!d_V[i] || !d_H[i]) return bfail(b, PUFE_ERR_INVALID_ARG, "null V or H pointer");
    for (int i = 0; i < n; ++i)
        if (b->ctxs[i]->plan_gen != b->gens[i])
            return bfail(b, PUFE_ERR_STATE, "problem " + std::to_string(i) +
                                                " was set up or tuned again after pufe_batch_create; create the batch anew");
    for (int k = 0; k < 3 * n_k; ++k) {
        if (!std::isfinite(kpts[k])) return bfail(b, PUFE_ERR_INVALID_ARG, "non-finite k-point");
        if (out_dtype == PUFE_OUT_F64_GAMMA && std::fmod(kpts[k], 1.0) != 0.0)
            return bfail(b, PUFE_ERR_INVALID_ARG, "real output needs Gamma");
    }
    hipStream_t st = (hipStream_t)stream;
    CHECK_HIP_B(b, hipSetDevice(b->device), "hipSetDevice");
    std::vector<uintptr_t> key;
    key.push_back((uintptr_t)precision);
    key.push_back((uintptr_t)out_dtype);
    key.push_back((uintptr_t)n_k);
    for (int i = 0; i < n; ++i) {
        key.push_back((uintptr_t)d_V[i]);
        key.push_back((uintptr_t)d_H[i]);
        key.push_back((uintptr_t)(d_S ? d_S[i] : nullptr));
    }
    for (int k = 0; k < 3 * n_k; ++k) {
        uint64_t bits;
        std::memcpy(&bits, &kpts[k], sizeof bits);
        key.push_back((uintptr_t)bits);
    }
    if (!b->exec || key != b->key) {
        if (b->exec) (void)hipGraphExecDestroy(b->exec);
        if (b->graph) (void)hipGraphDestroy(b->graph);
        b->exec = nullptr;
        b->graph = nullptr;
        std::vector<CtxDev> cd(n);
        for (int i = 0; i < n; ++i) {
            pufe_ctx *c = b->ctxs[i];
            cd[i] = tables_of(c);
            cd[i].V = d_V[i];
            cd[i].H = d_H[i];
            cd[i].S = d_S ? d_S[i] : nullptr;
        }
        CHECK_HIP_B(b, hipMemcpy(b->d_ctxs.p, cd.data(), sizeof(CtxDev) * n, hipMemcpyHostToDevice), "upload tables");
        KPoints kps;
        std::memset(&kps, 0, sizeof kps);
        kps.nk = n_k;
        for (int k = 0; k < n_k; ++k)
            for (int d = 0; d < 3; ++d) kps.kap[k][d] = kpts[3 * k + d];
        CHECK_HIP_B(b, hipStreamBeginCapture(b->cap, hipStreamCaptureModeThreadLocal), "begin capture");
        hipError_t e = hipSuccess;
        if (precision == PUFE_PREC_FP64) {
            // one persistent launch per class (the queue counter is reset by each)
            for (int k = 0; k < kBatchClasses && e == hipSuccess; ++k) {
                const int cnt = (int)(b->item_off[k + 1] - b->item_off[k]);
                if (cnt == 0) continue;
                if (b->lds_f64[k] > kMaxDynLds) {
                    e = hipErrorInvalidValue;
                    break;
                }
                e = launch_contract_persistent(b->q[k], b->max_l, b->gen, b->d_ctxs.p, b->d_items.p + b->item_off[k], cnt,
                                               b->d_counter.p, b->grid_f64[k], b->lds_f64[k], b->cap);
            }
            if (e == hipSuccess && !b->items_wide.empty()) {
                if (b->lds_wide > kMaxDynLds) e = hipErrorInvalidValue;
                else
                    e = launch_contract_wide_persistent(b->max_l, b->gen, b->d_ctxs.p, b->d_items_wide.p,
                                                        (int)b->items_wide.size(), b->d_counter.p, b->grid_wide,
                                                        b->lds_wide, b->cap);
            }
            if (e == hipSuccess)
                e = launch_classical_moments(b->d_ctxs.p, b->d_mom_items[6].p, (int)b->mom_items[6].size(), nullptr, b->cap);
            for (int w = 5; w >= 0 && e == hipSuccess; --w)
                e = launch_moments(w / 3 ? 8 : 4, 4 * (w % 3 + 1), b->max_l, b->gen, b->skew, b->d_ctxs.p, b->d_mom_items[w].p, (int)b->mom_items[w].size(),
                                   b->d_mom_tasks.p, nullptr, nullptr, b->mom_lds[w], b->cap);
            if (e == hipSuccess)
                e = launch_chunk_reduce_batch(b->d_ctxs.p, b->d_reduce_f64.p, (int)b->reduce_f64.size(), b->cap);
            if (e == hipSuccess) e = launch_moment_reduce(b->d_ctxs.p, b->d_mom_reduce.p, (int)b->mom_reduce.size(), b->cap);
            if (e == hipSuccess)
                e = launch_moment_expand(b->d_ctxs.p, b->d_mom_expand.p, (int)b->mom_expand.size(), nullptr, b->cap);
        } else {
            const int k = precision == PUFE_PREC_BF16X3 ? 0 : 1;
            if (b->lds_split[k] > kMaxDynLds) e = hipErrorInvalidValue;
            else
                e = launch_split_persistent(k + 2, b->max_l, b->gen, b->d_ctxs.p, b->d_items_split.p, (int)b->items_split.size(), b->d_counter.p,
                                            b->grid_split[k], b->lds_split[k], b->cap);
        }
        if (e == hipSuccess && precision != PUFE_PREC_FP64)
            e = launch_chunk_reduce_batch(b->d_ctxs.p, b->d_reduce.p, (int)b->reduce.size(), b->cap);
        if (e == hipSuccess)
            e = launch_gather(b->d_ctxs.p, b->d_blocks.p, b->gather, nullptr, nullptr, nullptr, kps, out_dtype,
                              false, nullptr, nullptr, 0, 0, b->cap);
        hipGraph_t g = nullptr;
        hipError_t e2 = hipStreamEndCapture(b->cap, &g);
        if (e != hipSuccess) {
            if (g) (void)hipGraphDestroy(g);
            return bfail(b, PUFE_ERR_HIP, std::string("capture: ") + hipGetErrorString(e));
        }
        CHECK_HIP_B(b, e2, "end capture");
        b->graph = g;
        CHECK_HIP_B(b, hipGraphInstantiate(&b->exec, b->graph, nullptr, nullptr, 0), "instantiate graph");
        b->key = key;
    }
    CHECK_HIP_B(b, hipGraphLaunch(b->exec, st), "graph launch");
    return PUFE_OK;
}

const char *pufe_batch_last_error_message(const pufe_batch *b) { return b ? b->err.c_str() : "no batch"; }

}  // extern "C"
