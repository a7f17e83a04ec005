// Assembly of the block-sparse H and S from the element matrices (gather.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.hpp"
#include "tables.hpp"

namespace pufe {

constexpr int kMaxBlockElems = 8;   // elements that hold both vertices of a block

// An assembly list: its entries, how many at its end are small (at most
// kSmallBlock entries each, and at least kManySmall of them), the largest block.
struct GatherSizes {
    int blocks = 0, small = 0, max_entries = 0;
};
constexpr int kSmallBlock = 16, kManySmall = 32768;

// H and S of the k-points kps: every stored block of the listed problems
// written once.  list: entries of block_pack with the problem added to w, blocks
// (v, w) with v <= w; contributions of contr_pack in element order.  partial, H, S: the buffers
// of a single-problem call (partial null: each problem's own, also H and S);
// bloch: the element matrices hold real and imaginary rows.  f (null: none; else
// of a single problem): the projector sums f[(k n_pfun + J) n_dof + i] with the
// strengths pfun_h, whose term H_ij += sum_J h_J f_J^i conj(f_J^j) the blocks take.
hipError_t launch_gather(const CtxDev *ctxs, const int4 *list, const GatherSizes &sz, const double *partial, void *H, void *S,
                         const KPoints &kps, int out_dtype, bool bloch, const double2 *f, const double *pfun_h, int n_pfun,
                         int64_t n_dof, hipStream_t st);

}  // namespace pufe
