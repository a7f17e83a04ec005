"""The projectors' coefficients in moment form and their term added by the
assembly, at the edges of both: Gauss rules below, at and above a multiple of
four (stages of all planes down to one), elements of few tasks and of several
items of them, both tensor-product orders, blocks whose projector sums fit a
wave's stage and blocks whose do not, several k-points in one launch.

Tolerance: H to 1e-12 as every FP64 assembly; the term alone to 1e-9, the local
part's rounding (1e-15 of a norm up to 1e4 times the term's) with a margin.
"""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1611_00731_amd as P  # noqa: E402
from workloads.potential import potential_at  # noqa: E402

KPTS = [(0.0, 0.0, 0.0), (0.12, -0.24, 0.37), (0.5, 0.0, -0.25)]
CASES = {
    "one, 2 points": ("one", (3, 3, 2), 1, 2, 1, dict(a=4.6)),
    "lih, 5 points": ("lih", (3, 2, 2), 2, 5, 1, dict(a=5.0)),
    "ceal, 4 points, many tasks": ("ceal", (2, 2, 2), 1, 4, 1, dict(a=4.4, rc=3.0, re=2.4)),
    "lih, 9 points": ("lih", (2, 2, 2), 2, 9, 0, dict(a=5.0)),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_projector_moments_match_oracle(name):
    cell, mesh, order, gauss, levels, extra = CASES[name]
    prob = W.with_projectors(W.small(cell, mesh=mesh, fe_order=order, levels=levels, n=gauss, **extra))
    print("[case]", name, flush=True)
    o = oracle.Oracle(prob)
    xyz, _, _ = o.quadrature()
    V = potential_at(torch.from_numpy(xyz).cuda(), prob)
    p = P.Problem(prob).setup()
    H, _ = p.assemble(V, KPTS)
    for k, kap in enumerate(KPTS):
        Ho, _ = o.assemble_dense(V.cpu().numpy(), kap)
        Vn = o.nonlocal_dense(kap)
        Hg = p.to_dense(H[k]).cpu().numpy()
        assert np.linalg.norm(Hg - Ho - Vn) < 1e-12 * np.linalg.norm(Ho + Vn)
        assert np.linalg.norm(Hg - Ho - Vn) < 1e-9 * np.linalg.norm(Vn)
    p.close()
