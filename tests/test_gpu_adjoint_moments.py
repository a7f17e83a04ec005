"""The FP64 adjoint in moment form against the oracle's dense adjoint at the
edges of its stages and tasks: one to several row tiles (the lines of a plane
side by side in the matrix instruction for one and two), Gauss rules that are no
multiple of four, stages of several planes, one plane and part of a plane, both
tensor-product orders, tabulated radial parts, one leaf and several per element.

Tolerance: float64 sums of at most 1e5 terms of mixed sign, whose rounding stays
below 1e5 x 2^-53 = 1.1e-11 of the largest partial sums; the results are of the
order of these.
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
from test_gpu_backward import bsr_index, rel  # noqa: E402
from workloads.potential import potential_at  # noqa: E402

CASES = {
    # cell, mesh, order, Gauss points, levels, extra
    "one tile, 2 points": ("lih", (4, 4, 4), 2, 2, 0, dict(a=9.0, rc=2.0, re=1.0)),
    "one and two tiles, 5 points": ("lih", (3, 3, 4), 1, 5, 1, dict(a=7.0, rc=2.1, re=1.4)),
    "many tiles, 4 points": ("ceal", (2, 2, 2), 1, 4, 1, dict(a=4.4, rc=3.0, re=2.4)),
    "part of a plane, 9 points": ("ceal", (2, 2, 2), 2, 9, 0, dict(a=4.4, rc=3.0, re=2.4)),
    "three steps along x, 10 points": ("lih", (2, 2, 2), 2, 10, 0, dict(a=4.8, rc=2.1, re=1.7)),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_adjoint_moments_match_oracle(name):
    cell, mesh, order, gauss, levels, extra = CASES[name]
    prob = W.small(cell, mesh=mesh, fe_order=order, levels=levels, n=gauss, **extra)
    print("[case]", name, flush=True)
    o = oracle.Oracle(prob)
    xyz, _, _ = o.quadrature()
    V = potential_at(torch.from_numpy(xyz).cuda(), prob).cpu().numpy()
    Cp, Cq = W.adjoint_factor(o.n_dof, rank=4, seed=2), W.adjoint_factor(o.n_dof, rank=2, seed=3)
    Pd, Qd = Cp @ Cp.conj().T, Cq @ Cq.conj().T
    kap = (0.31, 0.05, -0.22)
    dV_o, dR_o = o.backward_dense(V, kap, Pd, Qd)
    p = P.Problem(prob).setup()
    rows, cols = bsr_index(p.layout())
    Pb, Qb = torch.from_numpy(Pd[rows, cols]).cuda(), torch.from_numpy(Qd[rows, cols]).cuda()
    dV, dR = p.backward(torch.from_numpy(V).cuda(), kap, Pb, Qb)
    assert rel(dV.cpu().numpy(), dV_o) < 1e-11
    assert np.abs(dR.cpu().numpy() - dR_o).max() < 1e-11 * np.abs(dR_o).max()
    p.close()
