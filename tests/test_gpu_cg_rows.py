"""The Hartree solve on either side of the size (2048 vertices) at which its
matrix rows go from four waves to one, and with rows longer than 27 blocks: the
residual of the returned solution in the oracle's stiffness matrix.

Tolerance: the solve stops at a relative residual of 1e-13; recomputed from the
solution, the residual carries the rounding of K x, 1e-16 times the condition
of the matrix (below 1e4 here).
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


@pytest.mark.parametrize("mesh,order,proj", [((16, 16, 8), 1, False), ((13, 13, 13), 1, False), ((13, 13, 13), 2, False),
                                             ((4, 4, 3), 2, True)])
def test_residual_of_the_solution(mesh, order, proj):
    prob = W.small("lih", mesh=mesh, fe_order=order, levels=0, n=3, a=7.0)
    if proj:
        prob = W.with_projectors(prob)
    print("[case]", mesh, order, proj, flush=True)
    o = oracle.Oracle(prob)
    n = np.random.default_rng(5).uniform(0.1, 1.0, o.n_qp)
    K, m, b = o.fe_stiffness(), o.fe_load(np.ones(o.n_qp)), o.fe_load(n)
    r = 4 * np.pi * (b - b.sum() / m.sum() * m)
    p = P.Problem(prob).setup()
    _, v, it, res = p.hartree(torch.from_numpy(n).cuda())
    assert it > 0 and res <= 1e-13
    assert np.linalg.norm(K @ v.cpu().numpy() - r) <= 1e-11 * np.linalg.norm(r)
    p.close()
