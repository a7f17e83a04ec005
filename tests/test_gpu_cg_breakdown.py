"""The Hartree solve's end with a tolerance below rounding, which runs into
p . K p <= 0 (K is singular: once the residual is rounding, the directions drift
into its kernel) or, on the larger mesh, on until the residual underflows, and on
a zero right-hand side: the solve ends before its iteration limit, the same way
each time, and returns a solution that has the residual it reports.

Tolerance: recurrence and solution are updated with the same steps, so the
reported residual and that of the solution in the oracle's K differ by rounding:
a few hundred iterations times 1e-16 times the condition of K (below 1e3), 1e-10.
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


@pytest.mark.parametrize("mesh,order", [((4, 3, 3), 1), ((4, 3, 3), 2), ((9, 8, 8), 1)])
def test_solve_ends_without_the_tolerance(mesh, order):
    prob = W.small("lih", mesh=mesh, fe_order=order, levels=0, n=4, a=5.0)
    print("[case]", mesh, order, flush=True)
    o = oracle.Oracle(prob)
    n = np.random.default_rng(2).uniform(0.1, 1.0, o.n_qp)
    K, m, b = o.fe_stiffness(), o.fe_load(np.ones(o.n_qp)), o.fe_load(n)
    rhs = 4 * np.pi * (b - b.sum() / m.sum() * m)
    p = P.Problem(prob).setup()
    nd = torch.from_numpy(n).cuda()
    _, first, it, res = p.hartree(nd, tol=1e-300, max_iter=20000)
    assert 0 < it < 20000
    assert abs(np.linalg.norm(K @ first.cpu().numpy() - rhs) / np.linalg.norm(rhs) - res) <= 1e-10
    for _ in range(4):
        _, v, it2, res2 = p.hartree(nd, tol=1e-300, max_iter=20000)
        assert (it2, res2) == (it, res) and torch.equal(v, first)
    _, v, it, res = p.hartree(torch.zeros_like(nd))
    assert it == 0 and res == 0.0 and not bool(v.any())
    p.close()
