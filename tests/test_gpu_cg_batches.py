"""The Hartree solve's conjugate gradients around the ends of its batches of
iterations (17 launches between two looks of the host at the outcome): an
iteration limit of k is met exactly, the iterates are those of the textbook
recurrence on the same operator, and the full solve meets the oracle.

Tolerances: after at most 18 iterations the recurrence has amplified rounding
(1e-16) by less than 1e6; the solution is held to 1e-10 as in the other tests
of the solve.
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


@pytest.mark.parametrize("order", [1, 2, 3])
def test_iteration_limits(order):
    prob = W.small("lih", mesh=(4, 3, 3), fe_order=order, levels=0, n=4, a=5.0)
    print("[case] order", order, flush=True)
    o = oracle.Oracle(prob)
    n = np.random.default_rng(2).uniform(0.1, 1.0, o.n_qp)
    nd = torch.from_numpy(n).cuda()
    p = P.Problem(prob).setup()
    K, m, b = o.fe_stiffness(), o.fe_load(np.ones(o.n_qp)), o.fe_load(n)
    r = 4 * np.pi * (b - b.sum() / m.sum() * m)
    x, d, rr, r0, k = np.zeros_like(r), r.copy(), r @ r, np.linalg.norm(r), 0
    for limit in (1, 2, 15, 16, 17, 18):
        while k < limit:
            q = K @ d
            a = rr / (d @ q)
            x, r = x + a * d, r - a * q
            d, rr, k = r + (r @ r) / rr * d, r @ r, k + 1
        if np.sqrt(rr) / r0 < 1e-9:
            break
        _, v, it, res = p.hartree(nd, tol=1e-13, max_iter=limit)
        want = x - (m @ x) / m.sum()
        assert it == limit
        assert abs(res - np.sqrt(rr) / r0) <= 1e-6 * res + 1e-12
        assert np.linalg.norm(v.cpu().numpy() - want) <= 1e-9 * np.linalg.norm(want)
    vh, _, it, res = p.hartree(nd)
    ref = o.hartree(n)[0]
    assert res <= 1e-13 and it > 0
    assert np.linalg.norm(vh.cpu().numpy() - ref) <= 1e-10 * np.linalg.norm(ref)
    p.close()
