"""The FP64 contraction in moment form against the oracle's element matrices, on
problems large enough that it is chosen: Gauss rules below, at and above a
multiple of four (up to three steps along x), one to eleven row tiles (work groups
of four and of eight waves, one and two stage buffers), both tensor-product
orders, a triclinic cell, tabulated radial parts.

Tolerance: sums of at most 1e6 products in float64; relative to the matrix's
norm their rounding is below 1e-13, and expanding the moments into the element's
functions adds products of at most 27 terms of like size: 1e-12.
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

CASES = {
    # cell, mesh, order, Gauss points, levels, extra, tabulated
    "two tiles, 3 points": ("lih", (8, 8, 8), 2, 3, 3, dict(a=7.0, rc=2.6, re=1.6), False),
    "one tile, 7 points": ("one", (8, 8, 8), 1, 7, 2, dict(a=6.0, rc=2.5, re=1.4), False),
    "many tiles, 5 points": ("ceal", (6, 6, 6), 2, 5, 2, dict(a=6.0, rc=3.4, re=2.2), False),
    "many tiles, 9 points": ("ceal", (5, 5, 5), 1, 9, 1, dict(a=6.0, rc=3.4, re=2.2), False),
    "triclinic, 6 points": ("triclinic", 6, 2, 6, 1, {}, False),
    "tabulated, 4 points": ("lih", (8, 8, 8), 2, 4, 3, dict(a=7.0, rc=2.6, re=1.6), True),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_moments_match_oracle(name):
    cell, mesh, order, gauss, levels, extra, tab = CASES[name]
    if cell == "triclinic":
        prob = W.ceal_triclinic(mesh=mesh, levels=levels, n=gauss, n_ref=8, tol=1e-4)
    else:
        prob = W.small(cell, mesh=mesh, fe_order=order, levels=levels, n=gauss, **extra)
    if tab:
        prob = W.with_tabulated_radials(prob)
    o = oracle.Oracle(prob)
    xyz, _, off = o.quadrature()
    V = potential_at(torch.from_numpy(xyz).cuda(), prob)
    p = P.Problem(prob).setup()
    if prob["quad"]["mode"] == "error":   # on the oracle's rule
        p.set_rule(*o.leaves())
    Vh = V.cpu().numpy()
    nloc = np.array([len(o.element_dofs(e)[0]) for e in range(p.sizes["n_elem"])])
    print("[case]", name, "points", len(Vh), "functions", nloc.min(), nloc.max(), flush=True)
    order_ = np.argsort(nloc, kind="stable")
    for e in order_[[0, len(order_) // 3, 2 * len(order_) // 3, -1]]:
        He, Se = (m.cpu().numpy() for m in p.element_matrices(int(e), V))
        Ho, So = o.element_matrices(int(e), Vh[off[e]:off[e + 1]])
        assert np.linalg.norm(He - Ho) < 1e-12 * np.linalg.norm(Ho)
        assert np.linalg.norm(Se - So) < 1e-12 * np.linalg.norm(So)
    p.close()

