"""The choice of form of the FP64 contraction: problems that run through moments, in
whole or in part, over the rules and sizes where that kernel's branches change (Gauss
rules below, at and above a multiple of four, one to eleven row tiles, both orders,
sheared cells, tabulated radial parts), and problems whose many small elements leave
the direct kernels the faster.  The matrices agree with those of the direct kernels
everywhere, and elements that the plan says work through moments (the largest among
them) with the oracle.

Tolerance: as in the other tests of either form, 1e-12 of the matrix's norm.
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

LIH = dict(a=7.0, rc=2.6, re=1.6)
CEAL = dict(a=6.0, rc=3.4, re=2.2)
SHEARED = [[7.0, 0.3, -0.2], [0.1, 6.8, 0.25], [0.2, -0.3, 7.3]]
CASES = {
    "one tile, order 2, 7 points": lambda: W.small("one", mesh=(8, 8, 8), fe_order=2, levels=2, n=7, a=6.0, rc=2.5, re=1.4),
    "one tile, order 1, 10 points": lambda: W.small("one", mesh=(8, 8, 8), fe_order=1, levels=2, n=10, a=6.0, rc=2.5, re=1.4),
    "many tiles, 3 points": lambda: W.small("ceal", mesh=(6, 6, 6), fe_order=2, levels=2, n=3, **CEAL),
    "many tiles, 5 points": lambda: W.small("ceal", mesh=(6, 6, 6), fe_order=2, levels=2, n=5, **CEAL),
    "many tiles, order 1, 9 points": lambda: W.small("ceal", mesh=(5, 5, 5), fe_order=1, levels=1, n=9, **CEAL),
    "triclinic, 8 points": lambda: W.ceal_triclinic(mesh=6, levels=1, n=8, n_ref=10, tol=1e-5),
    "sheared, 12 points": lambda: W.small("lih", mesh=(8, 8, 8), fe_order=2, levels=0, n=12, rc=2.6, re=1.6, lattice=SHEARED),
    "tabulated, 4 points": lambda: W.with_tabulated_radials(W.small("lih", mesh=(8, 8, 8), fe_order=2, levels=3, n=4, **LIH)),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_moment_form_is_taken_and_matches(name):
    prob = CASES[name]()
    o = oracle.Oracle(prob)
    p, q = P.Problem(prob).setup(), P.Problem(prob)
    P.pufe_set_moment_limit(q.ctx, 0)
    q.setup()
    if prob["quad"]["mode"] == "error":
        for x in (p, q):
            x.set_rule(*o.leaves())
    xyz, _, off = o.quadrature()
    V = potential_at(torch.from_numpy(xyz).cuda(), prob)
    nloc = np.array([len(o.element_dofs(e)[0]) for e in range(p.sizes["n_elem"])])
    moment = P.pufe_get_forms(p.ctx)[0]
    at = np.flatnonzero(moment & (nloc > (prob["fe_order"] + 1) ** 3))   # with enrichment
    at = at[np.argsort(nloc[at], kind="stable")]
    print("[case]", name, "in moment form", moment.sum(), "of", len(moment), "enriched", len(at), flush=True)
    assert len(at) >= 16 and nloc[at[-1]] == nloc.max() and not P.pufe_get_forms(q.ctx)[0].any()
    k = [(0.0, 0.0, 0.0), (0.1, -0.2, 0.3)]
    for a, b in zip(p.assemble(V, k), q.assemble(V, k)):
        assert float(torch.linalg.norm(a - b)) <= 1e-12 * float(torch.linalg.norm(b))
    Vh = V.cpu().numpy()
    for e in at[[0, len(at) // 3, 2 * len(at) // 3, -1]]:
        He, Se = (m.cpu().numpy() for m in p.element_matrices(int(e), V))
        Ho, So = o.element_matrices(int(e), Vh[off[e]:off[e + 1]])
        assert np.linalg.norm(He - Ho) < 1e-12 * np.linalg.norm(Ho)
        assert np.linalg.norm(Se - So) < 1e-12 * np.linalg.norm(So)
    for x in (p, q):
        x.close()


@pytest.mark.parametrize("mesh,order,gauss,levels", [(16, 2, 4, 0), (12, 2, 4, 1), (20, 2, 3, 1), (24, 1, 3, 1)])
def test_many_small_elements_stay_with_the_direct_kernels(mesh, order, gauss, levels):
    # the moments' stores and the expansion cost more here than the points save
    # (measured 1041 against 377 us, 474/318, 1905/868)
    print("[case]", mesh, order, gauss, levels, flush=True)
    p = P.Problem(W.small("lih", mesh=(mesh,) * 3, fe_order=order, levels=levels, n=gauss, a=7.6, rc=3.0, re=2.0)).setup()
    assert not P.pufe_get_forms(p.ctx)[0].any()
    p.close()
