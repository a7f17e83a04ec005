"""The problems of the tests of the moment form do run in it: on each, elements that
the plan says work through moments (the largest one among them) are held against the
oracle, over the range of their sizes.

Tolerance: as in those tests, 1e-12 of the matrix's norm.
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
from test_gpu_moments import CASES  # noqa: E402
from workloads.potential import potential_at  # noqa: E402


@pytest.mark.parametrize("name", sorted(CASES))
def test_elements_in_moment_form_match_oracle(name):
    cell, mesh, order, gauss, levels, extra, tab = CASES[name]
    if cell == "triclinic":
        prob = W.ceal_triclinic(mesh=mesh, levels=levels, n=gauss, n_ref=8, tol=1e-4)
    else:
        prob = W.small(cell, mesh=mesh, fe_order=order, levels=levels, n=gauss, **extra)
    if tab:
        prob = W.with_tabulated_radials(prob)
    o = oracle.Oracle(prob)
    p = P.Problem(prob).setup()
    if prob["quad"]["mode"] == "error":
        p.set_rule(*o.leaves())
    xyz, _, off = o.quadrature()
    V = potential_at(torch.from_numpy(xyz).cuda(), prob)
    nloc = np.array([len(o.element_dofs(e)[0]) for e in range(p.sizes["n_elem"])])
    moment = P.pufe_get_forms(p.ctx)[0]
    at = np.flatnonzero(moment & (nloc > (order + 1) ** 3))   # with enrichment
    at = at[np.argsort(nloc[at], kind="stable")]
    print("[case]", name, "in moment form", moment.sum(), "of", len(moment), "enriched", len(at), flush=True)
    assert len(at) >= 16 and nloc[at[-1]] == nloc.max()
    Vh = V.cpu().numpy()
    for e in at[[0, len(at) // 3, 2 * len(at) // 3, -1]]:
        He, Se = (m.cpu().numpy() for m in p.element_matrices(int(e), V))
        Ho, So = o.element_matrices(int(e), Vh[off[e]:off[e + 1]])
        assert np.linalg.norm(He - Ho) < 1e-12 * np.linalg.norm(Ho)
        assert np.linalg.norm(Se - So) < 1e-12 * np.linalg.norm(So)
    p.close()
