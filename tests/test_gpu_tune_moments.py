"""FP64 tuning of a problem whose elements all work through moments: no candidate
changes its launches, so the choice, and with it the plan, stays what it was; a
problem with elements on the direct kernels is tuned as before.
"""
import json

import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1611_00731_amd as P  # noqa: E402


def tuned(limit, cache, precision="fp64"):
    prob = W.small("one", mesh=(8, 8, 8), fe_order=2, levels=2, n=7, a=6.0, rc=2.5, re=1.4)
    p = P.Problem(prob)
    P.pufe_set_moment_limit(p.ctx, limit)
    p.setup()
    all_moment = bool(P.pufe_get_forms(p.ctx)[0].all())
    V = torch.ones(p.sizes["n_qp"], dtype=torch.float64, device="cuda")
    before = p.assemble(V)
    P.pufe_tune(p.ctx, precision, cache)
    after = p.assemble(V)
    p.close()
    return all_moment, before, after, list(json.loads(cache.read_text()).values())[-1]


def test_all_elements_in_moment_form(tmp_path):
    print("[case] all elements in moment form", flush=True)
    every, before, after, choice = tuned(-1, tmp_path / "a.json")
    assert every
    assert (choice["items"], choice["block"], choice["q"], choice["wide"]) == (4096, 4, 24, 6) and choice["ms"] > 0
    assert all(torch.equal(a, b) for a, b in zip(before, after))


@pytest.mark.parametrize("limit,precision", [(0, "fp64"), (-1, "bf16x6")])
def test_other_plans_are_tuned(limit, precision, tmp_path):
    print("[case]", limit, precision, flush=True)
    _, before, after, choice = tuned(limit, tmp_path / "a.json", precision)
    assert choice["items"] in (1024, 2048, 4096, 8192, 16384) and 0 < choice["ms"] < 1e3
    for a, b in zip(before, after):
        assert float(torch.linalg.norm(a - b)) <= 1e-12 * float(torch.linalg.norm(b))
