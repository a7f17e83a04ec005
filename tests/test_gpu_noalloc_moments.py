"""The allocation-free entry on problems in moment form (in part): its sums lie behind the
partial tiles in the fixed workspace, or in a buffer of their own where they do not
fit there.  Either way it gives what pufe_assemble gives, bit for bit, after
pufe_setup, pufe_set_rule and pufe_tune, and while pufe_assemble works on another
potential on another stream.
"""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1611_00731_amd as P  # noqa: E402

MIB = 1 << 20
WORKSPACE = 64 * MIB
CASES = {
    # mesh, order, Gauss points, re; a bound of the sums' bytes from above or below
    "workspace": ((6, 6, 6), 2, 10, 1.6, 32 * MIB, True),
    "own buffer": ((10, 10, 10), 2, 10, 2.4, WORKSPACE, False),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_noalloc_in_moment_form(name, tmp_path):
    mesh, order, gauss, re, limit, fits = CASES[name]
    prob = W.small("lih", mesh=mesh, fe_order=order, levels=0, n=gauss, a=7.0, rc=2.6, re=re)
    q = P.Problem(prob)
    P.pufe_set_moment_limit(q.ctx, limit)
    assert bool(P.pufe_get_forms(q.setup().ctx)[0].any()) == fits   # which place they take
    q.close()
    p = P.Problem(prob).setup()
    T = (p.sizes["max_nloc"] + 15) // 16
    if fits:
        assert p.sizes["n_elem"] * T * (T + 1) // 2 * 4096 < WORKSPACE - limit - MIB
    g = torch.Generator(device="cuda").manual_seed(3)
    k = [(0.1, -0.2, 0.3), (0.25, 0.25, -0.25)]
    V, V2 = (torch.rand(p.sizes["n_qp"], dtype=torch.float64, device="cuda", generator=g) for _ in range(2))
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    for how in ("setup", "rule", "tuned"):
        print("[case]", name, how, flush=True)
        if how == "rule":
            p.set_rule(*p.leaves())
        if how == "tuned":
            P.pufe_tune(p.ctx, "fp64", tmp_path / "tune.json")
        assert P.pufe_get_forms(p.ctx)[0].any()
        H, S = p.assemble(V, k)
        H2, S2 = p.assemble(V2, k)
        out = [torch.full_like(H, float("nan")) for _ in range(4)]
        for _ in range(3):
            torch.cuda.synchronize()
            P.pufe_assemble_noalloc(p.ctx, V, k, "fp64", "c128", out[0], out[1], stream=s1)
            P.pufe_assemble(p.ctx, V2, k, "fp64", "c128", out[2], out[3], stream=s2)
            torch.cuda.synchronize()
            assert all(torch.equal(a, b) for a, b in zip(out, (H, S, H2, S2)))
    p.close()
