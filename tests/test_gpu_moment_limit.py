"""Problems whose moment forms do not get their device memory: assembly, element
matrices, allocation-free entry, batch and adjoint run on the direct kernels, after
pufe_setup, pufe_set_rule and pufe_tune alike, and agree with the moment forms.

Tolerance: both forms sum the same products in float64 in another order; relative
to the norm 1e-12 (matrices and dL/dV), 1e-11 (forces), as in the tests of either
form against the oracle.
"""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1611_00731_amd as P  # noqa: E402

K = (0.1, -0.2, 0.3)


def near(a, b, tol):
    return float(torch.linalg.norm(a - b)) <= tol * float(torch.linalg.norm(b))


def problem(prob, limit):
    p = P.Problem(prob)
    P.pufe_set_moment_limit(p.ctx, limit)
    p.setup()
    with pytest.raises(P.PufeError) as err:
        P.pufe_set_moment_limit(p.ctx, -1)
    assert err.value.code == -5
    return p


def check(p, q, V, G):
    """p without, q with moments."""
    assert not P.pufe_get_forms(p.ctx)[0].any() and P.pufe_get_forms(q.ctx)[0].all()
    Hp, Sp = p.assemble(V, [K])
    Hq, Sq = q.assemble(V, [K])
    assert near(Hp, Hq, 1e-12) and near(Sp, Sq, 1e-12)
    Hn, Sn = torch.full_like(Hp, float("nan")), torch.full_like(Sp, float("nan"))
    P.pufe_assemble_noalloc(p.ctx, V, [K], "fp64", "c128", Hn, Sn)
    assert torch.equal(Hn, Hp) and torch.equal(Sn, Sp)
    for a, b in zip(p.element_matrices(21, V), q.element_matrices(21, V)):
        assert near(a, b, 1e-12)
    for args in ((G, G), (G, None), (None, G)):
        dp, dq = p.backward(V, K, *args), q.backward(V, K, *args)
        assert near(dp[1], dq[1], 1e-11)
        assert near(dp[0], dq[0], 1e-12) if args[0] is not None else not bool(dp[0].any() or dq[0].any())
    assert not P.pufe_get_forms(p.ctx)[1] and P.pufe_get_forms(q.ctx)[1]


def test_direct_kernels_without_memory_for_moments(tmp_path):
    prob = W.small("lih", mesh=(6, 6, 6), fe_order=2, levels=0, n=10, a=7.0, rc=2.6, re=1.6)
    p, q = problem(prob, 1 << 20), problem(prob, -1)
    g = torch.Generator(device="cuda").manual_seed(3)
    V = torch.rand(p.sizes["n_qp"], dtype=torch.float64, device="cuda", generator=g)
    G = torch.rand((p.sizes["nnz"], 2), dtype=torch.float64, device="cuda", generator=g)
    for how in ("setup", "rule", "tuned"):
        print("[case]", how, flush=True)
        if how == "rule":
            p.set_rule(*q.leaves())
        if how == "tuned":
            P.pufe_tune(p.ctx, "fp64", tmp_path / "tune.json")
        check(p, q, V, G)
    batch = P.Batch([p, q])
    Hs, Ss = batch.alloc(1, device="cuda")
    batch.assemble([V, V], [K], Hs, Ss)
    (Hp, Sp), (Hq, Sq) = p.assemble(V, [K]), q.assemble(V, [K])
    assert near(Hs[0], Hp, 1e-12) and near(Hs[1], Hq, 1e-12) and near(Ss[0], Sp, 1e-12) and near(Ss[1], Sq, 1e-12)
    # the split-precision adjoint needs none of the moment form's buffers, before or after FP64
    r = problem(prob, 0)
    d6, f6 = r.backward(V, K, G, G, precision="bf16x6")
    assert torch.equal(d6, q.backward(V, K, G, G, precision="bf16x6")[0])
    assert near(r.backward(V, K, G, G)[0], q.backward(V, K, G, G)[0], 1e-12)
    assert torch.equal(r.backward(V, K, G, G, precision="bf16x6")[1], f6)
    for x in (p, q, r):
        x.close()
