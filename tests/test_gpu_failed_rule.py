"""A rule that pufe_set_rule refuses after it has begun to take it in (an element of
few functions with two million leaves beside one of many: its work items' leaf lists
do not fit in LDS): the context is left without a rule, so that no launch reads
tables of two, and pufe_set_rule or pufe_setup makes it whole again.  A rule that is refused
as malformed leaves the context as it was.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1611_00731_amd as P  # noqa: E402


def uniform(level):
    """Leaves of one element, all at one level, in canonical order."""
    code = np.arange(8 ** level)
    ijk = np.zeros((len(code), 3), np.int64)
    for b in range(level):
        for d in range(3):
            ijk[:, d] |= ((code >> (3 * b + d)) & 1) << b
    return np.full(len(code), level), ijk


def test_refused_rules():
    prob = W.small("ceal", mesh=(6, 6, 6), fe_order=1, levels=0, n=1, a=6.0, rc=2.0, re=1.5)
    p = P.Problem(prob)
    P.pufe_set_moment_limit(p.ctx, 0)
    p.setup()
    lay, nfs = p.layout(), p.sizes["n_fe_slots"]
    V = torch.ones(p.sizes["n_qp"], dtype=torch.float64, device="cuda")
    want = p.assemble(V)
    lev, ijk, off = p.leaves()
    with pytest.raises(P.PufeError) as err:
        p.set_rule(lev, ijk, off[:1].tolist() + (off[1:] + 1).tolist())
    assert err.value.code == -1 and all(torch.equal(a, b) for a, b in zip(p.assemble(V), want))
    # the elements with the most and the fewest functions, by their corners' functions
    n = np.array(prob["mesh"])
    grid = np.stack(np.meshgrid(*[np.arange(k) for k in n[::-1]], indexing="ij"), -1).reshape(-1, 3)[:, ::-1]
    per = np.diff(lay["dof_offset"]) - nfs
    corner = [(grid + [(c >> d) & 1 for d in range(3)]) % n for c in range(8)]
    fun = sum(per[(c[:, 2] * n[1] + c[:, 1]) * n[0] + c[:, 0]] for c in corner)
    big, small = int(np.argmax(fun)), int(np.argmin(fun))
    print("[case] functions", fun[big], fun[small], flush=True)
    assert fun[small] == 0 and fun[big] > 150
    levels, cells, offset = [], [], [0]
    for e in range(len(fun)):
        a, b = uniform(7) if e in (big, small) else uniform(0)
        levels.append(a)
        cells.append(b)
        offset.append(offset[-1] + len(a))
    H = torch.empty((1, p.sizes["nnz"], 2), dtype=torch.float64, device="cuda")
    for again in (lambda: p.set_rule(lev, ijk, off), p.setup):
        with pytest.raises(P.PufeError) as err:
            p.set_rule(np.concatenate(levels), np.concatenate(cells), offset)
        assert err.value.code == -2
        for call in (lambda: P.pufe_assemble(p.ctx, V, [(0.0, 0.0, 0.0)], "fp64", "c128", H), lambda: p.leaves(),
                     lambda: p.backward(V, (0.0, 0.0, 0.0)), lambda: P.Batch([p]),
                     lambda: P.pufe_set_moment_limit(p.ctx, -1)):
            with pytest.raises(P.PufeError) as err:
                call()
            assert err.value.code == -5
        again()
        assert all(torch.equal(a, b) for a, b in zip(p.assemble(V), want))
    p.close()
