"""A batch whose problem's tables were replaced in part by a call that failed does not
replay the graph it captured over the former ones: it is refused, as after a call
that succeeded, and a batch made anew gives the former values.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1611_00731_amd as P  # noqa: E402


def test_batch_after_a_refused_rule():
    # all elements in direct form; with two million leaves each on the element of the
    # most functions and on one without enrichment, the latter gets few items, whose
    # leaf lists do not fit in LDS
    prob = W.small("ceal", mesh=(6, 6, 6), fe_order=1, levels=0, n=1, a=6.0, rc=2.0, re=1.5)
    p = P.Problem(prob)
    P.pufe_set_moment_limit(p.ctx, 0)
    p.setup()
    V = torch.ones(p.sizes["n_qp"], dtype=torch.float64, device="cuda")
    kpts = [(0.0, 0.0, 0.0)]
    batch = P.Batch([p])
    Hs, Ss = batch.alloc(1, device="cuda")

    def run(b):
        b.assemble([V], kpts, Hs, Ss)
        torch.cuda.synchronize()
        return Hs[0].clone(), Ss[0].clone()

    want = run(batch)
    lev, ijk, off = p.leaves()
    lay, n, nfs = p.layout(), np.array(prob["mesh"]), p.sizes["n_fe_slots"]
    grid = np.stack(np.meshgrid(*[np.arange(k) for k in n[::-1]], indexing="ij"), -1).reshape(-1, 3)[:, ::-1]
    per = np.diff(lay["dof_offset"]) - nfs
    corner = [(grid + [(c >> d) & 1 for d in range(3)]) % n for c in range(8)]
    fun = sum(per[(c[:, 2] * n[1] + c[:, 1]) * n[0] + c[:, 0]] for c in corner)
    code = np.arange(8 ** 7)
    fine = np.zeros((len(code), 3), np.int64)
    for b in range(7):
        for d in range(3):
            fine[:, d] |= ((code >> (3 * b + d)) & 1) << b
    deep = (int(np.argmax(fun)), int(np.argmin(fun)))
    count = [len(code) if e in deep else 1 for e in range(len(fun))]
    levels = np.repeat([7 if e in deep else 0 for e in range(len(fun))], count)
    cells = np.concatenate([fine if e in deep else np.zeros((1, 3), np.int64) for e in range(len(fun))])
    with pytest.raises(P.PufeError) as err:
        p.set_rule(levels, cells, np.concatenate([[0], np.cumsum(count)]))
    assert err.value.code == -2
    for again in (lambda: None, lambda: p.set_rule(lev, ijk, off)):
        again()
        with pytest.raises(P.PufeError) as err:
            run(batch)
        assert err.value.code == -5
    new = P.Batch([p])
    assert all(torch.equal(a, b) for a, b in zip(run(new), want))
    batch.close()
    new.close()
    p.close()
