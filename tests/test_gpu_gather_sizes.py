"""Assembly at the ends of its block sizes: very many blocks of a few entries, eight of
which share a wave (alone and beside the larger blocks of enriched vertices, with
projectors, with the Bloch-periodic enrichment, in a batch with a problem that has
none), and a few blocks of hundreds of entries, which several waves share, against the
oracle's dense matrices.

Tolerance: as in the other tests of the assembly, 1e-12 relative for double outputs
(nonlocal term included), 2e-7 for single precision.
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

K = [(0.0, 0.0, 0.0), (0.31, -0.12, 0.2), (-0.25, 0.25, 0.4), (0.1, 0.2, 0.3), (0.5, 0.0, -0.5)]


def rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("kind,mesh,form", [("one", (15, 14, 13), ""), ("one", (15, 14, 13), "projectors"),
                                            ("one", (15, 14, 13), "bloch"), ("ceal", (2, 3, 2), ""),
                                            ("ceal", (3, 2, 2), "projectors")])
def test_small_and_large_blocks(kind, mesh, form):
    prob = W.small(kind, mesh=mesh, fe_order=1, levels=0, n=3, a=6.0, rc=2.0, re=1.0 if kind == "one" else 2.4)
    if form == "projectors":
        prob = W.with_projectors(prob)
    if form == "bloch":
        prob = W.with_bloch_enrichment(prob)
    o = oracle.Oracle(prob)
    p = P.Problem(prob).setup()
    b = p.layout()["bval_offset"]
    print("[case]", kind, mesh, form, "blocks", len(b) - 1, "entries", np.diff(b).min(), np.diff(b).max(), flush=True)
    assert kind == "ceal" or np.count_nonzero(np.diff(b) <= 16) > 2 * 32768
    xyz, _, _ = o.quadrature()
    V = potential_at(torch.from_numpy(xyz).cuda(), prob)
    Vh = V.cpu().numpy()
    H, S = p.assemble(V, K)
    Hf, Sf = p.assemble(V, K, out_dtype="c64")
    assert rel(Hf.double().cpu().numpy(), H.cpu().numpy()) < 2e-7 and rel(Sf.double().cpu().numpy(), S.cpu().numpy()) < 2e-7
    Hr, Sr = p.assemble(V, K[:1], out_dtype="f64")
    assert torch.equal(Hr[0], H[0, :, 0]) and torch.equal(Sr[0], S[0, :, 0])
    for k in (1, 4):
        Ho, So = o.assemble_dense_bloch(Vh, K[k]) if form == "bloch" else o.assemble_dense(Vh, K[k])
        if form == "projectors":
            Ho = Ho + o.nonlocal_dense(K[k])
        Hd, Sd = p.to_dense(H[k]).cpu().numpy(), p.to_dense(S[k]).cpu().numpy()
        assert rel(Hd, Ho) < 1e-12 and rel(Sd, So) < 1e-12, k
        if form != "projectors":   # whose complex products carry their own rounding in each triangle of a diagonal block
            assert np.array_equal(Hd, Hd.conj().T)
    if form == "":
        q = P.Problem(W.small("lih", mesh=(3, 2, 2), fe_order=2, levels=0, n=3, a=5.0)).setup()
        Vq = torch.linspace(-1.0, 0.5, q.sizes["n_qp"], dtype=torch.float64, device="cuda")
        Hq, Sq = q.assemble(Vq, K)
        for order in ((p, q), (q, p)):
            batch = P.Batch(order)
            Hs, Ss = batch.alloc(len(K), device="cuda")
            batch.assemble([V if x is p else Vq for x in order], K, Hs, Ss)
            for x, h, s in zip(order, Hs, Ss):
                want = (H, S) if x is p else (Hq, Sq)
                assert rel(h.cpu().numpy(), want[0].cpu().numpy()) < 1e-13 and rel(s.cpu().numpy(), want[1].cpu().numpy()) < 1e-13
        q.close()
    p.close()
