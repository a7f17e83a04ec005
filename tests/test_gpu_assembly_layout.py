"""Assembly of H and S from the element matrices where its index arithmetic can
go wrong: meshes of two elements (every block meets every boundary), odd and
unequal meshes, each element order, more k-points than one launch takes, and
each output type, against the oracle's dense matrices.

Tolerance: an entry sums at most 8 element contributions of matrices that agree
with the oracle's to 1e-13; 1e-12 relative for double outputs (the bound of the
other parity tests), 2e-7 for single precision (half a unit in the last place of
float32 is 6e-8 per entry).
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


def rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("mesh,order,bloch", [((2, 2, 2), 2, False), ((3, 2, 5), 1, False), ((2, 3, 2), 3, False),
                                              ((2, 2, 3), 2, True), ((3, 3, 2), 1, True)])
def test_every_block_and_output_type(mesh, order, bloch):
    prob = W.small("lih", mesh=mesh, fe_order=order, levels=0, n=4, a=5.0)
    if bloch:
        prob = W.with_bloch_enrichment(prob)
    print("[case]", mesh, order, bloch, flush=True)
    rng = np.random.default_rng(3)
    kpts = [(0.0, 0.0, 0.0)] + [tuple(rng.uniform(-0.5, 0.5, 3)) for _ in range(17)]
    o = oracle.Oracle(prob)
    V = potential_at(torch.from_numpy(o.quadrature()[0]).cuda(), prob)
    p = P.Problem(prob).setup()
    H, S = p.assemble(V, kpts)
    Hf, Sf = p.assemble(V, kpts, out_dtype="c64")
    H1, none = p.assemble(V, kpts, with_S=False)
    Hr, Sr = p.assemble(V, kpts[:1], out_dtype="f64")
    assert none is None and torch.equal(H1, H)
    assert torch.equal(Hr[0], H[0, :, 0]) and torch.equal(Sr[0], S[0, :, 0])
    assert rel(Hf.double().cpu().numpy(), H.cpu().numpy()) < 2e-7 and rel(Sf.double().cpu().numpy(), S.cpu().numpy()) < 2e-7
    dense = o.assemble_dense_bloch if bloch else o.assemble_dense
    for k in (0, 1, 15, 16, 17):
        Ho, So = dense(V.cpu().numpy(), kpts[k])
        Hd, Sd = p.to_dense(H[k]).cpu().numpy(), p.to_dense(S[k]).cpu().numpy()
        assert rel(Hd, Ho) < 1e-12 and rel(Sd, So) < 1e-12, k
        assert np.array_equal(Hd, Hd.conj().T)
    p.close()
