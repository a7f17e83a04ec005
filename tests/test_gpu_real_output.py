"""Real output at k-points equivalent to Gamma: any integers, however large, give the
matrices of Gamma itself, bit for bit (the periodic form's boundary phase is one).
"""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1611_00731_amd as P  # noqa: E402


@pytest.mark.parametrize("precision", ["fp64", "bf16x6"])
def test_integer_k_points_are_gamma(precision):
    prob = W.small("lih", mesh=(3, 2, 2), fe_order=2, levels=1, n=3, a=5.0)
    p = P.Problem(prob).setup()
    V = torch.linspace(-1.0, 0.5, p.sizes["n_qp"], dtype=torch.float64, device="cuda")
    kpts = [(0.0, 0.0, 0.0), (1.0, -2.0, 3.0), (1e9, 0.0, 7.0), (3e14, 1e15, -2.0**52), (0.0, 2.0**60, 1e300)]
    H, S = p.assemble(V, kpts, precision=precision, out_dtype="f64")
    for k in range(1, len(kpts)):
        print("[case]", precision, kpts[k], flush=True)
        assert torch.equal(H[k], H[0]) and torch.equal(S[k], S[0])
    batch = P.Batch([p])
    Hs, Ss = batch.alloc(len(kpts), "f64", device="cuda")
    batch.assemble([V], kpts, Hs, Ss, precision=precision, out_dtype="f64")
    for k in range(len(kpts)):
        assert torch.equal(Hs[0][k], H[0]) and torch.equal(Ss[0][k], S[0])
    p.close()
