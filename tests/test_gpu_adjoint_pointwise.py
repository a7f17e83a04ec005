"""dL/dV of the FP64 adjoint point by point, where it is a sum of squares: P is one
on the enriched functions of one vertex, so dL/dV = w M^2 sum_f Psi_f^2 with the
hat M of that vertex, which falls to zero on the far faces of its elements.  Each
factor is a product, so the error of a point is held relative to its own value.

Tolerance, points above 1e-8 of the largest value: the hats carry the rounding of
the element coordinate, 2^-53 over the distance to the face (0.025 in reference
coordinates here), the radial part six times that of 1 - (r/rc)^2 (above 0.04
there); squared, and once each for the library and the oracle, 2e-13 in all.
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


@pytest.mark.parametrize("order", [1, 2])
def test_density_of_one_vertex(order):
    prob = W.small("one", mesh=(4, 4, 4), fe_order=order, levels=1, n=7, a=4.0, rc=2.4, re=1.4)
    print("[case] order", order, flush=True)
    o = oracle.Oracle(prob)
    p = P.Problem(prob).setup()
    p.set_rule(*o.leaves())   # leaves that touch the refinement distance may go either way
    lay, nfs = p.layout(), p.sizes["n_fe_slots"]
    dof, n = lay["dof_offset"], o.n_dof
    v = int(np.argmax(np.diff(dof)))
    Pd = np.zeros((n, n), complex)
    Pd[range(dof[v] + nfs, dof[v + 1]), range(dof[v] + nfs, dof[v + 1])] = 1.0
    V = np.zeros(o.n_qp)
    want, _ = o.backward_dense(V, (0.0, 0.0, 0.0), Pd, np.zeros_like(Pd))
    Pb = np.zeros((p.sizes["nnz"], 2))
    k = lay["brow_ptr"][v] + list(lay["bcol"][lay["brow_ptr"][v]:lay["brow_ptr"][v + 1]]).index(v)
    w = dof[v + 1] - dof[v]
    for s in range(nfs, w):
        Pb[lay["bval_offset"][k] + s * w + s, 0] = 1.0
    dV, _ = p.backward(torch.from_numpy(V).cuda(), (0.0, 0.0, 0.0), torch.from_numpy(Pb).cuda())
    got, at = dV.cpu().numpy(), want > 1e-8 * want.max()
    err = np.abs(got - want)[at] / want[at]
    print("[case] points", at.sum(), "largest error of a point", err.max(), flush=True)
    assert at.sum() > 1000 and err.max() <= 2e-13
    p.close()
