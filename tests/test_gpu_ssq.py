"""Singular pairs (ssq.hip) at every order of the rule against the oracle's
blocks: groups that do not divide a batch of 128 points (orders 3, 5, 6, 7),
one point per group (order 1), both tangential bases and both schemes."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from oracle import core, galerkin  # noqa: E402
from paper_2604_21181_amd import mbem  # noqa: E402
from workloads.meshes import icosphere_p2  # noqa: E402


@pytest.mark.parametrize("frame", [0, 1])
@pytest.mark.parametrize("paper", [0, 1])
@pytest.mark.parametrize("order", [1, 2, 3, 4, 5, 6, 7, 8])
def test_orders_against_oracle(order, paper, frame):
    # every pair of the 20-triangle sphere but the opposite ones is singular
    xyz, tri = icosphere_p2(20, (1.0, 0.9, 1.2))
    k0, eps = 1.3, 2.2 + 0.1j
    P = galerkin.Problem(xyz, tri, k0, eps, nss=order, variant=paper, frame=frame)
    Ko = core.fill(P.xyz, P.tri6, P.phys, nss=order)
    for prec, tol in ((mbem.MBEM_FP64, 1e-11), (mbem.MBEM_MIXED, 1e-5)):
        # FP64: sums of up to 4 x 10^4 points, rounding 1.1e-16 each; complex64
        # blocks: a few dozen roundings of 6e-8 per entry
        S = mbem.Solver(xyz, tri, k0, eps, precision=prec, ssq_order=order, quadrature=paper, frame=frame)
        try:
            S.fill()
            one = S.perm[:2 * S.nn]
            for K, ref in zip(S.export_blocks(), Ko):
                R = np.asarray(ref)[np.ix_(one, one)]
                assert np.linalg.norm(K.cpu().numpy() - R) <= tol * np.linalg.norm(R)
        finally:
            S.close()
