"""d sigma_ext / d eps_r without the derivative operator (shape.hip,
k_deps_regular and k_deps_ssq) against lambda^T (dZ/deps) x with the filled
operator of mbem_fill_deps: last tiles of 42, 48 and 52 points, both tangential
bases, lossy and lossless, Sauter-Schwab orders that leave batches short."""
import math

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2604_21181_amd import mbem  # noqa: E402
from workloads.meshes import cubesphere_p2, icosphere_p2, uv_sphere_p2  # noqa: E402

MESHES = {"uv70": lambda: uv_sphere_p2(7, 6, (1.0, 0.8, 0.9)), "ico80": lambda: icosphere_p2(80),
          "cube300": lambda: cubesphere_p2(5, (1.0, 1.0, 1.2))}
KH, POL = [0.0, 0.0, 1.0], [1.0, 0.0, 0.0]


@pytest.mark.parametrize("precision,frame,order", [(0, 0, 4), (0, 1, 4), (1, 0, 4), (0, 0, 3), (0, 1, 2)])
@pytest.mark.parametrize("eps", [3.0, -2.0 + 0.5j])
@pytest.mark.parametrize("mesh", sorted(MESHES))
def test_against_the_derivative_operator(mesh, eps, precision, frame, order):
    xyz, tri = MESHES[mesh]()
    k0 = 1.8
    S = mbem.Solver(xyz, tri, k0, eps, precision=precision, frame=frame, ssq_order=order)
    try:
        S.fill()
        S.precond_setup(60)
        x, _, code = S.solve(S.rhs([KH], [POL]), tol=1e-10, maxit=400)
        assert code == 0
        out, _, lam = S.grad_sigma_ext(x[0], KH, POL, tol=1e-10)
        dop, _ = mbem.mbem_fill_deps(S.ctx, S.mesh, S.params)
        try:
            y = torch.empty_like(x[0])
            mbem.mbem_matvec(S.ctx, dop, x[0].contiguous(), y, 1)
        finally:
            mbem.mbem_op_destroy(dop)
        v = complex((lam * y).sum())
        # sums of about N terms of size |lam| |y| / N, each from 150 points
        scale = float(lam.norm() * y.norm()) * 4.0 * math.pi / k0
        assert abs(out[1] + v.imag * 4.0 * math.pi / k0) <= 1e-12 * scale
        assert abs(out[2] + v.real * 4.0 * math.pi / k0) <= 1e-12 * scale
    finally:
        S.close()
