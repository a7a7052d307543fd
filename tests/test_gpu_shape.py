"""The shape gradient's pairs (shape.hip) against differences of sigma_ext along
a direction of all node coordinates.  k_shape_regular (tiles of 64 x 64 points,
each pair once for both sides): meshes that leave the last tile short, with the
tile's steps divided over four, two and one wavefronts.  k_shape_ssq (batches of
64 points of two regions): Sauter-Schwab orders that leave the last batch short
or the only one nearly empty."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2604_21181_amd import mbem  # noqa: E402
from workloads.meshes import cubesphere_p2, uv_sphere_p2  # noqa: E402

MESHES = {"uv70": lambda: uv_sphere_p2(7, 6, (1.0, 0.8, 0.9)),        # 8 tiles, 42 points in the last
          "cube300": lambda: cubesphere_p2(5, (1.0, 1.0, 1.2)),       # 33 tiles, 52
          "cube432": lambda: cubesphere_p2(6, (1.0, 0.9, 1.1))}       # 48 tiles, 16
KH, POL = [0.0, 0.0, 1.0], [1.0, 0.0, 0.0]


def _sigma(xyz, tri, eps, frame, grad, order=0):
    S = mbem.Solver(xyz, tri, 1.8, eps, frame=frame, ssq_order=order)
    try:
        S.fill()
        S.precond_setup(100)
        x, _, code = S.solve(S.rhs([KH], [POL]), tol=1e-13, maxit=400)
        assert code == 0
        out = S.grad_sigma_ext(x[0], KH, POL, tol=1e-13, shape=grad)
        return out[0][0], out[4].cpu().numpy() if grad else None
    finally:
        S.close()


def _compare(xyz, tri, eps, frame, order=0):
    _, dx = _sigma(xyz, tri, eps, frame, True, order)
    # a smooth displacement of every node, of the size of the body
    rng = np.random.default_rng(5)
    D = np.sin(xyz @ rng.normal(size=(3, 3)) + rng.normal(size=3))
    h = 1e-3
    f = {k: _sigma(xyz + k * h * D, tri, eps, frame, False, order)[0] for k in (-2, -1, 1, 2)}
    ref = (8.0 * (f[1] - f[-1]) - (f[2] - f[-2])) / (12.0 * h)
    # h^4 = 1e-12 of the fifth derivative, and 1e-12 sigma / h from rounding and
    # the solves; a wrong tile changes the sum by a part in a thousand
    scale = (np.abs(dx) * np.abs(D)).sum()
    assert abs(float((dx * D).sum()) - ref) <= 1e-7 * scale


@pytest.mark.parametrize("frame", [0, 1])
@pytest.mark.parametrize("eps", [3.0, -2.0 + 0.5j])
@pytest.mark.parametrize("mesh", sorted(MESHES))
def test_against_differences(mesh, eps, frame):
    _compare(*MESHES[mesh](), eps, frame)


@pytest.mark.parametrize("frame", [0, 1])
@pytest.mark.parametrize("order", [2, 3, 5])
def test_sauter_schwab_orders(order, frame):
    _compare(*MESHES["uv70"](), 3.0, frame, order)
