"""The far field as a product of phases and currents (post.hip, k_farfield)
against the sum over quadrature points evaluated here: direction counts around
its tiles of 16, one to nine solutions (groups of four), meshes whose 7 nt
points leave 2 over the fours and whose runs are short and long, both
tangential bases, and phases beyond the short range reduction."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from oracle import galerkin  # noqa: E402
from paper_2604_21181_amd import mbem  # noqa: E402
from workloads.meshes import icosphere_p2, uv_sphere_p2  # noqa: E402

MESHES = {"ico20": lambda: icosphere_p2(20, (1.0, 0.9, 1.2)), "uv70": lambda: uv_sphere_p2(7, 6, (1.0, 0.8, 0.7)),
          "ico320": lambda: icosphere_p2(320)}


def _directions(n):
    r = np.random.default_rng(n).normal(size=(n, 3))
    return r / np.linalg.norm(r, axis=1)[:, None]


def _check(mesh, k0, frame, nv, nd, tol):
    xyz, tri = MESHES[mesh]()
    P = galerkin.Problem(xyz, tri, k0, 3.0, frame=frame)
    S = mbem.Solver(xyz, tri, k0, 3.0, frame=frame)
    try:
        rng = np.random.default_rng(nv + nd)
        x = rng.normal(size=(nv, S.N)) + 1j * rng.normal(size=(nv, S.N))
        r = _directions(nd)
        dev = torch.as_tensor(x[:, S.perm].copy(), device=S.device)
        F = S.farfield(dev, r).cpu().numpy()
        for v in range(nv):
            ref = galerkin.far_field(P, x[v], r)
            assert np.abs(F[v] - ref).max() <= tol * np.abs(ref).max(), (v, nv, nd)
    finally:
        S.close()


# sums of at most 2240 terms of size max|current|, far above sqrt(2240) eps of
# the result's scale: 1e-12 leaves a factor of a hundred
@pytest.mark.parametrize("frame", [0, 1])
@pytest.mark.parametrize("nv,nd", [(1, 1), (1, 17), (2, 15), (3, 16), (4, 33), (5, 2), (9, 100)])
@pytest.mark.parametrize("mesh", sorted(MESHES))
def test_against_oracle(mesh, nv, nd, frame):
    _check(mesh, 1.4, frame, nv, nd, 1e-12)


def test_more_directions_than_a_launch():
    _check("ico20", 1.4, 0, 1, 32768 + 17, 1e-12)


def test_phases_beyond_the_short_reduction():
    # phases up to 4e6 carry a rounding of 4 x 4e6 eps each
    _check("uv70", 4.0e6, 0, 2, 21, 1e-8)


def test_not_a_number_stays_in_its_solution_and_direction():
    xyz, tri = MESHES["uv70"]()
    S = mbem.Solver(xyz, tri, 1.4, 3.0)
    try:
        x = torch.ones((3, S.N), dtype=torch.complex128, device=S.device)
        r = _directions(20)
        want = S.farfield(x, r)
        x[1, 0] = complex(float("nan"), 0.0)
        r[7] = np.inf
        F = torch.view_as_real(S.farfield(x, r)).cpu().numpy()
        bad = ~np.isfinite(F).all(axis=(2, 3))
        assert bad[1].any() and bad[0, 7] and bad[2, 7]
        want = torch.view_as_real(want).cpu().numpy()
        keep = np.arange(20) != 7
        for v in (0, 2):
            assert np.abs(F[v, keep] - want[v, keep]).max() <= 1e-12 * np.abs(want[v]).max()
    finally:
        S.close()
