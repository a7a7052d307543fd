"""The FP64 regular-pair fill by batches and bands (pairs.hip) against the
oracle's blocks: one band and several, triangle counts that leave a last batch
or band short, both rules and both tangential bases, and a node in more
batches than the gather takes at a time (against the complex64 fill)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from oracle import core, galerkin  # noqa: E402
from paper_2604_21181_amd import mbem  # noqa: E402
from workloads.meshes import cubesphere_p2, icosphere_p2, uv_sphere_p2  # noqa: E402

MESHES = {
    "ico20": lambda: icosphere_p2(20, (1.0, 0.9, 1.2)),          # four batches at most
    "uv70": lambda: uv_sphere_p2(7, 6, (1.0, 0.8, 0.7)),         # 70 triangles, one band
    "cube192": lambda: cubesphere_p2(4, (1.0, 1.0, 1.3)),        # around the first band limit
    "uv410": lambda: uv_sphere_p2(41, 6, (1.0, 0.9, 0.8)),       # several bands, poles of valence 41
}


@pytest.mark.parametrize("frame", [0, 1])
@pytest.mark.parametrize("paper", [0, 1])
@pytest.mark.parametrize("mesh", sorted(MESHES))
def test_blocks_against_oracle(mesh, paper, frame):
    xyz, tri = MESHES[mesh]()
    k0, eps = 1.7, 2.6 + 0.2j
    P = galerkin.Problem(xyz, tri, k0, eps, variant=paper, frame=frame)
    Ko = core.fill(P.xyz, P.tri6, P.phys, nss=P.nss)
    S = mbem.Solver(xyz, tri, k0, eps, quadrature=paper, frame=frame)
    try:
        one = S.perm[:2 * S.nn]
        for rep in range(2):                 # the second fill reuses every buffer
            S.fill()
            for K, ref in zip(S.export_blocks(), Ko):
                R = np.asarray(ref)[np.ix_(one, one)]
                # sums of at most ~ 40 contributions of ~ 150 points, each a few
                # dozen roundings of 1.1e-16: far below 1e-11 of the block
                assert np.linalg.norm(K.cpu().numpy() - R) <= 1e-11 * np.linalg.norm(R)
                assert np.abs(K.cpu().numpy() - R).max() <= 1e-10 * np.abs(R).max()
    finally:
        S.close()


def test_eps_derivative_several_bands():
    """dZ/deps_r by central differences of the FP64 fill: the truncation error
    is h^2 / 6 of the third derivative, about 1e-7 at h = 1e-3."""
    xyz, tri = MESHES["uv410"]()
    h, k0, eps = 1e-3, 1.7, 2.6 + 0.2j
    blocks = []
    for e in (eps + h, eps - h):
        S = mbem.Solver(xyz, tri, k0, e)
        S.fill()
        blocks.append([K.cpu() for K in S.export_blocks()])
        S.close()
    S = mbem.Solver(xyz, tri, k0, eps)
    try:
        for D, a, b in zip(S.deps_blocks(), *blocks):
            fd = (a - b) / (2 * h)
            assert float((D.cpu() - fd).norm()) <= 1e-5 * float(fd.norm())
    finally:
        S.close()


def test_node_in_more_batches_than_a_turn_takes():
    """Poles of valence 900: 180 batches hold a pole, more than the 170 slots of
    one turn of the gather.  A pole-pole entry sums 810 000 element pairs, whose
    roundings of 1.1e-16 add up to about 1e-13."""
    xyz, tri = uv_sphere_p2(900, 2)
    k0, eps, nss = 1.0, 2.0, 2
    P = galerkin.Problem(xyz, tri, k0, eps, nss=nss)
    Ko = core.fill(P.xyz, P.tri6, P.phys, nss=nss)
    S = mbem.Solver(xyz, tri, k0, eps, ssq_order=nss)
    try:
        S.fill()
        one = torch.as_tensor(S.perm[:2 * S.nn])
        for K, ref in zip(S.export_blocks(), Ko):
            R = torch.as_tensor(np.asarray(ref))[one][:, one]
            K = K.cpu()
            assert float((K - R).norm()) <= 1e-11 * float(R.norm())
            assert float((K - R).abs().max()) <= 1e-10 * float(R.abs().max())
    finally:
        S.close()
