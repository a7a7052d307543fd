"""The transposed product (adjoint.hip, k_gemvt_part and k_combine_t) inside the
adjoint solve: the residual of its solution against the exported dense system,
for chunks of 8 to 64 rows with a short last one, all storage forms, mass rows
longer than the workgroup's groups and the near store."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2604_21181_amd import mbem  # noqa: E402
from workloads.meshes import cubesphere_p2, icosphere_p2, uv_sphere_p2  # noqa: E402

MESHES = {"ico20": lambda: icosphere_p2(20), "uv410": lambda: uv_sphere_p2(41, 6), "cube768": lambda: cubesphere_p2(8)}
FORMS = {"fp64": dict(), "mixed": dict(precision=1), "store": dict(precision=1, near_store=True)}


@pytest.mark.parametrize("form", sorted(FORMS))
@pytest.mark.parametrize("mesh", sorted(MESHES))
def test_residual_of_the_adjoint_solve(mesh, form):
    xyz, tri = MESHES[mesh]()
    S = mbem.Solver(xyz, tri, 1.4, 3.0 + 0.2j, **FORMS[form])
    try:
        S.fill()
        S.precond_setup(60)
        g = torch.randn(S.N, dtype=torch.complex128, device=S.device, generator=torch.Generator(S.device).manual_seed(3))
        lam, st, code = S.solve_adjoint(g, tol=1e-11, maxit=400)
        assert code == 0
        r = S.export_dense().T.contiguous() @ lam[0] - g
        # the solve's own residual, and N = 6e3 sums of 6e3 terms: 1e-12
        assert float(r.norm()) <= 1.2e-11 * float(g.norm())
    finally:
        S.close()
