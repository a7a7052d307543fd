"""Right-hand sides solved in step (mbem_solve with several columns) against the
same columns solved one by one: group sizes up to and past the limit of 16,
columns that converge after very different step counts, zero columns, the
iteration limit, with and without preconditioner, every storage form."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2604_21181_amd import mbem  # noqa: E402
from workloads.meshes import icosphere_p2, uv_sphere_p2  # noqa: E402

MESHES = {"uv70": lambda: uv_sphere_p2(7, 6), "ico320": lambda: icosphere_p2(320)}
FORMS = {"fp64": dict(), "mixed": dict(precision=1), "store": dict(precision=1, near_store=True)}


def _columns(S, n):
    """Plane waves, a random column, a column of Z P^-1 (one or two steps), a
    zero column, in turn."""
    rng = np.random.default_rng(n)
    out = []
    for c in range(n):
        if c % 4 == 0:
            k = rng.normal(size=3)
            k /= np.linalg.norm(k)
            p = np.cross(k, rng.normal(size=3))
            out.append(S.rhs([k], [p / np.linalg.norm(p)])[0])
            continue
        v = torch.as_tensor(rng.normal(size=S.N) + 1j * rng.normal(size=S.N), device=S.device)
        if c % 4 == 2:
            v = S.matvec(S.precond_apply(v))
        out.append(v if c % 4 != 3 else torch.zeros_like(v))
    return torch.stack(out)


@pytest.mark.parametrize("n", [2, 3, 5, 18])
@pytest.mark.parametrize("form", sorted(FORMS))
@pytest.mark.parametrize("mesh", sorted(MESHES))
def test_group_as_one_by_one(mesh, form, n):
    xyz, tri = MESHES[mesh]()
    S = mbem.Solver(xyz, tri, 1.4, 3.0 + 0.2j, **FORMS[form])
    try:
        S.fill()
        S.precond_setup(60)
        B = _columns(S, n)
        tol = 1e-10
        X, st, code = S.solve(B, tol)
        assert code == 0 and st.rel_resid <= tol
        its = 0
        for c in range(n):
            x, s1, code = S.solve(B[c], tol)
            assert code == 0
            its += s1.iters
            # both residuals below tol: the solutions differ by at most 2 tol
            # times a condition number of a few hundred
            assert float((X[c] - x[0]).norm()) <= 1e-6 * float(x.norm()), c
        assert abs(st.iters - its) <= n           # rounding moves a column's count by a step
    finally:
        S.close()


@pytest.mark.parametrize("block", [1, 7, 33, 512])
@pytest.mark.parametrize("form", ["fp64", "mixed"])
def test_block_sizes(form, block):
    """Odd blocks, a short last block, one block: the fused preconditioner step
    for one, two and three systems against the dense system."""
    xyz, tri = MESHES["uv70"]()
    S = mbem.Solver(xyz, tri, 1.4, 3.0 + 0.2j, **FORMS[form])
    try:
        S.fill()
        S.precond_setup(block)
        Z = S.export_dense()
        B = _columns(S, 4)[:3]
        for n in (1, 2, 3):
            X, _, code = S.solve(B[:n], 1e-10)
            assert code == 0
            R = X @ Z.T.contiguous() - B[:n]
            # the solve's own criterion, and sums of 568 terms
            assert bool((R.norm(dim=1) <= 1.1e-10 * B[:n].norm(dim=1)).all())
    finally:
        S.close()


@pytest.mark.parametrize("form", ["fp64", "mixed"])
def test_without_preconditioner_and_at_the_limit(form):
    xyz, tri = MESHES["uv70"]()
    S = mbem.Solver(xyz, tri, 1.4, 3.0, **FORMS[form])
    try:
        S.fill()
        S.precond_setup(0)
        B = torch.stack([S.rhs([[0, 0, 1.0]], [[1.0, 0, 0]])[0], S.rhs([[1.0, 0, 0]], [[0, 1.0, 0]])[0]])
        X, st, code = S.solve(B, 1e-8)
        assert code == 0
        for c in range(2):
            x, _, code = S.solve(B[c], 1e-8)
            assert code == 0 and float((X[c] - x[0]).norm()) <= 1e-4 * float(x.norm())
        _, st, code = S.solve(B, 1e-8, maxit=1, max_refine=1)
        assert code == mbem.MBEM_ENOCONV and st.iters == 2 and st.rel_resid > 1e-8
    finally:
        S.close()


def test_a_column_that_is_not_finite_is_named():
    xyz, tri = MESHES["uv70"]()
    S = mbem.Solver(xyz, tri, 1.4, 3.0)
    try:
        S.fill()
        B = torch.ones((3, S.N), dtype=torch.complex128, device=S.device)
        B[1, 5] = complex(float("nan"), 0.0)
        with pytest.raises(mbem.MbemError, match="column 1"):
            S.solve(B, 1e-8)
    finally:
        S.close()


def test_compressed_operator():
    xyz, tri = MESHES["ico320"]()
    S = mbem.Solver(xyz, tri, 1.4, 3.0)
    try:
        S.fill_compressed()
        S.precond_setup(60)
        B = _columns(S, 3)
        X, _, code = S.solve(B, 1e-8)
        assert code == 0
        for c in range(3):
            x, _, code = S.solve(B[c], 1e-8)
            assert code == 0 and float((X[c] - x[0]).norm()) <= 1e-12 * float(x.norm())
    finally:
        S.close()
