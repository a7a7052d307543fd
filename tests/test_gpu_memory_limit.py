"""Calls with little device memory left: solves with several right-hand sides
take smaller groups and keep no memory that a later call needs, fills take
smaller bands, and a call that fails leaves nothing half made."""
import pytest

from workloads import icosphere_p2

pytestmark = pytest.mark.gpu

MIB = 1 << 20


def _take(n):
    """Takes device memory until n bytes are free."""
    import torch
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    held = []
    for _ in range(2):           # a large block frees some memory of the runtime's own
        more = torch.cuda.mem_get_info()[0] - n
        if more > 0:
            held.append(torch.empty(more, dtype=torch.uint8, device="cuda"))
    assert torch.cuda.mem_get_info()[0] <= n + 4 * MIB
    return held


@pytest.fixture(scope="module")
def most():
    """All but 5 GiB, taken once: giving so much back takes the driver a while."""
    import torch
    held = _take(5 << 30)
    yield
    held.clear()
    torch.cuda.empty_cache()


@pytest.fixture
def leave(most):
    import torch
    held = []
    yield lambda n: held.extend(_take(n))
    held.clear()
    torch.cuda.empty_cache()


def _problem(mbem, nrhs):
    import torch
    xyz, tri = icosphere_p2(1280)
    ctx = mbem.mbem_ctx_create(0)
    mesh = mbem.mbem_mesh_create(ctx, xyz, tri)
    p = mbem.make_params(1.0, 2.0)
    op, _ = mbem.mbem_fill(ctx, mesh, p)                 # 1202 MiB, and 224 MiB of scratch
    mbem.mbem_precond_setup(ctx, op, 100)
    b = torch.randn(nrhs, 4 * xyz.shape[0], dtype=torch.complex128, device="cuda")
    return ctx, mesh, p, op, b, torch.zeros_like(b)


def _close(mbem, ctx, mesh, *ops):
    for op in ops:
        mbem.mbem_op_destroy(op)
    mbem.mbem_mesh_destroy(mesh)
    mbem.mbem_ctx_destroy(ctx)


@pytest.mark.parametrize("room", [1100, 500])
def test_solve_with_little_memory(leave, room):
    """Sixteen systems of 100 steps take 520 MiB; in 500 they need smaller
    groups.  The solutions agree to the tolerance, for a conditioning below 100."""
    import torch
    from paper_2604_21181_amd import mbem
    ctx, mesh, p, op, b, x = _problem(mbem, 16)
    ref = torch.zeros_like(b)
    code, _ = mbem.mbem_solve(ctx, op, b, ref, 16, 1e-9, maxit=100)
    assert code == 0
    leave(room * MIB)
    code, st = mbem.mbem_solve(ctx, op, b, x, 16, 1e-9, maxit=100)
    assert code == 0 and st.rel_resid <= 1e-9
    assert float((x - ref).norm()) <= 1e-6 * float(ref.norm())
    _close(mbem, ctx, mesh, op)


def test_a_group_solve_keeps_no_memory_from_the_next_fill(leave):
    """1700 MiB and the kept 224 hold either the workspace of sixteen systems of
    160 steps (830 MiB) or a second operator and its scratch (1426 MiB), in turn
    but not together."""
    from paper_2604_21181_amd import mbem
    ctx, mesh, p, op, b, x = _problem(mbem, 16)
    leave(1700 * MIB)
    code, _ = mbem.mbem_solve(ctx, op, b, x, 16, 1e-9, maxit=160)
    assert code == 0
    second, _ = mbem.mbem_fill(ctx, mesh, p)
    _close(mbem, ctx, mesh, op, second)


def test_block_solve_after_a_copy_that_did_not_fit(most):
    """The complex64 copy of the operator takes three blocks of 200 MiB; 250 MiB
    and the kept scratch hold at most two."""
    import torch
    from paper_2604_21181_amd import mbem
    ctx, mesh, p, op, b, x = _problem(mbem, 4)
    ref = torch.zeros_like(b)
    room = _take(250 * MIB)
    with pytest.raises(mbem.MbemError, match="complex64 operator copy"):
        mbem.mbem_solve_block(ctx, op, b, x, 4, 1e-8)
    del room[:]
    torch.cuda.empty_cache()
    code, st = mbem.mbem_solve_block(ctx, op, b, x, 4, 1e-8)
    assert code == 0
    mbem.mbem_solve(ctx, op, b, ref, 4, 1e-9)
    assert float((x - ref).norm()) <= 1e-5 * float(ref.norm())
    _close(mbem, ctx, mesh, op)


@pytest.mark.parametrize("room", [1340, 1250])
@pytest.mark.parametrize("frame", [0, 1])
@pytest.mark.parametrize("paper", [0, 1])
def test_fill_with_little_memory(leave, paper, frame, room):
    """Three blocks of 401 MiB and the tables leave 120 and 30 MiB for the bands'
    scratch, which takes 224.  The blocks agree to the rounding of the singular
    pairs' additions, whose order varies: 1e-16 of the blocks' scale each."""
    import torch
    from paper_2604_21181_amd import mbem
    xyz, tri = icosphere_p2(1280)
    p = mbem.make_params(1.3, 2.6 + 0.1j, quadrature=paper, frame=frame)
    x = torch.randn(4 * xyz.shape[0], dtype=torch.complex128, device="cuda")
    y = []
    for n in (None, room):
        ctx = mbem.mbem_ctx_create(0)
        mesh = mbem.mbem_mesh_create(ctx, xyz, tri)
        if n:
            leave(n * MIB)
        op, _ = mbem.mbem_fill(ctx, mesh, p)
        y.append(torch.zeros_like(x))
        mbem.mbem_matvec(ctx, op, x, y[-1])
        _close(mbem, ctx, mesh, op)
    assert float((y[0] - y[1]).norm()) <= 1e-13 * float(y[0].norm())
