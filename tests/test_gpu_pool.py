"""Memory handed out again by a context (pool.cpp): operators of changing size
one after another, an operator used from a second context and stream, and
threads with a context each, all against values computed in a fresh context."""
import threading

import numpy as np
import pytest

from workloads import icosphere_p2

pytestmark = pytest.mark.gpu

CASES = [(80, dict()), (320, dict(precision=1)), (80, dict(precision=1, near_store=True)), (20, dict()),
         (320, dict(frame=1)), (80, dict())]


def _one_pass(mbem, ctx, nt, kw, stream=None):
    """Fill, setup, right-hand side and solve with handles of ctx; x."""
    import torch
    xyz, tri = icosphere_p2(nt)
    mesh = mbem.mbem_mesh_create(ctx, xyz, tri)
    p = mbem.make_params(1.2, 3.0 + 0.1j, **kw)
    op, _ = mbem.mbem_fill(ctx, mesh, p)
    mbem.mbem_precond_setup(ctx, op, 30)
    n = 4 * xyz.shape[0]
    b = torch.zeros(1, n, dtype=torch.complex128, device="cuda")
    x = torch.zeros_like(b)
    torch.cuda.synchronize()
    mbem.mbem_rhs_planewave(ctx, mesh, p, [0, 0, 1.0], [1.0, 0, 0], b)
    code, _ = mbem.mbem_solve(ctx, op, b, x, 1, 1e-10)
    assert code == 0
    mbem.mbem_op_destroy(op)
    mbem.mbem_mesh_destroy(mesh)
    return x.cpu().numpy()


def _fresh(mbem, nt, kw):
    ctx = mbem.mbem_ctx_create(0)
    try:
        return _one_pass(mbem, ctx, nt, kw)
    finally:
        mbem.mbem_ctx_destroy(ctx)


def _near(a, b, kw):
    # the same kernels on the same inputs: the singular pairs' atomics round
    # in another order (1e-16 in FP64 blocks, 6e-8 in complex64 blocks; a
    # conditioning of at most 100)
    tol = 1e-5 if kw.get("precision") and not kw.get("near_store") else 1e-9
    return np.linalg.norm(a - b) <= tol * np.linalg.norm(b)


def test_handles_of_changing_size_in_one_context():
    from paper_2604_21181_amd import mbem
    ref = [_fresh(mbem, nt, kw) for nt, kw in CASES]
    ctx = mbem.mbem_ctx_create(0)
    try:
        for rep in range(2):
            for (nt, kw), r in zip(CASES, ref):
                assert _near(_one_pass(mbem, ctx, nt, kw), r, kw), (rep, nt, kw)
    finally:
        mbem.mbem_ctx_destroy(ctx)


def test_operator_used_from_another_context():
    """The second context reads the operator on its own stream; destroying it
    and filling the next one must not touch blocks still being read."""
    import torch
    from paper_2604_21181_amd import mbem
    xyz, tri = icosphere_p2(320)
    c1 = mbem.mbem_ctx_create(0)
    side = torch.cuda.Stream()
    c2 = mbem.mbem_ctx_create(0, side.cuda_stream)
    n = 4 * xyz.shape[0]
    x = torch.randn(n, dtype=torch.complex128, device="cuda")
    try:
        mesh = mbem.mbem_mesh_create(c1, xyz, tri)
        got = []
        for eps in (2.0, 3.0, 2.0, 3.0):
            p = mbem.make_params(1.0, eps)
            op, _ = mbem.mbem_fill(c1, mesh, p)
            y = torch.zeros(40, n, dtype=torch.complex128, device="cuda")
            torch.cuda.synchronize()
            for r in range(40):
                mbem.mbem_matvec_noalloc(c2, op, x, y[r])     # enqueued only
            mbem.mbem_op_destroy(op)
            got.append(y)
        torch.cuda.synchronize()
        for y in got:
            assert bool((y == y[0]).all())
        # two fills of the same permittivity: the singular pairs' FP64 atomics
        # round in another order
        for a, b in ((0, 2), (1, 3)):
            assert float((got[a][0] - got[b][0]).norm()) <= 1e-13 * float(got[a][0].norm())
        assert float((got[0][0] - got[1][0]).norm()) > 1e-3 * float(got[0][0].norm())
        mbem.mbem_mesh_destroy(mesh)
    finally:
        mbem.mbem_ctx_destroy(c2)
        mbem.mbem_ctx_destroy(c1)


def test_threads_with_a_context_each():
    import torch
    from paper_2604_21181_amd import mbem
    ref = {c: _fresh(mbem, *CASES[c]) for c in (0, 1, 4)}
    bad = []

    def work(c):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                ctx = mbem.mbem_ctx_create(0)
                for _ in range(4):
                    if not _near(_one_pass(mbem, ctx, *CASES[c]), ref[c], CASES[c][1]):
                        bad.append(c)
                mbem.mbem_ctx_destroy(ctx)
        except Exception as e:      # reported by the main thread
            bad.append(e)

    threads = [threading.Thread(target=work, args=(c,)) for c in (0, 1, 4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad, bad
