"""A graph-captured batch whose instances fall into one, two or three chains (fused products; short tubes as three
kernels; long tubes): every replay equals the single solves bit for bit, also between the caller's own work on the
stream, on another stream and under capture of the caller's stream."""
import numpy as np
import pytest

from tests.gpu_util import to_gpu

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2103_11847_amd as dk  # noqa: E402

K = 6


@pytest.fixture()
def made():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = dk.dctk_create(0)
    held = []

    def make(ps):
        rng = np.random.default_rng(sum(ps))
        out = []
        for i, p in enumerate(ps):
            n = 40 + 3 * i
            A = rng.standard_normal((p, n, n)) / n
            op = dk.dctk_op_create(ctx, dk.DCTK_TUBE_TH, dk.DCTK_F32, to_gpu(A, torch.float64), n)
            ws = dk.dctk_krylov_create(ctx, op, dk.DCTK_KRYLOV_GKB, K)
            C = to_gpu(rng.standard_normal((p, n, n)), torch.float32)
            held.append((op, ws))
            out.append((ws, C, torch.empty_like(C)))
        return ctx, out
    yield make
    torch.cuda.synchronize()
    for op, ws in held:
        dk.dctk_krylov_destroy(ws)
        dk.dctk_op_destroy(op)
    dk.dctk_destroy(ctx)


@pytest.mark.parametrize("ps", [(3, 3), (3, 8), (8, 31, 3), (3, 31, 8, 5, 2, 16)])
def test_chains(made, ps):
    ctx, insts = made(ps)
    opts = dk.make_opts(K)
    ref = []
    for ws, C, X in insts:
        dk.dctk_lsqr_tik_solve(ctx, ws, C, X, opts)
        ref.append(X.clone())
    plan = dk.dctk_batch_create(ctx, [i[0] for i in insts], [i[1] for i in insts], [i[2] for i in insts], opts)

    def check(what):
        for (_, _, X), r in zip(insts, ref):
            assert torch.equal(X, r), what
            X.fill_(float("nan"))
    try:
        for rep in range(3):
            dk.dctk_batch_run(ctx, plan)
            check("replay %d" % rep)      # the caller's stream waits for every chain
        # inputs changed on the stream right before the run: doubled data doubles X exactly (powers of two)
        for _, C, _ in insts:
            C.mul_(2.0)
        dk.dctk_batch_run(ctx, plan)
        for _, C, _ in insts:
            C.mul_(0.5)
        for (_, _, X), r in zip(insts, ref):
            assert torch.equal(X, 2.0 * r)
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        dk.dctk_set_stream(ctx, s)
        with torch.cuda.stream(s):
            dk.dctk_batch_run(ctx, plan)
            check("another stream")
            g = torch.cuda.CUDAGraph()
            s.synchronize()
            g.capture_begin(capture_error_mode="thread_local")
            dk.dctk_batch_run(ctx, plan)
            g.capture_end()
            for rep in range(3):
                g.replay()
                check("captured %d" % rep)
        s.synchronize()
        dk.dctk_set_stream(ctx, torch.cuda.current_stream())
    finally:
        torch.cuda.synchronize()
        dk.dctk_batch_destroy(plan)
