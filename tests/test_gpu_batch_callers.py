"""Batches of several chains with reorthogonalised steps, with the learned stop and of two callers at once: every
instance equals its own single solve (the learned stop: the batch as one chain on the caller's stream) bit for bit."""
import numpy as np
import pytest

from tests.gpu_util import to_gpu

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2103_11847_amd as dk  # noqa: E402

PS = (3, 31, 8, 5, 2, 16)   # fused products; short tubes and long ones as three kernels


class Insts:
    def __init__(self, ctx, ps, k, seed):
        rng = np.random.default_rng(seed)
        self.ctx, self.ws, self.C, self.X, self.ops = ctx, [], [], [], []
        for i, p in enumerate(ps):
            n = 36 + 5 * i
            A = rng.standard_normal((p, n, n)) / n + np.eye(n)
            op = dk.dctk_op_create(ctx, dk.DCTK_TUBE_TH, dk.DCTK_F32, to_gpu(A, torch.float64), n)
            self.ops.append(op)
            self.ws.append(dk.dctk_krylov_create(ctx, op, dk.DCTK_KRYLOV_GKB, k))
            self.C.append(to_gpu(rng.standard_normal((p, n, n)), torch.float32))
            self.X.append(torch.empty_like(self.C[-1]))

    def singles(self, opts):
        out = []
        for ws, C, X in zip(self.ws, self.C, self.X):
            dk.dctk_lsqr_tik_solve(self.ctx, ws, C, X, opts)
            out.append(X.clone())
            X.fill_(float("nan"))
        return out

    def plan(self, opts, graph=True, **kw):
        return dk.dctk_batch_create(self.ctx, self.ws, self.C, self.X, opts, graph, **kw)

    def equal(self, ref):
        same = all(torch.equal(X, r) for X, r in zip(self.X, ref))
        for X in self.X:
            X.fill_(float("nan"))
        return same

    def free(self):
        torch.cuda.synchronize()
        for ws, op in zip(self.ws, self.ops):
            dk.dctk_krylov_destroy(ws)
            dk.dctk_op_destroy(op)


@pytest.fixture()
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = dk.dctk_create(0)
    yield c
    torch.cuda.synchronize()
    dk.dctk_destroy(c)


@pytest.mark.parametrize("reorth", ["DCTK_REORTH_V", "DCTK_REORTH_FULL"])
def test_reorthogonalised(ctx, reorth):
    k = 9
    opts = dk.make_opts(k, getattr(dk, reorth))
    b = Insts(ctx, PS, k, 3)
    ref = b.singles(opts)
    plan = b.plan(opts)
    for rep in range(4):
        dk.dctk_batch_run(ctx, plan)
        assert b.equal(ref), rep
    torch.cuda.synchronize()
    dk.dctk_batch_destroy(plan)
    b.free()


def test_learned_stop(ctx):
    k = 20
    opts = dk.make_opts(k, dk.DCTK_REORTH_NONE, 0, -1.0)
    net = dk.dctk_mlp_create(ctx, 11)
    dk.dctk_mlp_set_scaling(net, -3.0, 1.0, 6.0, 12.0)
    b = Insts(ctx, PS, k, 4)
    one = b.plan(opts, False, mlp=net, gate=1.05)
    dk.dctk_batch_run(ctx, one)
    limits = dk.dctk_batch_learned(ctx, one, len(PS))
    ref = [X.clone() for X in b.X]
    assert len(set(limits[0])) > 1 and all(torch.isfinite(r).all() for r in ref)
    dk.dctk_batch_destroy(one)
    plan = b.plan(opts, True, mlp=net, gate=1.05)
    for rep in range(4):
        for X in b.X:
            X.fill_(float("nan"))
        dk.dctk_batch_run(ctx, plan)
        assert dk.dctk_batch_learned(ctx, plan, len(PS)) == limits
        assert b.equal(ref), rep
    dk.dctk_batch_destroy(plan)
    dk.dctk_mlp_destroy(net)
    b.free()


def test_two_callers():
    """Runs from two streams, the first held back: neither disturbs the other."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    k = 6
    opts = dk.make_opts(k)
    streams = [torch.cuda.Stream() for _ in range(2)]
    ctxs = [dk.dctk_create(0, s) for s in streams]
    insts, refs, plans = [], [], []
    for c, s, seed in zip(ctxs, streams, (5, 6)):
        with torch.cuda.stream(s):
            b = Insts(c, PS, k, seed)
            refs.append(b.singles(opts))
            plans.append(b.plan(opts))
            insts.append(b)
    torch.cuda.synchronize()
    for rep in range(4):
        with torch.cuda.stream(streams[0]):
            torch.cuda._sleep(20000000)   # some 10 ms
        for c, s, p in zip(ctxs, streams, plans):
            with torch.cuda.stream(s):
                for _ in range(1 + rep % 2):
                    dk.dctk_batch_run(c, p)
        for s, b, r in zip(streams, insts, refs):
            with torch.cuda.stream(s):
                assert b.equal(r), rep
    torch.cuda.synchronize()
    for p in plans:
        dk.dctk_batch_destroy(p)
    for b in insts:
        b.free()
    for c in ctxs:
        dk.dctk_destroy(c)
