"""Solves with paired transforms do not depend on the operator's scale: A and C times a power of two scale every
Golub-Kahan scalar by it and leave X as it is.  A paired transform writes the next product's input before that vector's norm is
known, so the slice product would hold ||A||^2 in FP32 if the input carried the vector's own scale.

Every FP32 and BF16 operation of the solve commutes with a power of two while nothing leaves the range of normal numbers,
and |A| = 2^-66 .. 2^66 leaves none when the input is scaled; FP64 scalars commute as well.  So both solves agree to 1e-6
relative, far above a rounding difference of the projected solve and far below what subnormals lose (1e-4 at 1e-20)."""
import numpy as np
import pytest

from tests.gpu_util import rel, to_gpu, to_np

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2103_11847_amd as dk  # noqa: E402

K, LAM = 8, 0.05


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = dk.dctk_create(0)
    yield c
    dk.dctk_destroy(c)


def solve(ctx, gdt, A, B, C, scale):
    op = dk.dctk_op_create(ctx, dk.DCTK_TUBE_TH, gdt, to_gpu(A * scale, torch.float64), C.shape[2],
                           None if B is None else to_gpu(B, torch.float64))
    for adj in (0, 1):
        dk.dctk_op_set_path(op, adj, 0, 0)
    ws = dk.dctk_krylov_create(ctx, op, dk.DCTK_KRYLOV_GKB, K)
    X = torch.full((A.shape[0], A.shape[2], C.shape[2]), float("nan"), device="cuda:0")
    dk.dctk_lsqr_tik_solve(ctx, ws, to_gpu(C * scale, torch.float32), X, dk.make_opts(K, lam=LAM * scale))
    r = dk.dctk_krylov_read(ctx, ws, K, dk.DCTK_KRYLOV_GKB)
    out = np.array(r["alpha"]) / scale, np.array(r["beta"]) / scale, to_np(X)
    dk.dctk_krylov_destroy(ws)
    dk.dctk_op_destroy(op)
    return out


@pytest.mark.parametrize("e", [-70, -62, 66])
@pytest.mark.parametrize("gdt,p,n,two", [("f32", 3, 40, False), ("f32", 5, 72, False), ("f32", 8, 33, False),
                                         ("f32", 8, 136, True), ("f32", 12, 70, False), ("f32", 31, 65, False),
                                         ("bf16", 20, 48, False)])
def test_operator_scale(ctx, gdt, p, n, two, e):
    rng = np.random.default_rng(100 * p + n)
    A = rng.standard_normal((p, n, n)) / np.sqrt(n * p)
    B = rng.standard_normal((p, n, n)) / np.sqrt(n * p) if two else None
    C = rng.standard_normal((p, n, n))
    t = dk.DCTK_F32 if gdt == "f32" else dk.DCTK_BF16
    want, got = solve(ctx, t, A, B, C, 1.0), solve(ctx, t, A, B, C, 2.0 ** e)
    for g, w, what in zip(got, want, ("alpha", "beta", "X")):
        assert rel(g, w) <= 1e-6, (what, rel(g, w))
