"""Golub-Kahan steps on short tubes (p <= 8) whose products run as three kernels with paired transforms, against
the same solve on the fused products (p <= 8 takes both) and against the oracle: every p, slices of aligned and
odd size, more positions than one turn of the workgroups covers, rectangular, two-sided.

Both paths hold FP32 vectors; 6 Golub-Kahan steps move X by a few 2^-24 per step and product of K terms, so the
two agree to 1e-5 (the FP32 product bound) and the restoration to the oracle's within the same."""
import numpy as np
import pytest

from oracle import krylov
from oracle.cprod import Operator
from tests.gpu_util import rel, to_gpu, to_np

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2103_11847_amd as dk  # noqa: E402

K, LAM = 6, 0.05


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = dk.dctk_create(0)
    yield c
    dk.dctk_destroy(c)


def solve(ctx, A, B, C, path):
    op = dk.dctk_op_create(ctx, dk.DCTK_TUBE_TH, dk.DCTK_F32, to_gpu(A, torch.float64), C.shape[2],
                           None if B is None else to_gpu(B, torch.float64))
    for adj in (0, 1):
        dk.dctk_op_set_path(op, adj, path, 0)
    ws = dk.dctk_krylov_create(ctx, op, dk.DCTK_KRYLOV_GKB, K)
    X = torch.full((A.shape[0], A.shape[2], C.shape[2]), float("nan"), device="cuda:0")
    dk.dctk_lsqr_tik_solve(ctx, ws, to_gpu(C, torch.float32), X, dk.make_opts(K, lam=LAM))
    out = to_np(X)
    dk.dctk_krylov_destroy(ws)
    dk.dctk_op_destroy(op)
    return out


CASES = [(p, 24, 24, 24, False) for p in range(1, 9)] + [(2, 33, 17, 19, False), (5, 31, 47, 33, False),
                                                         (8, 65, 63, 67, False), (3, 40, 40, 36, True),
                                                         (8, 30, 26, 22, True), (3, 96, 640, 644, False)]


@pytest.mark.parametrize("p,n1,n2,s,two", CASES)
def test_paired_short_tubes(ctx, p, n1, n2, s, two):
    rng = np.random.default_rng(100 * p + n1)
    A = rng.standard_normal((p, n1, n2)) / np.sqrt(n1 * p)
    B = rng.standard_normal((p, s, s)) / np.sqrt(s * p) if two else None
    C = rng.standard_normal((p, n1, s)).astype(np.float32).astype(np.float64)
    X = solve(ctx, A, B, C, 0)
    if not two:
        assert rel(X, solve(ctx, A, B, C, 1)) <= 1e-5
    if n2 <= 100:
        ref = krylov.dc_gk(Operator(A, B) if two else Operator(A), C, K, lam=LAM)
        assert rel(X, ref["X"]) <= 1e-5
