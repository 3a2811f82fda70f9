"""The O(p log p) tube transforms of 128 <= p <= 1024 whose FFT runs in registers, at the edges of their tiles (64
positions at p = 128 and 32 above in FP32, half that in FP64): fewer positions than a tile, whole tiles, odd counts,
more tiles than one turn of the workgroups covers; and the same kernels inside products and solves (scaled input,
its stored copy, src, partial sums) on slices of odd size.

Tolerances: the transforms' documented ones, FP64 1e-14 p and FP32 1e-6 + 8e-9 p (the diagonal of M magnifies the
FFT's rounding by up to 2p / pi in its last rows); where many positions are covered by comparing with the same columns
transformed in a short call, the two are the same kernel on the same numbers and must agree exactly.  A product is two
transforms and K <= 24 terms: three times that.  A solve is 5 steps
of two products, and lambda = 0.05 magnifies what they leave by |A| / lambda < 50: 500 times a product's."""
import numpy as np
import pytest

from oracle import krylov
from oracle import tube as otube
from oracle.cprod import Operator
from tests.gpu_util import rel, to_gpu, to_np

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2103_11847_amd as dk  # noqa: E402

VT = {dk.DCTK_F64: torch.float64, dk.DCTK_F32: torch.float32}
WHICH = [dk.DCTK_MAT_L, dk.DCTK_MAT_LINV, dk.DCTK_MAT_LINVT, dk.DCTK_MAT_LT]
TYPES = [dk.DCTK_F32, dk.DCTK_F64]


def tol(dtype, p):
    return 1e-14 * p if dtype == dk.DCTK_F64 else 1e-6 + 8e-9 * p


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = dk.dctk_create(0)
    yield c
    dk.dctk_synchronize(c)
    dk.dctk_destroy(c)


@pytest.mark.parametrize("dtype", TYPES)
@pytest.mark.parametrize("p", [128, 256, 512, 1024])
def test_tile_edges(ctx, dtype, p):
    nb = (64 if p == 128 else 32) // (2 if dtype == dk.DCTK_F64 else 1)
    L = otube.transform_matrix(p, "th")
    Li = otube.inverse_transform_matrix(p, "th")
    G = {dk.DCTK_MAT_L: L, dk.DCTK_MAT_LINV: Li, dk.DCTK_MAT_LINVT: Li.T, dk.DCTK_MAT_LT: L.T}
    rng = np.random.default_rng(p)
    for count in (1, 2, 3, nb - 1, nb, nb + 1, 2 * nb, 3 * nb + 5):
        x = to_gpu(rng.standard_normal((p, count)), VT[dtype])
        for which in WHICH:
            out = torch.full_like(x, float("nan"))
            dk.dctk_tube_fast(ctx, dk.DCTK_TUBE_TH, which, x, out)
            assert rel(to_np(out), G[which] @ to_np(x)) <= tol(dtype, p), (count, which)


@pytest.mark.parametrize("dtype", TYPES)
@pytest.mark.parametrize("p", [128, 256, 512, 1024])
def test_many_tiles(ctx, dtype, p):
    # two turns of 1024 (p <= 256), 512 or 256 resident workgroups and a ragged end
    nb = (64 if p == 128 else 32) // (2 if dtype == dk.DCTK_F64 else 1)
    count = nb * (2100 if p <= 256 else 530) + 7
    x = torch.randn((p, count), dtype=VT[dtype], device="cuda:0")
    cols = [0, nb * 3, (count // nb // 2) * nb, (count // nb - 1) * nb]
    for which in WHICH:
        out = torch.full_like(x, float("nan"))
        dk.dctk_tube_fast(ctx, dk.DCTK_TUBE_TH, which, x, out)
        assert bool(torch.isfinite(out).all())
        for c in cols:
            part = x[:, c:c + nb].contiguous()
            ref = torch.full_like(part, float("nan"))
            dk.dctk_tube_fast(ctx, dk.DCTK_TUBE_TH, which, part, ref)
            dk.dctk_synchronize(ctx)
            assert torch.equal(out[:, c:c + nb], ref), (c, which)


@pytest.mark.parametrize("dtype", TYPES)
@pytest.mark.parametrize("p,n1,n2,s", [(128, 24, 20, 13), (256, 9, 7, 5), (512, 12, 8, 8), (1024, 5, 4, 3)])
def test_products_and_solves(ctx, dtype, p, n1, n2, s):
    rng = np.random.default_rng(p + n1)
    A = rng.standard_normal((p, n1, n2)) / np.sqrt(n1 * p)
    X0 = to_gpu(rng.standard_normal((p, n2, s)), VT[dtype])
    C0 = to_gpu(rng.standard_normal((p, n1, s)), VT[dtype])
    ref = Operator(A)
    op = dk.dctk_op_create(ctx, dk.DCTK_TUBE_TH, dtype, to_gpu(A, torch.float64), s)
    Y = to_gpu(np.ones((p, n1, s)), VT[dtype])
    dk.dctk_cprod(ctx, op, -0.5, X0, 2.0, Y)
    assert rel(to_np(Y), -0.5 * ref.apply(to_np(X0)) + 2.0) <= 3 * tol(dtype, p)
    X = torch.full_like(X0, float("nan"))
    dk.dctk_cprod_T(ctx, op, 1.0, C0, 0.0, X)
    assert rel(to_np(X), ref.adjoint(to_np(C0))) <= 3 * tol(dtype, p)
    ws = dk.dctk_krylov_create(ctx, op, dk.DCTK_KRYLOV_GKB, 5)
    dk.dctk_lsqr_tik_solve(ctx, ws, C0, X, dk.make_opts(5, lam=0.05))
    assert rel(to_np(X), krylov.dc_gk(ref, to_np(C0), 5, lam=0.05)["X"]) <= 1500 * tol(dtype, p)
    dk.dctk_krylov_destroy(ws)
    dk.dctk_op_destroy(op)
