"""FP32 slice products on the BF16 matrix cores (an FP32 number as three bfloat16 numbers): edges of the
tiles and of the 32-long chunks, both operand orders, and the values the split cannot represent.

With p = 1 the transforms are the identity, so a product is one GEMM: every element must lie within
(K + 6 ceil(K / 32) + 2) 2^-23 (|A| |X|) of the FP64 product -- one rounding per term of a 32-long chunk and
per accumulation, in any order -- plus the FP32 rounding of A (2^-24), which the operator makes."""
import numpy as np
import pytest

from tests.gpu_util import rel, to_gpu, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dk():
    import torch
    assert torch.cuda.is_available()
    import paper_2103_11847_amd as dk
    return dk


@pytest.fixture(scope="module")
def ctx(dk):
    c = dk.dctk_create(0)
    yield c
    dk.dctk_destroy(c)


def product(dk, ctx, A, B, X, tile, adjoint):
    import torch
    p, n1, n2 = A.shape
    op = dk.dctk_op_create(ctx, dk.DCTK_TUBE_TH, dk.DCTK_F32, to_gpu(A, torch.float64), X.shape[2],
                           None if B is None else to_gpu(B, torch.float64))
    dk.dctk_op_set_path(op, 1 if adjoint else 0, 0, tile)
    Xg = to_gpu(X, torch.float32)
    Y = torch.full((p, n2 if adjoint else n1, X.shape[2]), float("nan"), device="cuda:0", dtype=torch.float32)
    (dk.dctk_cprod_T if adjoint else dk.dctk_cprod)(ctx, op, 1.0, Xg, 0.0, Y)
    torch.cuda.synchronize()
    dk.dctk_op_destroy(op)
    return Y


def bound(A, X):
    K = A.shape[-1]
    return ((K + 6 * -(-K // 32) + 2) * 2.0 ** -23 + 2.0 ** -24) * (np.abs(A) @ np.abs(X)) + 1e-37


@pytest.mark.parametrize("tile", [64, 128])
@pytest.mark.parametrize("n1,n2,s", [(1, 1, 1), (3, 33, 5), (64, 32, 64), (65, 31, 63), (129, 64, 127), (130, 211, 66),
                                     (128, 96, 128), (200, 257, 131)])
def test_edges(dk, ctx, n1, n2, s, tile):
    rng = np.random.default_rng(n1 * 1000 + n2)
    A = rng.standard_normal((1, n1, n2)) * np.exp(rng.uniform(-6, 6, (1, n1, n2)))
    X = (rng.standard_normal((1, n2, s)) * np.exp(rng.uniform(-6, 6, (1, n2, s)))).astype(np.float32).astype(np.float64)
    R = rng.standard_normal((1, n1, s)).astype(np.float32).astype(np.float64)
    Y = to_np(product(dk, ctx, A, None, X, tile, False))
    assert (np.abs(Y - A @ X) <= bound(A, X)).all()
    At = A.transpose(0, 2, 1)
    Z = to_np(product(dk, ctx, A, None, R, tile, True))
    assert (np.abs(Z - At @ R) <= bound(At, R)).all()


@pytest.mark.parametrize("tile", [64, 128])
@pytest.mark.parametrize("n,s", [(40, 37), (66, 64), (96, 130)])
def test_two_sided(dk, ctx, n, s, tile):
    """The adjoint's right factor has its contraction index contiguous (both operands in k)."""
    rng = np.random.default_rng(n + s)
    A, B = rng.standard_normal((1, n, n)), rng.standard_normal((1, s, s))
    X = rng.standard_normal((1, n, s)).astype(np.float32).astype(np.float64)
    for adjoint in (False, True):
        Y = to_np(product(dk, ctx, A, B, X, tile, adjoint))
        L, Rt = (A.transpose(0, 2, 1), B.transpose(0, 2, 1)) if adjoint else (A, B)
        # the intermediate's error passes through the second factor
        tol = bound(L, X) @ np.abs(Rt) * 1.01 + bound(np.abs(L) @ np.abs(X), np.abs(Rt))
        assert (np.abs(Y - L @ X @ Rt) <= tol).all()


def test_largest_tile(dk, ctx):
    """64 slices of 510 x 509 outputs: 256 x 256 tiles, one per CU, ragged in both directions, K = 70."""
    from oracle.cprod import Operator
    rng = np.random.default_rng(5)
    A, X = rng.standard_normal((64, 510, 70)), rng.standard_normal((64, 70, 509))
    ref = Operator(A).apply(X.astype(np.float32).astype(np.float64))
    assert rel(to_np(product(dk, ctx, A, None, X, 0, False)), ref) <= 1e-5


@pytest.mark.parametrize("tile", [64, 128])
@pytest.mark.parametrize("what", ["inf", "-inf", "nan", "huge", "tiny", "subnormal", "A inf"])
def test_values_beyond_the_split(dk, ctx, what, tile):
    """Infinities, NaN, numbers that round to infinity in bfloat16 and numbers below 2^-110 give what the FP32
    instruction gives (the 32 x 32 tiles)."""
    import torch
    rng = np.random.default_rng(3)
    A, X = rng.standard_normal((1, 100, 70)), rng.standard_normal((1, 70, 90)).astype(np.float32)
    if what in ("inf", "-inf", "nan"):
        X[0, 69, 17] = float(what)
    elif what == "huge":
        X[0, 3, 17] = np.float32(3.4e38)
        A[0, :, 3] = 0.5
    elif what == "tiny":
        X *= np.float32(2.0 ** -115)
    elif what == "subnormal":
        X *= np.float32(2.0 ** -130)
    else:
        A[0, 99, 0] = np.inf
    got, want = product(dk, ctx, A, None, X, tile, False), product(dk, ctx, A, None, X, 32, False)
    assert torch.equal(got.isnan(), want.isnan()) and torch.equal(got.isinf(), want.isinf())
    assert torch.equal(got[got.isinf()], want[want.isinf()])
    if what in ("tiny", "subnormal"):
        assert torch.equal(got, want)
    fine = want.isfinite()
    assert torch.allclose(got[fine], want[fine], rtol=1e-4, atol=1e-3 if what != "tiny" else 0.0)
