"""FP32 slice products on the BF16 matrix cores with operands that three bfloat16 numbers do not hold (below 2^-110) beside
or times large ones, so that the results are ordinary numbers: small entries of either operand, small rows, columns and
padding beside normal ones, subnormal operands whose three parts are all zero.

p = 1, one product: every element within the bound of the FP32 product, (K + 6 ceil(K / 32) + 2) 2^-23 (|A| |X|), plus the
FP32 rounding of A (2^-24 of it, and 2^-150 for a subnormal entry) -- the bound holds for the FP32 instruction and does
not for operands that lost bits."""
import numpy as np
import pytest

from tests.gpu_util import to_gpu, to_np

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2103_11847_amd as dk  # noqa: E402


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = dk.dctk_create(0)
    yield c
    dk.dctk_destroy(c)


def product(ctx, A, B, X, tile, adjoint):
    op = dk.dctk_op_create(ctx, dk.DCTK_TUBE_TH, dk.DCTK_F32, to_gpu(A, torch.float64), X.shape[2],
                           None if B is None else to_gpu(B, torch.float64))
    dk.dctk_op_set_path(op, 1 if adjoint else 0, 0, tile)
    Xg = to_gpu(X, torch.float32)
    Y = torch.full((A.shape[0], A.shape[2 if adjoint else 1], X.shape[2]), float("nan"), device="cuda:0")
    (dk.dctk_cprod_T if adjoint else dk.dctk_cprod)(ctx, op, 1.0, Xg, 0.0, Y)
    out = to_np(Y)
    dk.dctk_op_destroy(op)
    return out


def f32(x):
    return x.astype(np.float32).astype(np.float64)


def check(Y, A, X):
    K = A.shape[-1]
    tol = ((K + 6 * -(-K // 32) + 2) * 2.0 ** -23 + 2.0 ** -24) * (np.abs(A) @ np.abs(X)) + 2.0 ** -148 * K
    assert (np.abs(Y - A @ X) <= tol).all(), np.max(np.abs(Y - A @ X) / tol)


N1, K, S = 200, 75, 150


def operands(what):
    rng = np.random.default_rng(11)
    A, X = f32(rng.standard_normal((1, N1, K))), f32(rng.standard_normal((1, K, S)))
    if what.startswith("A 2^"):        # all of A small, X large
        A = f32(A * 2.0 ** -int(what[4:]))
        X = f32(X * 2.0 ** 100)
    elif what.startswith("X 2^"):
        X = f32(X * 2.0 ** -int(what[4:]))
        A = f32(A * 2.0 ** 100)
    elif what == "small rows":         # normal rows in the same 16 x 16 block
        A[0, 1::3] = f32(A[0, 1::3] * 2.0 ** -122)
    elif what == "small columns":
        X[0, :, 5::7] = f32(X[0, :, 5::7] * 2.0 ** -121)
        A = f32(A * 2.0 ** 30)
    elif what == "one small column":   # the slice's last, beside the padding's normal numbers
        X[0, :, S - 1] = f32(X[0, :, S - 1] * 2.0 ** -123)
    elif what == "small terms":        # small entries of A meet large rows of X, and only those
        A[0, :, ::2] = f32(A[0, :, ::2] * 2.0 ** -118)
        A[0, :, 1::2] = 0.0
        X[0, ::2] = f32(X[0, ::2] * 2.0 ** 90)
    elif what == "decay":              # an unbanded Gaussian: ordinary results, entries down to the subnormals
        d = np.arange(N1)[:, None] - np.arange(K)[None, :]
        A[0] = f32(np.exp(-d ** 2 / 32.0))
        X[0, :, 20:40] = 0.0
    return A, X


WHAT = ["A 2^112", "A 2^120", "A 2^130", "A 2^142", "X 2^112", "X 2^124", "X 2^140", "small rows", "small columns",
        "one small column", "small terms", "decay"]


@pytest.mark.parametrize("tile", [64, 128])
@pytest.mark.parametrize("what", WHAT)
def test_one_product(ctx, what, tile):
    A, X = operands(what)
    check(product(ctx, A, None, X, tile, False), A, X)
    At = np.ascontiguousarray(A.transpose(0, 2, 1))
    check(product(ctx, At, None, X, tile, True), A, X)


@pytest.mark.parametrize("what", WHAT)
def test_both_contiguous_in_k(ctx, what):
    """The right factor of a two-sided adjoint: Z -> Z B^T after A = I."""
    A, X = operands(what)
    Z = product(ctx, np.eye(N1)[None], np.ascontiguousarray(np.pad(X[0], ((0, S - K), (0, 0))).T)[None],
                np.pad(A, ((0, 0), (0, 0), (0, S - K))), 64, True)
    check(Z, A, X)


def test_largest_tile(ctx):
    """64 slices of 510 x 509 outputs take the 256 x 256 tiles."""
    from oracle.cprod import Operator
    rng = np.random.default_rng(5)
    A, X = rng.standard_normal((64, 510, 40)) * 2.0 ** -120, f32(rng.standard_normal((64, 40, 509)) * 2.0 ** 90)
    Y, ref = product(ctx, A, None, X, 0, False), Operator(A).apply(X)
    assert np.linalg.norm(Y - ref) <= 1e-5 * np.linalg.norm(ref)


@pytest.mark.parametrize("small", [False, True])
def test_largest_tile_both_contiguous_in_k(ctx, small):
    """The right factor of a two-sided adjoint with 64 slices of 500 x 509 outputs: 256 x 256 tiles, ragged both ways."""
    from oracle.cprod import Operator
    rng = np.random.default_rng(6)
    A, B = rng.standard_normal((64, 24, 500)), rng.standard_normal((64, 509, 509))
    R = f32(rng.standard_normal((64, 24, 509)))
    if small:
        A, R = A * 2.0 ** -60, f32(R * 2.0 ** -58)   # the intermediate loses bits, B brings the results back
        B = B * 2.0 ** 90
    Z, ref = product(ctx, A, B, R, 0, True), Operator(A, B).adjoint(R)
    assert np.linalg.norm(Z - ref) <= 1e-5 * np.linalg.norm(ref)


@pytest.mark.parametrize("small", [False, True])
def test_five_workgroups_per_cu(ctx, small):
    """64 slices of 270 x 250 outputs: 1280 tiles of 64 x 64, one round of 256 CUs with five each, ragged both ways; the
    product, and the right factor of a two-sided adjoint."""
    from oracle.cprod import Operator
    rng = np.random.default_rng(8)
    A, X = rng.standard_normal((64, 270, 40)), f32(rng.standard_normal((64, 40, 250)))
    if small:
        A, X = A * 2.0 ** -118, f32(X * 2.0 ** 90)
    Y, ref = product(ctx, A, None, X, 0, False), Operator(A).apply(X)
    assert np.linalg.norm(Y - ref) <= 1e-5 * np.linalg.norm(ref)
    A, B = rng.standard_normal((64, 24, 270)), rng.standard_normal((64, 250, 250))
    R = f32(rng.standard_normal((64, 24, 250)))
    if small:
        A, R, B = A * 2.0 ** -60, f32(R * 2.0 ** -58), B * 2.0 ** 90
    Z, ref = product(ctx, A, B, R, 0, True), Operator(A, B).adjoint(R)
    assert np.linalg.norm(Z - ref) <= 1e-5 * np.linalg.norm(ref)
