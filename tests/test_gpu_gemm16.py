"""16-bit slice products of any size: every tile (32, 64, 128 and 256 rows) on sizes that leave partial 8-element
units, partial chunks of 64 k and partial tiles, one-sided and two-sided (both orientations of the right operand), down
to fewer than 8 columns or terms.

Every tile adds a sum's terms in the same order with the same instruction, so the tiles agree bit for bit.  Against the
oracle the operands' and (two-sided) the intermediate's rounding to 16 bits counts: unit roundoff u = 2^-11 (FP16) or
2^-8 (BF16), two or four independent roundings per term, so at most 4 u relative in the 2-norm with the condition of
the transforms (below 9 for p <= 17) in hand: 36 u."""
import numpy as np
import pytest

from oracle.cprod import Operator
from tests.gpu_util import rel, to_gpu, to_np

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2103_11847_amd as dk  # noqa: E402

U = {"f16": (dk.DCTK_F16, 2.0 ** -11), "bf16": (dk.DCTK_BF16, 2.0 ** -8)}
SIZES = [(9, 8, 8), (33, 9, 15), (64, 64, 64), (65, 63, 66), (31, 129, 70), (70, 257, 33), (130, 330, 129),
         (260, 127, 262), (5, 3, 9), (20, 40, 5), (40, 7, 8)]


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = dk.dctk_create(0)
    yield c
    dk.dctk_synchronize(c)
    dk.dctk_destroy(c)


@pytest.mark.parametrize("two", [False, True])
@pytest.mark.parametrize("n1,n2,s", SIZES)
@pytest.mark.parametrize("dt,p", [("f16", 9), ("bf16", 5), ("bf16", 17)])
def test_tiles_agree(ctx, dt, p, n1, n2, s, two):
    code, u = U[dt]
    rng = np.random.default_rng(1000 * p + n1 + n2)
    A = rng.standard_normal((p, n1, n2)) / np.sqrt(n2 * p)
    B = rng.standard_normal((p, s, s)) / np.sqrt(s * p) if two else None
    X0 = rng.standard_normal((p, n2, s)).astype(np.float32)
    Y0 = rng.standard_normal((p, n1, s)).astype(np.float32)
    ref = Operator(A, B) if two else Operator(A)
    op = dk.dctk_op_create(ctx, dk.DCTK_TUBE_TH, code, to_gpu(A, torch.float64), s,
                           to_gpu(B, torch.float64) if two else None)
    first = None
    for tile in (32, 64, 128, 256):
        for adj in (0, 1):
            dk.dctk_op_set_path(op, adj, 0, tile)
        Y = torch.full((p, n1, s), float("nan"), device="cuda:0")
        X = torch.full((p, n2, s), float("nan"), device="cuda:0")
        dk.dctk_cprod(ctx, op, 1.0, to_gpu(X0, torch.float32), 0.0, Y)
        dk.dctk_cprod_T(ctx, op, 1.0, to_gpu(Y0, torch.float32), 0.0, X)
        dk.dctk_synchronize(ctx)
        if first is None:
            first = (Y, X)
            assert rel(to_np(Y), ref.apply(X0.astype(np.float64))) <= 36 * u
            assert rel(to_np(X), ref.adjoint(Y0.astype(np.float64))) <= 36 * u
        assert torch.equal(Y, first[0]) and torch.equal(X, first[1]), tile
    dk.dctk_op_destroy(op)
