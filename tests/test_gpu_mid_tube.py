"""Transforms of 9 <= p <= 64 on the matrix cores in FP64, and of 9 <= p <= 15 in FP32: bare transforms, products
and solves (scaled input, epilogue with src, partial sums, paired transforms) against the oracle, at the edges of the
16-row bands and of the 64-position tiles, at counts that no vector access fits, and with more tiles than one turn
of the workgroups covers.

Bounds, u = 2^-53 or 2^-24: an element of a transform is p products and one scaling, so it is off by at most
(p + 1) u |G| |x| from G x with the library's own G, which is what its transform of the identity returns exactly;
that G is the oracle's to the condition of the transforms (below 100) times a few p u, 1e-12 and 1e-5.  A product is two transforms and K <= 40 terms between them: 1e-12 and 1e-5, relative, with the
condition of the transforms (below 100) in hand.  A solve is 5 steps of two products, and lambda = 0.05 magnifies
what they leave by at most |A| / lambda < 50: 1e-10 and 1e-4."""
import numpy as np
import pytest

from oracle import krylov
from oracle import tube as otube
from oracle.cprod import Operator
from tests.gpu_util import rel, to_gpu, to_np

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2103_11847_amd as dk  # noqa: E402

TYPES = {"f64": (dk.DCTK_F64, torch.float64, np.float64, 2.0 ** -53, 1e-12, 1e-10),
         "f32": (dk.DCTK_F32, torch.float32, np.float32, 2.0 ** -24, 1e-5, 1e-4)}
LENGTHS = [("f64", p) for p in (9, 15, 16, 17, 31, 32, 33, 48, 49, 64)] + [("f32", p) for p in (9, 12, 15)]
K, LAM = 5, 0.05


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = dk.dctk_create(0)
    yield c
    dk.dctk_destroy(c)


@pytest.mark.parametrize("count", [1, 63, 64, 66, 65 * 1024 + 4])
@pytest.mark.parametrize("dt,p", LENGTHS)
def test_transforms(ctx, dt, p, count):
    code, tt, nt, u, prod, _ = TYPES[dt]
    x = np.random.default_rng(p + count).standard_normal((p, count)).astype(nt)
    xt = to_gpu(x, tt)
    L = otube.transform_matrix(p, "th")
    Li = np.linalg.inv(L)
    for fn, adj, G in ((dk.dctk_tube_fwd, 0, L), (dk.dctk_tube_fwd, 1, Li.T), (dk.dctk_tube_inv, 0, Li),
                       (dk.dctk_tube_inv, 1, L.T)):
        out = torch.full_like(xt, float("nan"))
        fn(ctx, dk.DCTK_TUBE_TH, adj, xt, out)
        own = torch.full((p, p), float("nan"), dtype=tt, device="cuda:0")
        fn(ctx, dk.DCTK_TUBE_TH, adj, torch.eye(p, dtype=tt, device="cuda:0"), own)
        assert rel(to_np(own), G) <= prod, (fn.__name__, adj)
        own = to_np(own).astype(np.longdouble)
        bound = 2 * (p + 2) * u * (np.abs(own) @ np.abs(x))
        assert np.all(np.abs(to_np(out) - own @ x) <= bound), (fn.__name__, adj)


@pytest.mark.parametrize("n1,n2,s", [(24, 20, 20), (9, 7, 5), (40, 38, 33)])
@pytest.mark.parametrize("dt,p", LENGTHS)
def test_products_and_solves(ctx, dt, p, n1, n2, s):
    code, tt, nt, _, prod, sol = TYPES[dt]
    rng = np.random.default_rng(1000 * p + n1)
    A = rng.standard_normal((p, n1, n2)) / np.sqrt(n1 * p)
    C = rng.standard_normal((p, n1, s)).astype(nt).astype(np.float64)
    X0 = rng.standard_normal((p, n2, s)).astype(nt).astype(np.float64)
    ref = Operator(A)
    op = dk.dctk_op_create(ctx, dk.DCTK_TUBE_TH, code, to_gpu(A, torch.float64), s)
    Y = torch.full((p, n1, s), float("nan"), dtype=tt, device="cuda:0")
    X = torch.full((p, n2, s), float("nan"), dtype=tt, device="cuda:0")
    dk.dctk_cprod(ctx, op, 1.0, to_gpu(X0, tt), 0.0, Y)
    assert rel(to_np(Y), ref.apply(X0)) <= prod
    dk.dctk_cprod_T(ctx, op, 1.0, to_gpu(C, tt), 0.0, X)
    assert rel(to_np(X), ref.adjoint(C)) <= prod
    ws = dk.dctk_krylov_create(ctx, op, dk.DCTK_KRYLOV_GKB, K)
    X = torch.full((p, n2, s), float("nan"), dtype=tt, device="cuda:0")
    dk.dctk_lsqr_tik_solve(ctx, ws, to_gpu(C, tt), X, dk.make_opts(K, lam=LAM))
    assert rel(to_np(X), krylov.dc_gk(ref, C, K, lam=LAM)["X"]) <= sol
    dk.dctk_krylov_destroy(ws)
    dk.dctk_op_destroy(op)
