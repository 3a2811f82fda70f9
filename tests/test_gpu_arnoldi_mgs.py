"""Arnoldi steps: FP32 modified Gram-Schmidt coefficients from the triangular system (I + L) h = r (L the strictly lower
Gram triangle of the basis), FP64 ones term by term: vector lengths that are no multiple of 4 or of a workgroup, one to
64 basis vectors (whole and partial groups of 8), both vector types, repeated cycles.

FP64: H and the basis against the oracle's term-by-term MGS, 1e-9 relative (the tolerance of the other Arnoldi
tests: the recurrence amplifies 1e-16).  FP32: the relation M(V_j) = sum_i h_ij V_i of the vectors the library
itself holds, each product and vector rounded to FP32: (8 + j) 2^-24 ||M(V_j)|| plus the product's 1e-5."""
import numpy as np
import pytest

from oracle import krylov
from oracle.cprod import Operator
from tests.gpu_util import rel, to_gpu, to_np

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


def steps(ctx, gdt, A, C, k):
    vt = torch.float64 if gdt == dk.DCTK_F64 else torch.float32
    op = dk.dctk_op_create(ctx, dk.DCTK_TUBE_TH, gdt, to_gpu(A, torch.float64), C.shape[2])
    ws = dk.dctk_krylov_create(ctx, op, dk.DCTK_KRYLOV_ARNOLDI, k)
    Cg = to_gpu(C, vt)
    out = []
    for _ in range(2):   # a second run on the same workspace starts from its own first vector
        dk.dctk_arnoldi_init(ctx, ws, Cg)
        for _ in range(k):
            dk.dctk_arnoldi_step(ctx, ws)
        r = dk.dctk_krylov_read(ctx, ws, k, dk.DCTK_KRYLOV_ARNOLDI)
        V = []
        for j in range(k):
            t = torch.empty_like(Cg)
            dk.dctk_krylov_copy(ctx, ws, 0, j, t)
            V.append(to_np(t))
        out.append((np.array(r["H"]), V, r["steps"]))
    assert np.array_equal(out[0][0], out[1][0]) and all(np.array_equal(a, b) for a, b in zip(out[0][1], out[1][1]))
    dk.dctk_krylov_destroy(ws)
    dk.dctk_op_destroy(op)
    return out[0]


def problem(p, n, s, seed):
    rng = np.random.default_rng(seed)
    return rng.standard_normal((p, n, n)) / n + np.eye(n), rng.standard_normal((p, n, s))


@pytest.mark.parametrize("p,n,s,k", [(1, 3, 1, 2), (3, 5, 7, 8), (3, 17, 9, 9), (5, 33, 31, 17), (3, 64, 64, 7)])
def test_fp64_matches_oracle(ctx, p, n, s, k):
    A, C = problem(p, n, s, 10 * n + k)
    H, V, done = steps(ctx, dk.DCTK_F64, A, C, k)
    ar = krylov.Arnoldi(Operator(A), C, k, "mgs")
    for _ in range(k):
        assert ar.step()
    assert rel(H[:k, :k], ar.hessenberg()[:k, :k]) <= 1e-9
    assert max(rel(a, b) for a, b in zip(V, ar.V)) <= 1e-9


@pytest.mark.parametrize("p,n,s,k", [(3, 19, 21, 12), (3, 64, 48, 64), (31, 96, 50, 10)])
def test_fp32_relation(ctx, p, n, s, k):
    A, C = problem(p, n, s, n + k)
    H, V, done = steps(ctx, dk.DCTK_F32, A, C, k)
    assert done >= k - 1
    op = Operator(A)
    for j in range(k - 1):
        W = op.apply(V[j])
        R = W - sum(H[i, j] * V[i] for i in range(j + 2))
        assert np.linalg.norm(R) <= ((8 + j) * 2.0 ** -24 + 1e-5) * np.linalg.norm(W)
