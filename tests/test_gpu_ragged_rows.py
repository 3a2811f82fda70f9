"""Tube transforms of p <= 64 on slices of every size modulo 4 and at addresses that are no multiple of 16: 4-position
vectors need no alignment, and the one that would cross a slice's end is read early and put right.

The reference is the library's own G (its transform of the identity, exact) in extended precision: p products and a
scaling, at most 2 (p + 2) u |G| |x| per element, u = 2^-53 or 2^-24.  The positions around the output must keep what
they held.  Two-sided products and solves on odd slices (src, partial sums, paired transforms, 16-bit outputs) are
checked by moving every buffer to an odd address: the sums are the same ones in the same order, so bit for bit."""
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
    dk.dctk_synchronize(c)
    dk.dctk_destroy(c)


def at(x, off):
    """x on the GPU in a buffer that starts `off` elements behind an aligned one, 7 behind it."""
    buf = torch.full((off + x.numel() + 8,), 7.0, dtype=x.dtype, device="cuda:0")
    v = buf[off:off + x.numel()].view(x.shape)
    v.copy_(x)
    return buf, v


@pytest.mark.parametrize("dt", [torch.float32, torch.float64])
@pytest.mark.parametrize("p", [1, 3, 4, 5, 8, 9, 16, 31, 64])
def test_sizes_and_addresses(ctx, dt, p):
    u = 2.0 ** -24 if dt == torch.float32 else 2.0 ** -53
    rng = np.random.default_rng(p)
    for count in (1, 3, 4, 5, 6, 7, 63, 64, 65, 66, 67, 257, 1025, 1031):
        x = to_gpu(rng.standard_normal((p, count)), dt)
        for fn, adj in ((dk.dctk_tube_fwd, 0), (dk.dctk_tube_fwd, 1), (dk.dctk_tube_inv, 0), (dk.dctk_tube_inv, 1)):
            own = torch.empty((p, p), dtype=dt, device="cuda:0")
            fn(ctx, dk.DCTK_TUBE_TH, adj, torch.eye(p, dtype=dt, device="cuda:0"), own)
            G = to_np(own).astype(np.longdouble)
            bound = 2 * (p + 2) * u * (np.abs(G) @ np.abs(to_np(x)))
            for off in (0, 1, 3):
                _, xi = at(x, off)
                buf, out = at(torch.full_like(x, float("nan")), off)
                fn(ctx, dk.DCTK_TUBE_TH, adj, xi, out)
                dk.dctk_synchronize(ctx)
                assert np.all(np.abs(to_np(out) - G @ to_np(x)) <= bound), (count, fn.__name__, adj, off)
                assert bool((buf[:off] == 7).all()) and bool((buf[off + x.numel():] == 7).all())


@pytest.mark.parametrize("gdt", [dk.DCTK_F64, dk.DCTK_F32, dk.DCTK_BF16, dk.DCTK_F16])
@pytest.mark.parametrize("p,n1,n2,s", [(3, 9, 7, 5), (8, 7, 7, 7), (12, 5, 9, 9), (31, 11, 9, 7), (64, 5, 13, 5)])
def test_products_and_solves_at_odd_addresses(ctx, gdt, p, n1, n2, s):
    vt = torch.float64 if gdt == dk.DCTK_F64 else torch.float32
    rng = np.random.default_rng(p + n1)
    A = to_gpu(rng.standard_normal((p, n1, n2)) / np.sqrt(n1 * p), torch.float64)
    B = to_gpu(rng.standard_normal((p, s, s)) / np.sqrt(s * p), torch.float64)
    X0 = to_gpu(rng.standard_normal((p, n2, s)), vt)
    C0 = to_gpu(rng.standard_normal((p, n1, s)), vt)
    op = dk.dctk_op_create(ctx, dk.DCTK_TUBE_TH, gdt, A, s, B)
    ws = dk.dctk_krylov_create(ctx, op, dk.DCTK_KRYLOV_GKB, 3)
    seen = []
    for off in (0, 1):
        (_, X), (_, C) = at(X0, off), at(C0, off)
        yb, Y = at(C0, off)
        xb, S = at(torch.zeros_like(X0), off)
        dk.dctk_cprod(ctx, op, -0.5, X, 2.0, Y)
        dk.dctk_lsqr_tik_solve(ctx, ws, C, S, dk.make_opts(3, lam=0.05))
        dk.dctk_synchronize(ctx)
        for buf, n in ((yb, Y.numel()), (xb, S.numel())):
            assert bool((buf[:off] == 7).all()) and bool((buf[off + n:] == 7).all())
        seen.append((Y.clone(), S.clone()))
    assert all(torch.equal(a, b) and bool(torch.isfinite(a).all()) for a, b in zip(*seen))
    dk.dctk_krylov_destroy(ws)
    dk.dctk_op_destroy(op)
