"""The workloads that this library's speed is judged by, from the smallest product to a whole solve.

Every case goes through the public entry points of `paper_2103_11847_amd`.  The sizes are those of the
repository's workloads and tests: the small parity problem, the 256 x 256 colour image, the 1024 x 1024 colour
image of the paper, 32 frames of video, the 512 x 512 cube of 64 bands, tubes of 256 bands, the uneven batch.

  product    Y = M(X) and X = M*(Y): one forward product and one adjoint product of a prepared operator
             (the two directions of every Golub-Kahan and Arnoldi step);
  transform  the tube transform forward and back, as a program calls it by itself;
  gk         a DC-GK restoration (Golub-Kahan steps, lambda by GCV, X = V y);
  gmres      a DC-GMRES restoration (one Arnoldi cycle, lambda by GCV);
  batch      a planned batch of uneven DC-GK restorations, run as one graph.
"""
import math

import numpy as np
import torch

import paper_2103_11847_amd as dk

GEMM = {"f64": dk.DCTK_F64, "f32": dk.DCTK_F32, "bf16": dk.DCTK_BF16, "f16": dk.DCTK_F16}
SIZE = {"f64": 8, "f32": 4, "bf16": 2, "f16": 2}
COLOUR = (0.7, 0.15, 0.15)


def listed():
    return [
        # the smallest call: the 32 x 32 colour problem in FP64 (launches and host time count)
        product("product_small_f64", "f64", 3, 32, 32, 32),
        # one colour image, the ordinary interactive size (one fused kernel per product)
        product("product_colour_f32", "f32", 3, 256, 256, 256),
        # the paper's large colour image, blurred along rows and columns
        product("product_paper1024_f32", "f32", 3, 1024, 1024, 1024, two=True),
        # 32 frames of video, blurred within and across frames, 16-bit slice products
        product("product_video_f16", "f16", 32, 256, 256, 256, two=True),
        # a cropped cube: odd and rectangular slices, a tube length that is no power of two
        product("product_ragged_f32", "f32", 31, 243, 211, 197),
        # the hyperspectral cube, the library's default workload, in its two product types
        product("product_hyper_f32", "f32", 64, 512, 512, 512),
        product("product_hyper_bf16", "bf16", 64, 512, 512, 512),
        # 256 bands of a 512 x 512 scene, transformed along the tubes and back
        {"name": "transform_long_f32", "kind": "transform", "type": "f32", "p": 256, "rows": 512, "cols": 512},
        # a colour image restored, latency-bound
        solve("gk_colour_f32", "gk", "f32", 3, 256, 40),
        # a hyperspectral cube restored: the library's default solve
        solve("gk_hyper_f32", "gk", "f32", 64, 512, 40),
        # a video restored by DC-GMRES, two-sided, modified Gram-Schmidt
        solve("gmres_video_f32", "gmres", "f32", 32, 256, 40, two=True),
        # a queue of small uneven restorations
        {"name": "batch_uneven_f32", "kind": "batch", "type": "f32", "count": 16, "n_min": 64, "n_max": 256, "k": 10},
    ]


def product(name, dtype, p, n1, n2, s, two=False):
    c = {"kind": "product", "type": dtype, "p": p, "n1": n1, "n2": n2, "s": s, "two": two}
    return dict(c, name=name) if name else c


def solve(name, kind, dtype, p, n, k, two=False):
    c = {"kind": kind, "type": dtype, "p": p, "n": n, "k": k, "two": two}
    return dict(c, name=name) if name else c


def spread(rng, lo, hi):
    """A whole number in [lo, hi], even over its logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["product"] * 5 + ["transform", "gk", "gk", "gmres", "batch"])
    if kind == "product":
        while True:
            dtype = rng.choice(["f64", "f32", "f32", "f32", "bf16", "f16"])
            p = rng.choice([3, 8, 16, 31, 32, 64, 128, spread(rng, 2, 64)])
            n1 = spread(rng, 32, 640)
            shape = rng.choice(["square", "even", "any"])
            if shape != "any":
                n1 = max(32, n1 // 32 * 32 if shape == "square" else n1 // 2 * 2)
            n2, s = (n1, n1) if shape != "any" else (spread(rng, 32, 640), spread(rng, 32, 640))
            two = rng.random() < 0.3
            c = product("", dtype, p, n1, n2, s, two)
            if work(c)["flops"] * (2 if dtype == "f64" else 1) <= 8e10:
                return c
    if kind == "transform":
        p = rng.choice([16, 31, 64, 128, 256, 512, 1024, spread(rng, 3, 64)])
        most = max(64, min(512, int(math.sqrt(6.7e7 / p))))
        return {"kind": "transform", "type": rng.choice(["f32", "f32", "f64"]), "p": p,
                "rows": spread(rng, 32, most), "cols": spread(rng, 32, most)}
    if kind == "gk":
        p = rng.choice([3, 8, 31, 64, spread(rng, 3, 64)])
        return solve("", "gk", rng.choice(["f32", "f32", "f64"]), p, spread(rng, 64, 384 if p <= 32 else 256),
                     rng.randint(5, 10))
    if kind == "gmres":
        p = rng.choice([3, 16, 32, spread(rng, 3, 32)])
        return solve("", "gmres", rng.choice(["f32", "f64"]), p, spread(rng, 64, 256), rng.randint(6, 12),
                     two=rng.random() < 0.5)
    lo = spread(rng, 48, 128)
    return {"kind": "batch", "type": "f32", "count": rng.randint(4, 24), "n_min": lo,
            "n_max": lo + spread(rng, 32, 160), "k": rng.randint(6, 10)}


# ---- inputs --------------------------------------------------------------------------------------------------
def blur(n1, n2, sigma):
    """Banded Gaussian blur of n2 samples seen by n1 detectors."""
    r = int(math.ceil(2.5 * sigma))
    at = torch.arange(n1, device="cuda", dtype=torch.float64)[:, None] * (n2 / n1)
    d = at - torch.arange(n2, device="cuda", dtype=torch.float64)[None, :]
    t = torch.exp(-d * d / (2 * sigma * sigma)) / (sigma * math.sqrt(2 * math.pi))
    return torch.where(d.abs() <= r, t, torch.zeros_like(t))


def operator(rng, p, n1, n2, s, two):
    """A (p, n1, n2), and B (p, s, s) of a two-sided operator, in FP64: a blur mixed over three colours or a few
    frames, or one that widens and fades over the bands of a longer tube."""
    sigma = rng.uniform(1.5, 3.0)
    if p <= 8 or two:
        tube = COLOUR if p == 3 else (0.5, 0.25) + (0.0,) * max(0, p - 2)
        A = torch.stack([c * blur(n1, n2, sigma) for c in tube[:p]])
    else:
        A = torch.stack([0.005 ** (k / (p - 1)) * blur(n1, n2, sigma + 2.0 * k / (p - 1)) for k in range(p)])
    if not two:
        return A.contiguous(), None
    tube = (1.0,) + (0.0,) * (p - 1) if p == 3 else (0.5, 0.25) + (0.0,) * max(0, p - 2)
    B = torch.stack([c * blur(s, s, rng.uniform(1.0, 2.0)).t() for c in tube[:p]])
    return A.contiguous(), B.contiguous()


def scene(rng, p, n, s):
    """Gaussian blobs with smooth profiles along the tube, in [0, 1]."""
    i = torch.arange(n, device="cuda", dtype=torch.float64)
    j = torch.arange(s, device="cuda", dtype=torch.float64)
    t = torch.arange(p, device="cuda", dtype=torch.float64) / max(1, p - 1)
    X = torch.zeros((p, n, s), device="cuda", dtype=torch.float64)
    for _ in range(8):
        ci, cj, w = rng.uniform(0, n), rng.uniform(0, s), rng.uniform(max(n, s) / 16, max(n, s) / 4)
        at, wide, high = rng.uniform(0, 1), rng.uniform(0.15, 0.6), rng.uniform(0.2, 1.0)
        spot = torch.exp(-((i[:, None] - ci) ** 2 + (j[None, :] - cj) ** 2) / (2 * w * w))
        X += (high * torch.exp(-((t - at) ** 2) / (2 * wide * wide)))[:, None, None] * spot[None]
    return (X - X.min()) / (X.max() - X.min())


def instances(case):
    """(p, n) of a batch's restorations: n spread evenly from n_min to n_max, tubes of 3, 8 and 31 in turn."""
    lo, hi, c = case["n_min"], case["n_max"], case["count"]
    return [((3, 8, 31)[i % 3], lo + (hi - lo) * i // max(1, c - 1)) for i in range(c)]


def vec(dtype):
    return torch.float64 if dtype == "f64" else torch.float32


def problem(case, seed):
    """{A, B, X} of a product, {x, y} of a transform, {A, B, C} of a restoration, a list of those of a batch."""
    rng = np.random.default_rng(seed)
    g = torch.Generator(device="cuda").manual_seed(int(rng.integers(1 << 31)))

    def noise(*shape):
        return torch.randn(shape, generator=g, device="cuda", dtype=torch.float64)

    v = vec(case["type"])
    kind = case["kind"]
    if kind == "product":
        p, n1, n2, s = case["p"], case["n1"], case["n2"], case["s"]
        A, B = operator(rng, p, n1, n2, s, case["two"])
        X = scene(rng, p, n2, s)
        # what the adjoint product of a step is given: a residual, noise-like
        R = scene(rng, p, n1, s) * 0.1 + 0.01 * noise(p, n1, s)
        return {"A": A, "B": B, "X": (X + 0.01 * noise(p, n2, s)).to(v), "R": R.to(v)}
    if kind == "transform":
        shape = (case["p"], case["rows"], case["cols"])
        return {"x": (scene(rng, *shape) + 0.01 * noise(*shape)).to(v), "y": noise(*shape).to(v)}

    def restoration(p, n, two):
        A, B = operator(rng, p, n, n, n, two)
        C = apply(tubes(p), A, B, scene(rng, p, n, n))
        N = noise(p, n, n)
        nu = math.exp(rng.uniform(math.log(2e-3), math.log(2e-2)))
        return {"A": A, "B": B, "C": (C + nu * float(C.norm() / N.norm()) * N).to(v)}

    if kind == "batch":
        return [restoration(p, n, False) for p, n in instances(case)]
    return restoration(case["p"], case["n"], case["two"])


class State:
    """What a program holds: a context, operators and workspaces of it, and its buffers."""

    def __init__(self):
        self.ctx = dk.dctk_create(0)
        self.undo = []

    def operator(self, dtype, A, s, B):
        op = dk.dctk_op_create(self.ctx, dk.DCTK_TUBE_TH, GEMM[dtype], A, s, B)
        self.undo.append(lambda: dk.dctk_op_destroy(op))
        return op

    def workspace(self, op, kind, k):
        ws = dk.dctk_krylov_create(self.ctx, op, kind, k)
        self.undo.append(lambda: dk.dctk_krylov_destroy(ws))
        return ws

    def __del__(self):
        torch.cuda.synchronize()
        for f in reversed(self.undo):
            f()
        dk.dctk_destroy(self.ctx)


def prepare(case, seed):
    q = problem(case, seed)
    st = State()
    st.kind = case["kind"]
    if st.kind == "product":
        st.op = st.operator(case["type"], q["A"], case["s"], q["B"])
        st.X, st.R = q["X"], q["R"]
        st.Y, st.Z = torch.empty_like(st.R), torch.empty_like(st.X)
    elif st.kind == "transform":
        st.x, st.y = q["x"], q["y"]
        st.fx, st.iy = torch.empty_like(st.x), torch.empty_like(st.y)
    elif st.kind == "batch":
        st.k, st.C = case["k"], [r["C"] for r in q]
        st.X = [torch.empty_like(c) for c in st.C]
        ws = [st.workspace(st.operator("f32", r["A"], r["C"].shape[2], None), dk.DCTK_KRYLOV_GKB, st.k) for r in q]
        st.plan = dk.dctk_batch_create(st.ctx, ws, st.C, st.X, dk.make_opts(st.k))
        plan = st.plan
        st.undo.append(lambda: dk.dctk_batch_destroy(plan))
    else:
        st.C, st.X, st.k = q["C"], torch.empty_like(q["C"]), case["k"]
        op = st.operator(case["type"], q["A"], case["n"], q["B"])
        st.ws = st.workspace(op, dk.DCTK_KRYLOV_GKB if st.kind == "gk" else dk.DCTK_KRYLOV_ARNOLDI, st.k)
        st.opts = dk.make_opts(st.k)
    return st


def run(st):
    if st.kind == "product":
        dk.dctk_cprod(st.ctx, st.op, 1.0, st.X, 0.0, st.Y)
        dk.dctk_cprod_T(st.ctx, st.op, 1.0, st.R, 0.0, st.Z)
        return {"forward": st.Y, "adjoint": st.Z}
    if st.kind == "transform":
        dk.dctk_tube_fwd(st.ctx, dk.DCTK_TUBE_TH, 0, st.x, st.fx)
        dk.dctk_tube_inv(st.ctx, dk.DCTK_TUBE_TH, 0, st.y, st.iy)
        return {"forward": st.fx, "inverse": st.iy}
    if st.kind == "gk":
        # enqueued without a read-back, as a program with more work to enqueue does
        dk.dctk_lsqr_tik_solve(st.ctx, st.ws, st.C, st.X, st.opts, info=False)
        return st.X
    if st.kind == "gmres":
        st.X.zero_()
        dk.dctk_gmres_tik_solve(st.ctx, st.ws, st.C, st.X, 1, st.opts)
        return st.X
    dk.dctk_batch_run(st.ctx, st.plan)
    return st.X


# ---- what a pass cannot do without ----------------------------------------------------------------------------
def work(case):
    kind, b = case["kind"], SIZE[case["type"]]
    v = 8 if case["type"] == "f64" else 4
    if kind == "product":
        return both(product_work(case["p"], case["n1"], case["n2"], case["s"], case["two"], b, v),
                    product_work(case["p"], case["n2"], case["n1"], case["s"], case["two"], b, v))
    if kind == "transform":
        p, e = case["p"], case["p"] * case["rows"] * case["cols"]
        return {"bytes": 4 * e * v, "flops": 2 * 5 * e * max(1.0, math.log2(p))}
    if kind == "batch":
        got = {"bytes": 0.0, "flops": 0.0}
        for p, n in instances(case):
            got = both(got, solve_work("gk", p, n, case["k"], False, b, v))
        return got
    return solve_work(kind, case["p"], case["n"], case["k"], case["two"], b, v)


def both(x, y):
    return {m: x[m] + y[m] for m in x}


def product_work(p, m, n, s, two, b, v):
    """One product of an (m x n) operator: its slices, the vector in and the vector out; slice products and
    transforms (a fast one for the long tube)."""
    t = min(2.0 * p, 5 * math.log2(max(2, p)))
    return {"bytes": p * (m * n * b + (s * s * b if two else 0) + (m + n) * s * v),
            "flops": p * (2.0 * m * n * s + (2.0 * m * s * s if two else 0) + t * (m + n) * s)}


def solve_work(kind, p, n, k, two, b, v):
    """k steps: a product and (Golub-Kahan) an adjoint product each, the basis written once; for Arnoldi each
    step reads the basis so far; X = V y reads it once more."""
    step = product_work(p, n, n, n, two, b, v)
    steps = 2 * k + 1 if kind == "gk" else k
    e = p * n * n
    got = {m: w * steps for m, w in step.items()}
    got["bytes"] += v * e * (k + 2 * k if kind == "gk" else k + k * (k + 1) / 2)
    got["flops"] += 2.0 * e * (k if kind == "gk" else k + k * (k + 1))
    return got


# ---- the same in 64 bits, by plain torch and numpy ----------------------------------------------------------
def tubes(p):
    """M = W^-1 C (I + Z) of the paper's Remark 2.1 in closed form, and its inverse."""
    k = torch.arange(p, dtype=torch.float64)[:, None]
    t = torch.arange(p, dtype=torch.float64)[None, :]
    M = 2 * torch.cos(math.pi * torch.remainder(k * t, 2 * p) / p)
    M[:, 0] = 1.0
    return M.cuda(), torch.linalg.inv(M).cuda()


def along(G, X):
    return (G @ X.reshape(X.shape[0], -1)).reshape((G.shape[0],) + X.shape[1:])


def apply(MI, A, B, X):
    M, I = MI
    Y = torch.bmm(along(M, A), along(M, X))
    return along(I, Y if B is None else torch.bmm(Y, along(M, B)))


def apply_T(MI, A, B, Y):
    M, I = MI
    X = torch.bmm(along(M, A).transpose(1, 2).contiguous(), along(I.t(), Y))
    return along(M.t(), X if B is None else torch.bmm(X, along(M, B).transpose(1, 2).contiguous()))


def exact(case, seed):
    q = problem(case, seed)
    kind = case["kind"]
    if kind == "transform":
        M, I = tubes(case["p"])
        return {"forward": along(M, q["x"].double()), "inverse": along(I, q["y"].double())}
    if kind == "product":
        MI = tubes(case["p"])
        return {"forward": apply(MI, q["A"], q["B"], q["X"].double()),
                "adjoint": apply_T(MI, q["A"], q["B"], q["R"].double())}
    if kind == "batch":
        return [restored(r, "gk", case["k"]) for r in q]
    return restored(q, kind, case["k"])


def restored(q, kind, k):
    C = q["C"].double()
    MI = tubes(C.shape[0])
    basis, R = golub_kahan(MI, q["A"], q["B"], C, k) if kind == "gk" else arnoldi(MI, q["A"], q["B"], C, k)
    y = tikhonov(R, float(C.norm()))
    X = torch.zeros_like(C)
    for c, v in zip(y, basis):
        X += float(c) * v
    return X


def golub_kahan(MI, A, B, C, k):
    """Algorithm 4: the basis V_1..V_k and the lower bidiagonal (k + 1) x k matrix."""
    R = np.zeros((k + 1, k))
    U = C / C.norm()
    V = apply_T(MI, A, B, U)
    alpha = float(V.norm())
    V = V / alpha
    basis = [V]
    for j in range(k):
        R[j, j] = alpha
        U = apply(MI, A, B, V) - alpha * U
        beta = float(U.norm())
        U = U / beta
        R[j + 1, j] = beta
        V = apply_T(MI, A, B, U) - beta * V
        alpha = float(V.norm())
        V = V / alpha
        basis.append(V)
    return basis, R


def arnoldi(MI, A, B, C, k):
    """Algorithm 2: the basis V_1..V_k and the Hessenberg (k + 1) x k matrix."""
    H = np.zeros((k + 1, k))
    basis = [C / C.norm()]
    for j in range(k):
        W = apply(MI, A, B, basis[j])
        for i, v in enumerate(basis):
            H[i, j] = float((W * v).sum())
            W = W - H[i, j] * v
        H[j + 1, j] = float(W.norm())
        basis.append(W / H[j + 1, j])
    return basis, H


def tikhonov(R, beta):
    """argmin |R y - beta e1|^2 + lambda^2 |y|^2 with lambda at the minimum of the projected problem's GCV."""
    k = R.shape[1]
    P, sv, Qt = np.linalg.svd(R)
    g = beta * P[0, :]

    def gcv(lam):
        f = lam * lam / (sv * sv + lam * lam)
        return (np.sum((f * g[:k]) ** 2) + g[k] ** 2) / (1.0 + np.sum(f)) ** 2

    grid = np.logspace(math.log10(1e-8 * sv[0]), math.log10(sv[0]), 400)
    i = int(np.argmin([gcv(x) for x in grid]))
    a, b = math.log(grid[max(0, i - 1)]), math.log(grid[min(399, i + 1)])
    inv = (math.sqrt(5.0) - 1) / 2
    for _ in range(80):
        c, d = b - inv * (b - a), a + inv * (b - a)
        if gcv(math.exp(c)) < gcv(math.exp(d)):
            b = d
        else:
            a = c
    lam = math.exp(0.5 * (a + b))
    return Qt.T @ (sv * g[:k] / (sv * sv + lam * lam))
