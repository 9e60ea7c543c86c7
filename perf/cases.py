"""The work that programs built on this library have it do, as timed cases.

Each case is a plain dict: a family (`"path"`), sizes, kernel and options.
`listed()` names twelve of them, `draw(rng)` makes more of the same ranges,
`prepare` builds what a program holds before the call (points, right-hand
sides, solutions), `run` makes one pass through the public binding, `work`
counts what the pass cannot do without and `exact` computes its result in
float64 with torch alone.
"""

import math

import numpy as np
import torch

from paper_2207_06856_amd import gpmi

KINDS = {"rbf": gpmi.RBF, "matern52": gpmi.MATERN52, "matern32": gpmi.MATERN32,
         "matern12": gpmi.MATERN12}
PRECISIONS = {"fp16": gpmi.FP16, "fp32": gpmi.FP32, "bf16": gpmi.BF16}


def listed():
    return [
        # the smallest solves' product: a few hundred points, where launches count
        dict(name="product_tiny", path="product", n1=500, n2=0, d=2, r=8, kind="rbf",
             precision="fp16", ls=0.8),
        # a mid-sized batched problem's product, ragged, with many inputs
        dict(name="product_mid", path="product", n1=9999, n2=0, d=16, r=8, kind="matern52",
             precision="fp16", ls=3.0),
        # the mixed-precision solve's product: y and 15 probes on 100,000 points
        dict(name="product_100k", path="product", n1=100000, n2=0, d=8, r=16, kind="matern52",
             precision="fp16", ls=1.0),
        # the largest single-GPU problem's product
        dict(name="product_large", path="product", n1=1800000, n2=0, d=11, r=16, kind="rbf",
             precision="fp16", ls=1.5),
        # the float32 product of the reference solves, on a served problem's size
        dict(name="product_fp32", path="product", n1=40011, n2=0, d=8, r=16, kind="rbf",
             precision="fp32", ls=1.0),
        # predictive means at 100,000 test points from loaded weights
        dict(name="predict_100k", path="product", n1=100000, n2=100000, d=8, r=1, kind="rbf",
             precision="fp16", ls=1.0),
        # a product over the finite binary16 support, points on a wide square
        dict(name="truncated", path="truncated", n=400000, d=2, r=16, kind="rbf", half_width=10.0),
        # a plain float32 solve to a tight tolerance on a small data set
        dict(name="solve_small", path="solve", n=2000, d=3, r=1, kind="rbf", precision="fp32",
             ls=0.5, noise=0.1, tol=1e-4, rank=0, max_iter=400, points="box"),
        # one training step's solve at the training start: preconditioner and CG on [y, probes]
        dict(name="solve_train", path="solve", n=100000, d=8, r=16, kind="rbf", precision="fp16",
             ls=0.6931472, noise=2.0, tol=1.0, rank=100, max_iter=50, points="normal"),
        # the same step's gradient with one lengthscale per input
        dict(name="grad_100k", path="grad", n=100000, d=8, r=16, kind="rbf", ard=True),
        # a preconditioner of a mid-sized data set and one application of it
        dict(name="precond", path="precond", n=50021, d=11, rank=100, r=16, kind="matern52",
             ls=1.5, noise=0.05),
        # many small data sets fitted side by side
        dict(name="batched", path="batched", problems=48, n_lo=500, n_hi=20000, d_lo=2, d_hi=16,
             r=8, kind="rbf", rank=20, sizes=1),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["product"] * 6 + ["truncated", "solve", "solve", "grad", "precond",
                                         "batched"])
    kind = rng.choice(["rbf", "rbf", "matern52", "matern52", "matern32", "matern12"])
    if path == "product":
        precision = rng.choice(["fp16", "fp16", "fp16", "fp32", "fp32", "bf16"])
        n1 = _log_int(rng, 300, 60000 if precision == "fp32" else 400000)
        n2 = rng.choice([0, 0, _log_int(rng, 300, 100000)])
        d = rng.randint(1, 16)
        return dict(path=path, n1=n1, n2=n2, d=d, r=rng.choice([1, 8, 16, rng.randint(1, 32)]),
                    kind=kind, precision=precision, ls=round(0.5 * math.sqrt(d), 4))
    if path == "truncated":
        return dict(path=path, n=_log_int(rng, 20000, 500000), d=rng.randint(1, 3),
                    r=rng.choice([1, 8, 16]), kind="rbf",
                    half_width=round(rng.uniform(6.0, 15.0), 3))
    if path == "solve":
        if rng.random() < 0.5:
            return dict(path=path, n=_log_int(rng, 500, 6000), d=rng.randint(2, 6),
                        r=rng.randint(1, 8), kind=kind, precision="fp32", ls=0.5, noise=0.1,
                        tol=1e-4, rank=0, max_iter=400, points="box")
        return dict(path=path, n=_log_int(rng, 2000, 150000), d=rng.randint(2, 12),
                    r=rng.choice([8, 16, rng.randint(2, 16)]), kind=kind, precision="fp16",
                    ls=0.6931472, noise=round(rng.uniform(1.0, 2.0), 3), tol=1.0,
                    rank=rng.choice([0, 20, 100]), max_iter=50, points="normal")
    if path == "grad":
        return dict(path=path, n=_log_int(rng, 1000, 100000), d=rng.randint(2, 16),
                    r=rng.choice([8, 16]), kind=kind, ard=rng.random() < 0.7)
    if path == "precond":
        return dict(path=path, n=_log_int(rng, 1000, 200000), d=rng.randint(2, 12),
                    rank=rng.choice([10, 50, 100, rng.randint(5, 128)]), r=rng.choice([1, 8, 16]),
                    kind=kind, ls=1.5, noise=0.05)
    return dict(path=path, problems=rng.randint(4, 48), n_lo=500,
                n_hi=_log_int(rng, 2000, 20000), d_lo=2, d_hi=16, r=rng.choice([1, 8]), kind=kind,
                rank=rng.choice([0, 20]), sizes=rng.randint(2, 1000000))


# ------------------------------------------------------------------ inputs
def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _points(n, d, g, how="normal", half_width=1.0):
    if how == "normal":
        return torch.randn((n, d), device="cuda", generator=g)
    return (torch.rand((n, d), device="cuda", generator=g) * 2 - 1) * half_width


def _signs(n, m, g):
    return torch.randint(0, 2, (n, m), device="cuda", generator=g).float() * 2 - 1


def _targets(X, g):
    n, d = X.shape
    return torch.sin(2 * X).sum(1) / math.sqrt(d) + 0.1 * torch.randn(n, device="cuda", generator=g)


def _rhs(X, r, g):
    """[y, r - 1 Rademacher probes]"""
    return torch.cat([_targets(X, g)[:, None], _signs(X.shape[0], r - 1, g)], 1).contiguous()


def _batch_sizes(case):
    g = np.random.Generator(np.random.PCG64(case["sizes"]))
    lo, hi = math.log(case["n_lo"]), math.log(case["n_hi"])
    return [(int(round(math.exp(g.uniform(lo, hi)))), int(g.integers(case["d_lo"], case["d_hi"] + 1)),
             float(np.float32(math.exp(g.uniform(math.log(0.5), math.log(3.0))))),
             float(np.float32(g.uniform(0.5, 2.0)))) for _ in range(case["problems"])]


def _lengthscales(case):
    """The gradient's hyperparameters: relevance falls with the input's index."""
    d = case["d"]
    if not case["ard"]:
        return [round(0.5 * math.sqrt(d), 4)]
    return [round(0.5 * math.sqrt(d) * (1 + j / d), 4) for j in range(d)]


def prepare(case, seed):
    g = _generator(seed)
    path, s = case["path"], dict(case=case)
    if path == "product":
        X1 = _points(case["n1"], case["d"], g)
        X2 = _points(case["n2"], case["d"], g) if case["n2"] else X1
        r = case["r"]
        V = torch.randn((X2.shape[0], r), device="cuda", generator=g)
        if r > 1:                      # a residual's column beside probes
            V[:, 1:] = _signs(X2.shape[0], r - 1, g)
        s.update(X1=X1, X2=X2, V=V, noise=0.0 if case["n2"] else 0.05)
    elif path == "truncated":
        X = _points(case["n"], case["d"], g, "box", case["half_width"])
        s.update(X=X, V=_rhs(X, case["r"], g))
    elif path == "solve":
        X = _points(case["n"], case["d"], g, case["points"])
        s.update(X=X, B=_rhs(X, case["r"], g))
    elif path == "grad":
        X = _points(case["n"], case["d"], g)
        B = _rhs(X, case["r"], g)
        # solutions of the size and correlation with B that a solve at noise 0.5 leaves
        U = (B * 1.2 + 0.4 * torch.randn(B.shape, device="cuda", generator=g)).contiguous()
        s.update(X=X, B=B, U=U)
    elif path == "precond":
        X = _points(case["n"], case["d"], g)
        s.update(X=X, R=torch.randn((case["n"], case["r"]), device="cuda", generator=g))
    else:
        probs = []
        for n, d, ls, noise in _batch_sizes(case):
            X = _points(n, d, g)
            probs.append(dict(X=X, B=_rhs(X, case["r"], g), kind=KINDS[case["kind"]],
                              lengthscale=ls * math.sqrt(d) / 2, outputscale=1.0, noise=noise,
                              precond_rank=case["rank"]))
        s.update(problems=probs)
    return s


# ------------------------------------------------------------------ one pass
def run(state):
    c = state["case"]
    path = c["path"]
    if path == "product":
        return gpmi.kmvm(state["X1"], state["X2"], state["V"], KINDS[c["kind"]], [c["ls"]], 1.0,
                         state["noise"], add_noise=not c["n2"], precision=PRECISIONS[c["precision"]])
    if path == "truncated":
        return gpmi.kmvm_truncated(state["X"], state["X"], state["V"], KINDS[c["kind"]], [1.0], 1.0,
                                   0.05, add_noise=True)
    if path == "solve":
        kern = (KINDS[c["kind"]], [c["ls"]], 1.0, c["noise"])
        P = gpmi.Precond(state["X"], *kern, rank=c["rank"]) if c["rank"] else None
        U, st = gpmi.cg_solve(state["X"], state["B"], *kern, tol=c["tol"], max_iter=c["max_iter"],
                              precision=PRECISIONS[c["precision"]], precond=P)
        if P is not None:
            P.close()
        return U, st["converged"]
    if path == "grad":
        grad = gpmi.mll_grad(state["X"], state["B"], state["U"], KINDS[c["kind"]], _lengthscales(c),
                             1.0, 0.5)
        return grad.tolist()
    if path == "precond":
        P = gpmi.Precond(state["X"], KINDS[c["kind"]], [c["ls"]], 1.0, c["noise"], rank=c["rank"])
        out = dict(z=P.apply(state["R"]), pivots=P.pivots, trace=float(P.trace_residual))
        P.close()
        return out
    Us, _ = gpmi.cg_solve_batched(state["problems"])
    return Us


# ------------------------------------------------------------------ compulsory work
def _product_work(n1, n2, d, r, same):
    pairs = n1 * (n2 + 1) / 2 if same else n1 * n2
    points = n1 if same else n1 + n2
    # distance (2 d) and kernel value (1) per unique pair, 2 r per entry
    return dict(bytes=4.0 * (points * d + n2 * r + n1 * r),
                flops=float(pairs * (2 * d + 1) + 2.0 * n1 * n2 * r))


def _precond_work(n, d, rank, r):
    return dict(bytes=4.0 * n * d + 8.0 * n * rank + 8.0 * n * r,
                flops=float(n * rank * (2 * d + rank + rank + 4 * r)))


def work(case):
    path = case["path"]
    if path == "product":
        n2 = case["n2"] or case["n1"]
        return _product_work(case["n1"], n2, case["d"], case["r"], not case["n2"])
    if path == "truncated":
        # share of a box's pairs within the support radius 5.89 (edges left out)
        n, d, r = case["n"], case["d"], case["r"]
        ball = [2 * 5.89, math.pi * 5.89 ** 2, 4 / 3 * math.pi * 5.89 ** 3][d - 1]
        share = min(1.0, 0.8 * ball / (2 * case["half_width"]) ** d)
        w = _product_work(n, n, d, r, True)
        return dict(bytes=w["bytes"], flops=w["flops"] * share)
    if path == "solve":
        n, d, r = case["n"], case["d"], case["r"]
        w = _product_work(n, n, d, r, True)
        p = _precond_work(n, d, case["rank"], 10 * r)
        # ten iterations at least and the true residual at exit
        return dict(bytes=11 * w["bytes"] + p["bytes"], flops=11 * w["flops"] + p["flops"])
    if path == "grad":
        n, d, r = case["n"], case["d"], case["r"]
        per = 2 * d + 2 * r + 4 + (3 * d if case["ard"] else 2)
        return dict(bytes=4.0 * n * (d + 2 * r), flops=n * (n + 1) / 2.0 * per)
    if path == "precond":
        return _precond_work(case["n"], case["d"], case["rank"], case["r"])
    total = dict(bytes=0.0, flops=0.0)
    for n, d, _, _ in _batch_sizes(case):
        w = _product_work(n, n, d, case["r"], True)
        p = _precond_work(n, d, min(n, case["rank"]), 10 * case["r"])
        total["bytes"] += 11 * w["bytes"] + p["bytes"]
        total["flops"] += 11 * w["flops"] + p["flops"]
    return total


# ------------------------------------------------------------------ float64 values
def _sqdist(A, B):
    return torch.addmm(A.square().sum(1)[:, None] + B.square().sum(1)[None, :], A, B.t(),
                       alpha=-2.0).clamp_(min=0.0)


def _kernel(kind, q):
    """Kernel values from squared scaled distances."""
    if kind == "rbf":
        return torch.exp(-0.5 * q)
    t = q.sqrt()
    if kind == "matern12":
        return torch.exp(-t)
    if kind == "matern32":
        t = math.sqrt(3.0) * t
        return (1 + t) * torch.exp(-t)
    t = math.sqrt(5.0) * t
    return (1 + t + t * t / 3) * torch.exp(-t)


def _scaled(X, ls):
    return X.double() / torch.tensor(np.asarray(ls, np.float32).astype(np.float64), device=X.device)


def _chunks(n1, n2):
    step = max(1, min(n1, 200_000_000 // max(n2, 1)))
    return [(i, min(n1, i + step)) for i in range(0, n1, step)]


def _exact_product(kind, X1, X2, V, ls, noise):
    A, B, W = _scaled(X1, ls), _scaled(X2, ls), V.double()
    out = torch.empty((A.shape[0], W.shape[1]), device=A.device, dtype=torch.float64)
    for i, j in _chunks(A.shape[0], B.shape[0]):
        out[i:j] = _kernel(kind, _sqdist(A[i:j], B)) @ W
    return out + float(np.float32(noise)) * W if noise else out


def _slope(kind, q):
    """-2 dk/dq, the factor in dk/dl_m = slope (x_m - x'_m)^2 / l_m^3."""
    if kind == "rbf":
        return torch.exp(-0.5 * q)
    t = q.sqrt()
    if kind == "matern12":
        return torch.where(t > 0, torch.exp(-t) / t.clamp(min=1e-300), torch.zeros_like(t))
    if kind == "matern32":
        return 3.0 * torch.exp(-math.sqrt(3.0) * t)
    t = math.sqrt(5.0) * t
    return (5.0 / 3.0) * (1 + t) * torch.exp(-t)


def _exact_grad(case, s):
    ls = np.asarray(_lengthscales(case), np.float32).astype(np.float64)
    X, B, U = s["X"].double(), s["B"].double(), s["U"].double()
    m = case["r"] - 1
    C = torch.cat([-0.5 * U[:, :1], B[:, 1:] / (2.0 * m)], 1)
    A = _scaled(s["X"], ls)
    n, d = A.shape
    dl = torch.zeros(d, device=A.device, dtype=torch.float64)
    da = torch.zeros((), device=A.device, dtype=torch.float64)
    A2 = A.square()
    for i, j in _chunks(n, n):
        q = _sqdist(A[i:j], A)
        q[torch.arange(j - i, device=A.device), torch.arange(i, j, device=A.device)] = 0.0
        W = U[i:j] @ C.t()
        da += (_kernel(case["kind"], q) * W).sum()
        H = _slope(case["kind"], q).mul_(W)
        dl += (A2[i:j] * H.sum(1)[:, None]).sum(0) + (A2 * H.sum(0)[:, None]).sum(0)
        dl -= 2.0 * (A[i:j] * (H @ A)).sum(0)
    dl = dl.cpu().numpy()
    dl = (dl / ls) if case["ard"] else np.array([dl.sum() / ls[0]])
    ds = (U * C).sum().item()
    fit = 0.5 * (B[:, 0] * U[:, 0]).sum().item()
    return [float(v) for v in dl] + [da.item(), ds, fit]


def _exact_precond(case, s):
    A = _scaled(s["X"], [case["ls"]])
    n, k = A.shape[0], case["rank"]
    s2 = float(np.float32(case["noise"]))
    L = torch.zeros((n, k), device=A.device, dtype=torch.float64)
    diag = torch.ones(n, device=A.device, dtype=torch.float64)
    pivots = []
    for m in range(k):
        p = int(torch.argmax(diag)) if m else 0
        pivots.append(p)
        q = (A - A[p]).square().sum(1)
        col = _kernel(case["kind"], q) - L[:, :m] @ L[p, :m]
        col = col / torch.sqrt(diag[p])
        L[:, m] = col
        diag = diag - col * col
        diag[p] = 0.0
    R = s["R"].double()
    inner = torch.eye(k, device=A.device, dtype=torch.float64) + L.t() @ L / s2
    z = R / s2 - L @ torch.linalg.solve(inner, L.t() @ R) / (s2 * s2)
    return dict(z=z, pivots=np.array(pivots, dtype=np.int64), trace=float(diag.clamp(min=0).sum()))


def exact(case, seed):
    path = case["path"]
    if path == "product":
        if float(case["n1"]) * (case["n2"] or case["n1"]) > 4e10:
            return None
        s = prepare(case, seed)
        return _exact_product(case["kind"], s["X1"], s["X2"], s["V"], [case["ls"]], s["noise"])
    if path == "truncated":
        if float(case["n"]) ** 2 > 4e10:
            return None
        s = prepare(case, seed)
        return _exact_product(case["kind"], s["X"], s["X"], s["V"], [1.0], 0.05)
    if path == "solve":
        # a solve to tol 1.0 is not near the solution; one to 1e-4 is
        if case["tol"] > 0.01:
            return None
        s = prepare(case, seed)
        A = _scaled(s["X"], [case["ls"]])
        K = _kernel(case["kind"], _sqdist(A, A))
        K.diagonal().fill_(1.0 + float(np.float32(case["noise"])))
        return torch.cholesky_solve(s["B"].double(), torch.linalg.cholesky(K)), None
    if path == "grad":
        return _exact_grad(case, prepare(case, seed))
    if path == "precond":
        return _exact_precond(case, prepare(case, seed))
    return None
