"""The work that a user of this library has it do, one case per entry point, direction and size class.

Inputs follow the library's own workloads: feature rows in molecules of 10 to 300 rows, each molecule around one of
64 cluster means, targets a random-feature sample of the prior plus noise, lengthscales U(0.5, 2) per feature times
``ell`` (1: the workloads as written, whose kernel matrix is nearly diagonal; larger: fitted hyperparameters, whose
kernel matrix is correlated).  ``exact`` is plain torch and numpy in 64 bits.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2109_09817_amd import autograd, gp

DEV = "cuda:0"
LOG2PI = math.log(2.0 * math.pi)


def listed():
    return [
        # One product of a small model (the exact-GP-sized workload, n = 2,048, d = 32, [y | 8 probes]): the smallest call.
        dict(name="kmm_small", op="kmm", n=2048, d=32, t=9, kind="matern52", prec="bf16x3", ell=4.0, noise=1e-2),
        # The product of every CG iteration in training at n = 262,144 ([y | 15 probes]): the largest call.
        dict(name="kmm_train", op="kmm", n=262144, d=48, t=16, kind="matern52", prec="bf16x3", ell=2.0, noise=1e-3),
        # The FP64 product of the block solver in the low-noise regime (block of 50).
        dict(name="kmm_fp64", op="kmm", n=24576, d=48, t=50, kind="matern52", prec="fp64", ell=2.0, noise=1e-5),
        # A cross product K(Z, X) V in the FP32 form, ragged sizes, RBF.
        dict(name="kmm_cross", op="kmm", n=100003, m=3001, d=21, t=33, kind="rbf", prec="fp32", ell=3.0, noise=1e-3),
        # The differentiable product: forward, and backward to the hyperparameters and to V.
        dict(name="khatv_train", op="khatv", n=50001, d=48, t=16, kind="matern52", prec="bf16x3", ell=2.0, noise=1e-3),
        # One training evaluation of a small model (30 fixed iterations, 8 probes, rank 20).
        dict(name="mll_small", op="mll", n=2048, d=32, t=8, rank=20, iters=30, tol=0.0, kind="matern52", prec="bf16x3",
             ell=1.0, noise=1e-2),
        # One training evaluation of the n = 65,536 model (15 probes, rank 100).
        dict(name="mll_train", op="mll", n=65536, d=48, t=15, rank=100, iters=100, tol=1e-6, kind="matern52",
             prec="bf16x3", ell=2.0, noise=1e-2),
        # Serving, one small molecule: mean and variance of 24 rows against the n = 262,144 model, rank-256 cache.
        dict(name="predict_small", op="predict", n=262144, m=24, kc=256, d=48, kind="matern52", prec="bf16x3", ell=2.0,
             noise=1e-3),
        # Serving under load: a full batch of queued molecules.
        dict(name="predict_batch", op="predict", n=262144, m=1200, kc=256, d=48, kind="matern52", prec="bf16x3",
             ell=2.0, noise=1e-3),
        # The exact GP on a 50-molecule subset (one step of the hyperparameter protocol).
        dict(name="exact_subset", op="exact", n=7503, d=48, kind="matern52", ell=2.0, noise=1e-3),
        # The large-rank preconditioner of the block solver.
        dict(name="nystrom_build", op="nystrom", n=32768, rank=4096, d=48, kind="matern52", ell=3.0, noise=1e-3),
        # A block solve with it: 50 right-hand sides to 1e-6 in FP64.
        dict(name="block_solve", op="bpcg", n=8192, rank=1024, t=50, iters=300, tol=1e-6, d=48, kind="matern52",
             prec="fp64", ell=4.0, noise=1e-2),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: every entry point over its range, odd sizes included."""
    op = rng.choice(["kmm", "kmm", "kmm64", "cross", "khatv", "mll", "predict", "predict", "exact", "nystrom", "bpcg"])
    kind = rng.choice(["matern52", "matern52", "rbf"])
    d = rng.choice([5, 17, 21, 32, 32, 48, 48, 48, 64])
    ell = rng.choice([1.0, 2.0, 4.0])
    c = dict(d=d, kind=kind, ell=ell, noise=1e-2)
    if op == "kmm":
        return dict(c, op="kmm", n=_log(rng, 1000, 180000), t=rng.choice([1, 9, 16, 17, 33, 50]) if rng.random() < 0.7
                    else rng.randint(1, 64), prec=rng.choice(["bf16x3", "bf16x3", "bf16x3", "fp32"]))
    if op == "kmm64":
        return dict(c, op="kmm", n=_log(rng, 1000, 24000), t=rng.choice([1, 16, 50, 50]), prec="fp64", noise=1e-5)
    if op == "cross":
        return dict(c, op="kmm", n=_log(rng, 2000, 100000), m=_log(rng, 20, 4000), t=rng.randint(1, 40),
                    prec=rng.choice(["bf16x3", "fp32", "fp64"]))
    if op == "khatv":
        return dict(c, op="khatv", n=_log(rng, 1000, 50000), t=rng.choice([1, 9, 16, 33]), prec="bf16x3")
    if op == "mll":
        return dict(c, op="mll", n=_log(rng, 1000, 65000), t=rng.choice([8, 15, 15, 32]), rank=rng.choice([0, 20, 100]),
                    iters=100, tol=1e-6, prec="bf16x3", ell=rng.choice([1.0, 2.0]))
    if op == "predict":
        return dict(c, op="predict", n=_log(rng, 8000, 262144), m=_log(rng, 10, 1200), kc=rng.choice([0, 40, 256, 256]),
                    prec="bf16x3")
    if op == "exact":
        return dict(c, op="exact", n=_log(rng, 500, 7500))
    if op == "nystrom":
        return dict(c, op="nystrom", n=_log(rng, 4000, 32768), rank=_log(rng, 100, 4000), ell=3.0)
    return dict(c, op="bpcg", n=_log(rng, 2000, 8192), rank=_log(rng, 100, 1000), t=rng.choice([10, 50]), iters=300,
                tol=1e-6, prec="fp64")


# ---------------------------------------------------------------- inputs


def _inputs(case, seed):
    """X (n, d), lengthscales, targets y, and the generators for whatever else the case needs."""
    n, d = case["n"], case["d"]
    rng = np.random.default_rng(seed)
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    mu = 2.0 * torch.randn(64, d, generator=g, device=DEV, dtype=torch.float64)

    def rows(m):
        sizes = rng.integers(10, 301, size=m // 10 + 1)
        comp = np.repeat(rng.integers(0, 64, size=len(sizes)), sizes)[:m]
        return mu[torch.from_numpy(comp).to(DEV)] + torch.randn(m, d, generator=g, device=DEV, dtype=torch.float64)

    X = rows(n)
    ell = rng.uniform(0.5, 2.0, size=d) * case["ell"]
    om = rng.standard_normal((256, d)) / ell
    if case["kind"] == "matern52":
        om *= np.sqrt(5.0 / rng.chisquare(5.0, size=256))[:, None]
    ph = X @ torch.from_numpy(om.T.copy()).to(DEV) + torch.from_numpy(rng.uniform(0, 2 * math.pi, 256)).to(DEV)
    y = math.sqrt(2.0 / 256) * (torch.cos(ph) @ torch.from_numpy(rng.standard_normal(256)).to(DEV))
    y = y + math.sqrt(case["noise"]) * torch.randn(n, generator=g, device=DEV, dtype=torch.float64)
    return X.contiguous(), ell, y, rows, g, rng


def _block(y, t, g):
    V = torch.randn(t, y.shape[0], generator=g, device=DEV, dtype=torch.float64)
    V[0] = y
    return V


def prepare(case, seed):
    X, ell, y, rows, g, rng = _inputs(case, seed)
    s = dict(case=case, X=X, y=y, kern=gp.Kernel(ell, 1.0, case["noise"], case["kind"]))
    op, n = case["op"], case["n"]
    if op == "kmm":
        s["V"] = _block(y, case["t"], g)
        s["Z"] = rows(case["m"]).contiguous() if "m" in case else None
    elif op == "khatv":
        s["V"] = _block(y, case["t"], g).requires_grad_(True)
        s["G"] = torch.randn(case["t"], n, generator=g, device=DEV, dtype=torch.float64)
        s["log_theta"] = torch.from_numpy(np.log(np.concatenate([ell, [1.0, case["noise"]]]))).requires_grad_(True)
    elif op == "mll":
        s["seed"] = int(seed)
    elif op == "predict":
        # a resident model: weights alpha, a variance cache of unit-norm columns, and a request's rows
        alpha, R = _cache(y, case["kc"], g)
        s["Z"] = rows(case["m"]).contiguous()
        s["model"] = gp.PredictModel(s["kern"], X, alpha, R, precision=case["prec"])
        s["ws"] = gp.workspace(s["model"].workspace_bytes(case["m"]), X.device)
        s["mean"] = torch.empty(case["m"], dtype=torch.float64, device=DEV)
        s["var"] = torch.empty(case["m"], dtype=torch.float64, device=DEV) if case["kc"] else None
    elif op in ("nystrom", "bpcg"):
        s["landmarks"] = np.sort(rng.choice(n, case["rank"], replace=False))
        if op == "bpcg":
            s["B"] = _block(y, case["t"], g)
            s["pc"] = gp.nystrom_chol_precond(s["kern"], X, s["landmarks"])
    return s


def _cache(y, kc, g):
    alpha = y / y.norm()
    if not kc:
        return alpha, None
    R = torch.randn(kc, y.shape[0], generator=g, device=DEV, dtype=torch.float64)
    return alpha, (R / R.norm(dim=1, keepdim=True)).contiguous()


# ---------------------------------------------------------------- one pass


def run(s):
    c = s["case"]
    op = c["op"]
    if op == "kmm":
        return gp.kmm(s["kern"], s["X"], s["V"], Z=s["Z"], precision=c["prec"])
    if op == "khatv":
        W = autograd.KhatV.apply(s["log_theta"], s["X"], s["V"], c["kind"], c["prec"])
        gt, gv = torch.autograd.grad(W, (s["log_theta"], s["V"]), s["G"])
        return W.detach(), gt, gv
    if op == "mll":
        r = gp.mll_and_grad(s["kern"], s["X"], s["y"], probes=c["t"], rank=c["rank"], max_iter=c["iters"],
                            tol=c["tol"], seed=s["seed"], precision=c["prec"])
        return r.mll, r.grad
    if op == "predict":
        mean, var = s["model"](s["Z"], with_var=c["kc"] > 0, ws=s["ws"], mean=s["mean"], var=s["var"])
        return (mean,) if var is None else (mean, var)
    if op == "exact":
        r = gp.exact_mll_and_grad(s["kern"], s["X"], s["y"], with_grad=True, with_omega=True)
        return r.mll, r.grad, r.omega
    if op == "nystrom":
        return gp.nystrom_chol_precond(s["kern"], s["X"], s["landmarks"]).E
    return gp.bpcg(s["kern"], s["X"], s["B"], c["iters"], c["tol"], pc=s["pc"], precision=c["prec"]).W


def work(case):
    """Each input read once and each output written once; flops of the contractions: each distance of an unordered
    pair once, each kernel entry times each column."""
    op, n, d = case["op"], case["n"], case["d"]
    if op == "kmm":
        t = case["t"]
        if "m" in case:
            m = case["m"]
            return {"bytes": 8 * (n * d + m * d + n * t + m * t), "flops": 2 * m * n * (d + t)}
        return {"bytes": 8 * (n * d + 2 * n * t), "flops": n * n * d + 2 * n * n * t}
    if op == "khatv":  # two products, and one pass over pairs for C (t) and the d derivative forms
        t = case["t"]
        return {"bytes": 8 * (n * d + 4 * n * t), "flops": n * n * d + 4 * n * n * t + n * n * (t + 2 * d)}
    if op == "mll":  # factor, at least two products of the block, and the gradient's pass over pairs
        s, k = case["t"] + 1, case["rank"]
        it = case["iters"] if case["tol"] == 0.0 else 2
        return {"bytes": 8 * (n * d + n * k * k // 2 + it * n * s * 8),
                "flops": it * (n * n * d + 2 * n * n * s + 4 * n * k * s) + 2 * n * k * k + n * n * (s + 2 * d)}
    if op == "predict":  # 32 bits per value of the resident model
        m, t = case["m"], case["kc"] + 1
        return {"bytes": 4 * n * (d + t) + 8 * m * (d + 2), "flops": 2 * m * n * (d + t)}
    if op == "exact":
        return {"bytes": 8 * (n * d + 2 * n), "flops": n * n * n + 3 * n * n * d}
    if op == "nystrom":
        r = case["rank"]
        return {"bytes": 8 * (n * d + n * r), "flops": 2 * n * r * d + 5 * n * r * r}
    s, r = case["t"], case["rank"]  # at least two iterations
    return {"bytes": 8 * (n * d + n * r + 2 * n * s), "flops": 2 * (n * n * d + 2 * n * n * s + 4 * n * r * s)}


# ---------------------------------------------------------------- the same in 64 bits


def _profile(kind, r2):
    """k and psi = -2 dk / d(r^2) at squared scaled distances, s_f = 1."""
    if kind == "matern52":
        u = torch.sqrt(5.0 * r2)
        e = torch.exp(-u)
        return (1.0 + u + u * u / 3.0) * e, (5.0 / 3.0) * (1.0 + u) * e
    e = torch.exp(-0.5 * r2)
    return e, e


def _r2(A, B, direct):
    if direct:
        r2 = torch.zeros(A.shape[0], B.shape[0], dtype=torch.float64, device=DEV)
        for j in range(A.shape[1]):
            r2 += (A[:, j, None] - B[None, :, j]) ** 2
        return r2
    return ((A * A).sum(1)[:, None] + (B * B).sum(1)[None, :] - 2.0 * (A @ B.T)).clamp_min_(0.0)


def _chunks(rows, cols):
    step = max(1, min(rows, (1 << 28) // cols))
    return [(i, min(rows, i + step)) for i in range(0, rows, step)]


def _scaled(X, ell, ctr=None):
    ctr = X.mean(0) if ctr is None else ctr
    return (X - ctr) / torch.from_numpy(ell).to(DEV)


def _kmm(case, Xs, V, noise, Zs=None, direct=False):
    """(t, rows): K V, with the exact diagonal when square."""
    A = Xs if Zs is None else Zs
    Vt = V.T.contiguous()
    out = torch.empty(A.shape[0], V.shape[0], dtype=torch.float64, device=DEV)
    for i, j in _chunks(A.shape[0], Xs.shape[0]):
        k, _ = _profile(case["kind"], _r2(A[i:j], Xs, direct))
        if Zs is None:
            k[torch.arange(j - i, device=DEV), torch.arange(i, j, device=DEV)] = 1.0 + noise
        out[i:j] = k @ Vt
    return out.T.contiguous()


def _forms(case, Xs, C_rows, noise_form):
    """sum_ab C_ab dK_ab / dlog theta for C given by rows (C symmetrised by the sum)."""
    n, d = Xs.shape
    g = torch.zeros(d + 2, dtype=torch.float64, device=DEV)
    for i, j in _chunks(n, n):
        k, psi = _profile(case["kind"], _r2(Xs[i:j], Xs, False))
        dia = torch.arange(j - i, device=DEV), torch.arange(i, j, device=DEV)
        k[dia] = 1.0
        Cm = C_rows(i, j)
        g[d] += (k * Cm).sum()
        psi *= Cm
        psi[dia] = 0.0
        xa = Xs[i:j]
        g[:d] += (xa * xa * psi.sum(1)[:, None]).sum(0) - 2.0 * (xa * (psi @ Xs)).sum(0) + \
            (Xs * Xs * psi.sum(0)[:, None]).sum(0)
    g[d + 1] = noise_form
    return g


def _splitmix(x):
    with np.errstate(over="ignore"):
        z = x + np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        return z ^ (z >> np.uint64(31))


def _signs(seed, stream, count):
    key = _splitmix(np.array([seed], dtype=np.uint64))[0]
    h = _splitmix(key ^ (np.uint64(stream << 40) | np.arange(count, dtype=np.uint64)))
    return torch.from_numpy(np.where(h >> np.uint64(63), -1.0, 1.0)).to(DEV)


def _pivchol(case, Xs, k):
    n = Xs.shape[0]
    L = torch.zeros(n, k, dtype=torch.float64, device=DEV)
    delta = torch.ones(n, dtype=torch.float64, device=DEV)
    for m in range(k):
        v, p = delta.max(0)
        if v <= 1e-12:
            break
        kv, _ = _profile(case["kind"], ((Xs - Xs[p]) ** 2).sum(1))
        L[:, m] = (kv - L[:, :m] @ L[p, :m]) / v.sqrt()
        delta -= L[:, m] ** 2
        delta[p] = 0.0
    return L


def _mll(case, Xs, y, seed):
    n, t, k, s2 = case["n"], case["t"], case["rank"], case["noise"]
    logdet_p = 0.0
    L = _pivchol(case, Xs, k) if k else None
    if k:
        Lc = torch.linalg.cholesky(s2 * torch.eye(k, dtype=torch.float64, device=DEV) + L.T @ L)
        logdet_p = (n - k) * math.log(s2) + 2.0 * float(torch.log(torch.diagonal(Lc)).sum())
    B = torch.empty(n, t + 1, dtype=torch.float64, device=DEV)
    B[:, 0] = y
    for c in range(1, t + 1):
        e2 = _signs(seed, c, n)
        B[:, c] = L @ _signs(seed, c + 65536, k) + math.sqrt(s2) * e2 if k else e2
    apply = (lambda R: (R - L @ torch.cholesky_solve(L.T @ R, Lc)) / s2) if k else (lambda R: R.clone())
    K = torch.empty(n, n, dtype=torch.float64, device=DEV)
    for i, j in _chunks(n, n):
        K[i:j] = _profile(case["kind"], _r2(Xs[i:j], Xs, False))[0]
    K.diagonal().fill_(1.0 + s2)
    U, R = torch.zeros_like(B), B.clone()
    Z = apply(R)
    Z0, D = Z.clone(), Z.clone()
    gam = (R * Z).sum(0)
    gam0, bn = gam.clone(), B.norm(dim=0)
    active = torch.ones(t + 1, dtype=torch.bool, device=DEV)
    al, be, its = [], [], torch.zeros(t + 1, dtype=torch.int64, device=DEV)
    for _ in range(case["iters"]):
        Q = K @ D
        a = torch.where(active, gam / (D * Q).sum(0), torch.zeros_like(gam))
        U += a * D
        R -= a * Q
        its += active
        active = active & (R.norm(dim=0) > max(case["tol"], 1e-12) * bn)
        Z = apply(R)
        gn = (R * Z).sum(0)
        b = torch.where(active, gn / gam, torch.zeros_like(gam))
        gam = torch.where(active, gn, gam)
        D = torch.where(active, Z + b * D, torch.zeros_like(D))
        al.append(a.cpu().numpy())
        be.append(b.cpu().numpy())
        if not bool(active.any()):
            break
    del K
    logdet = 0.0
    for c in range(1, t + 1):
        J = int(its[c])
        a, b = np.array([v[c] for v in al[:J]]), np.array([v[c] for v in be[:J]])
        T = np.diag(1.0 / a)
        for j in range(1, J):
            T[j, j] += b[j - 1] / a[j - 1]
            T[j, j - 1] = T[j - 1, j] = math.sqrt(b[j - 1]) / a[j - 1]
        lam, q = np.linalg.eigh(T)
        logdet += float(gam0[c]) * float((q[0] ** 2 * np.log(lam)).sum())
    logdet = logdet_p + logdet / t
    mll = -0.5 * float(y @ U[:, 0]) - 0.5 * logdet - 0.5 * n * LOG2PI
    Z0[:, 0] = U[:, 0]
    w = torch.full((t + 1,), -0.5 / t, dtype=torch.float64, device=DEV)
    w[0] = 0.5
    Uw = U * w
    return mll, _forms(case, Xs, lambda i, j: Uw[i:j] @ Z0.T, s2 * float((Uw * Z0).sum())).cpu().numpy()


def exact(case, seed):
    op, n, noise = case["op"], case["n"], case["noise"]
    X, ell, y, rows, g, rng = _inputs(case, seed)
    Xs = _scaled(X, ell)
    eye = lambda r: torch.eye(r, dtype=torch.float64, device=DEV)  # noqa: E731
    if op == "kmm":
        V = _block(y, case["t"], g)
        Zs = _scaled(rows(case["m"]), ell, X.mean(0)) if "m" in case else None
        return _kmm(case, Xs, V, noise, Zs, direct=case["prec"] == "fp64")
    if op == "khatv":
        V = _block(y, case["t"], g)
        G = torch.randn(case["t"], n, generator=g, device=DEV, dtype=torch.float64)
        Gt = G.T.contiguous()
        gt = _forms(case, Xs, lambda i, j: Gt[i:j] @ V, noise * float((G * V).sum()))
        return _kmm(case, Xs, V, noise), gt.cpu(), _kmm(case, Xs, G, noise)
    if op == "mll":
        return _mll(case, Xs, y, int(seed))
    if op == "predict":
        alpha, R = _cache(y, case["kc"], g)
        Zs = _scaled(rows(case["m"]), ell, X.mean(0))
        V = alpha[None] if R is None else torch.cat([alpha[None], R])
        P = _kmm(case, Xs, V, 0.0, Zs)
        return (P[0],) if R is None else (P[0], 1.0 - (P[1:] ** 2).sum(0))
    if op == "exact":
        r2 = _r2(Xs, Xs, True)
        K = _profile(case["kind"], r2)[0] + noise * eye(n)
        Lk = torch.linalg.cholesky(K)
        Ki = torch.cholesky_solve(eye(n), Lk)
        om = torch.cholesky_solve(y[:, None], Lk)[:, 0]
        mll = -0.5 * float(y @ om) - float(torch.log(torch.diagonal(Lk)).sum()) - 0.5 * n * LOG2PI
        M = 0.5 * (om[:, None] * om[None, :] - Ki)
        gr = _forms(case, Xs, lambda i, j: M[i:j], noise * float(torch.diagonal(M).sum()))
        return mll, gr.cpu().numpy(), om
    if op == "nystrom":
        r = case["rank"]
        M = torch.from_numpy(np.sort(rng.choice(n, r, replace=False))).to(DEV)
        KX = _profile(case["kind"], _r2(Xs, Xs[M], True))[0]
        Lm = torch.linalg.cholesky(KX[M] + 1e-10 * r * eye(r))
        Ft = torch.linalg.solve_triangular(Lm, KX.T, upper=False)
        Lg = torch.linalg.cholesky(Ft @ Ft.T + noise * eye(r))
        return torch.linalg.solve_triangular(Lg, Ft, upper=False)
    rng.choice(n, case["rank"], replace=False)
    B = _block(y, case["t"], g)
    K = _profile(case["kind"], _r2(Xs, Xs, True))[0] + noise * eye(n)
    return torch.cholesky_solve(B.T.contiguous(), torch.linalg.cholesky(K)).T.contiguous()
