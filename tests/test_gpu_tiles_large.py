"""Branches of the tiled kernels that only large sizes and wide blocks reach, and the sums whose order is fixed to the bit."""
import numpy as np
import pytest

import oracle.kernel as ok
from _helpers import dev, host

pytestmark = pytest.mark.gpu


def _gk(th):
    from paper_2109_09817_amd import gp
    return gp.Kernel(th.ell, th.sf, th.noise, "matern52" if th.kind == ok.MATERN52 else "rbf")


@pytest.mark.parametrize("n", [3400, 6209, 7201])
def test_cholesky_and_inverse_beyond_one_launch_of_trailing_tiles(n):
    """A diagonal block carries up to 255 of the 128-wide trailing tiles beside it: 276 tiles take two launches (n = 3,400),
    more than 1,020 take larger shares (n = 6,209: 1,035).  The doubled inverse takes 128-wide batches from four pairs of
    1,024 rows (n = 7,201) or two of 2,048 on, the last one ragged.  Residual of K_hat omega = y: about 1e-16 times
    cond(K_hat) < 1e4 and the square root of n; bar 1e-10 (a tile left out or taken twice: above 1e-3)."""
    from paper_2109_09817_amd import gp
    rng = np.random.default_rng(n)
    X, y = rng.standard_normal((n, 5)), rng.standard_normal(n)
    th = ok.Theta(rng.uniform(0.3, 0.6, 5), 1.2, 0.1, ok.MATERN52)
    r = gp.exact_mll_and_grad(_gk(th), dev(X), dev(y), with_grad=False, with_omega=True)
    back = ok.khat_matmul(X, th, host(r.omega)[:, None])[:, 0]
    assert np.linalg.norm(back - y) <= 1e-10 * np.linalg.norm(y)


def test_large_rank_factor_with_whole_and_split_gram_tiles():
    """r = 4,001: 528 lower 128-wide tiles, 512 of them whole and 16 split in k, their products in slabs.  P^{-1} P v = v with
    P^{-1} = sigma^{-2} (I - E E^T) and P v by a dense solve: rounding is amplified by cond(K_MM) and cond(P), both below 1e4
    here, at most 1e-8; bar 1e-8 (a tile left out: above 1e-3)."""
    from paper_2109_09817_amd import gp
    n, r, s2 = 4600, 4001, 0.1
    rng = np.random.default_rng(r)
    X = rng.standard_normal((n, 6))
    th = ok.Theta(rng.uniform(0.3, 0.6, 6), 1.0, s2, ok.MATERN52)
    M = np.sort(rng.choice(n, r, replace=False))
    E = host(gp.nystrom_chol_precond(_gk(th), dev(X), M).E)
    KMX = ok.kernel(X[M], X, th)
    v = rng.standard_normal((n, 3))
    Pv = KMX.T @ np.linalg.solve(KMX[:, M] + 1e-10 * r * np.eye(r), KMX @ v) + s2 * v
    back = (Pv - E.T @ (E @ Pv)) / s2
    assert np.linalg.norm(back - v) <= 1e-8 * np.linalg.norm(v)


@pytest.mark.parametrize("s", [17, 33, 50, 64])
@pytest.mark.parametrize("solver", ["bcg", "bpcg"])
def test_block_solvers_with_wide_blocks(solver, s):
    """Two to four 16-column blocks in U += D alpha, R -= Q alpha and D = R + D beta, which write over one of their operands,
    at a ragged number of rows.  FP64 products to 1e-10 against the dense solve: bar 10 cond(K_hat) 1e-10, cond < 1e4."""
    from paper_2109_09817_amd import gp
    n = 1013
    rng = np.random.default_rng(s)
    X, B = rng.standard_normal((n, 6)), rng.standard_normal((s, n))
    th = ok.Theta(rng.uniform(1.0, 2.0, 6), 1.0, 0.1, ok.MATERN52)
    Kh = ok.khat(X, th)
    ev = np.linalg.eigvalsh(Kh)
    kappa = ev[-1] / ev[0]
    assert kappa < 1e4
    ref = np.linalg.solve(Kh, B.T).T
    for r in (0, 70):
        M = np.sort(rng.choice(n, r, replace=False)) if r else None
        if solver == "bcg":
            pc = gp.nystrom_precond(_gk(th), dev(X), M) if r else None
            res = gp.bcg(_gk(th), dev(X), dev(B), 300, 1e-10, pc=pc, precision="fp64")
        else:
            pc = gp.nystrom_chol_precond(_gk(th), dev(X), M) if r else None
            res = gp.bpcg(_gk(th), dev(X), dev(B), 300, 1e-10, pc=pc, precision="fp64")
        assert res.status == 0 and res.iters >= 2
        assert np.linalg.norm(host(res.W) - ref) <= 10 * kappa * 1e-10 * np.linalg.norm(ref)


@pytest.mark.parametrize("s", [64, 65, 130])
def test_woodbury_solve_in_groups_of_columns(s):
    """P^{-1} B = Z0 of an mBCG run for more columns than one group of 64 holds.  Against the dense solve; rounding is
    amplified by cond(P) <= 1e5 here: bar 1e-10."""
    from paper_2109_09817_amd import gp
    n, d, k = 700, 6, 40
    rng = np.random.default_rng(s)
    X, B = rng.standard_normal((n, d)), rng.standard_normal((s, n))
    kern = _gk(ok.Theta(rng.uniform(1.0, 2.0, d), 1.0, 1e-2, ok.MATERN52))
    pc = gp.pivchol(kern, dev(X), k)
    r = gp.mbcg(kern, dev(X), dev(B), 1, 0.0, pc=pc, precision="fp32")
    L = host(pc.L)
    ref = np.linalg.solve(L.T @ L + 1e-2 * np.eye(n), B.T).T
    assert np.linalg.norm(host(r.Z0) - ref) <= 1e-10 * np.linalg.norm(ref)
