"""Branches of the tiled kernels that only large sizes and wide blocks reach, and the sums whose order is fixed to the bit."""
from fractions import Fraction

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


def _fma(a, b, c):
    return float(Fraction(a) * Fraction(b) + Fraction(c))


@pytest.mark.parametrize("k", [3, 70, 128, 130])
def test_woodbury_solve_has_the_bits_of_its_scalar_loops(k):
    """Z0 = (B - L C^{-1} L^T B) / sigma^2, every sum a chain of FMAs in ascending order of its index: the matrix cores and
    the in-LDS solve (k <= 128) keep these bits, on which mBCG's results rest."""
    from paper_2109_09817_amd import gp
    n, d, s, noise = 150, 5, 2, 1e-2
    rng = np.random.default_rng(k)
    X, B = rng.standard_normal((n, d)), rng.standard_normal((s, n))
    kern = gp.Kernel(rng.uniform(1.0, 2.0, d), 1.0, noise)
    pc = gp.pivchol(kern, dev(X), k)
    Z0 = host(gp.mbcg(kern, dev(X), dev(B), 1, 0.0, pc=pc, precision="fp32").Z0)
    L, Cc = host(pc.L), host(pc.Cchol)  # L[j] = column j; Cc[j, i] = entry (i, j) of the factor
    for c in range(s):
        y = []
        for j in range(k):
            v = 0.0
            for i in range(n):
                v = _fma(L[j, i], B[c, i], v)
            y.append(v)
        for j in range(k):
            for i in range(j):
                y[j] = _fma(-Cc[i, j], y[i], y[j])
            y[j] = y[j] / Cc[j, j]
        for j in reversed(range(k)):
            for i in range(j + 1, k):
                y[j] = _fma(-Cc[j, i], y[i], y[j])
            y[j] = y[j] / Cc[j, j]
        ref = np.empty(n)
        for i in range(n):
            v = 0.0
            for j in range(k):
                v = _fma(L[j, i], y[j], v)
            ref[i] = (1.0 / noise) * (B[c, i] - v)
        np.testing.assert_array_equal(Z0[c], ref)


def _block_dot(a, b):
    """Sum of a b as the column reductions add it, up to 256 blocks of 256 rows: products, a tree over the lanes of each wave,
    the waves of a block in order, and the block sums once more in the same way."""
    def block_sum(v):
        w = np.zeros(256)
        w[:len(v)] = v
        w = w.reshape(4, 64)
        while w.shape[1] > 1:
            h = w.shape[1] // 2
            w = w[:, :h] + w[:, h:]
        r = 0.0
        for x in w[:, 0]:
            r = r + x
        return r
    p = a * b
    return block_sum([block_sum(p[i:i + 256]) for i in range(0, len(p), 256)])


@pytest.mark.parametrize("prec", ["bf16x3", "fp32", "fp64"])
@pytest.mark.parametrize("n", [1, 300, 1031])
def test_first_step_size_to_the_bit(n, prec):
    """alpha = (B . B) / (B . K_hat B), the product's dot added in its epilogue (mixed and FP32 forms) or by the column
    reduction (FP64): the same additions, on the values that gp_kmm returns for the same product."""
    from paper_2109_09817_amd import gp
    rng = np.random.default_rng(n)
    X, B = rng.standard_normal((n, 6)), rng.standard_normal((3, n))
    kern = gp.Kernel(np.full(6, 1.5), 1.1, 0.5)
    r = gp.mbcg(kern, dev(X), dev(B), 1, 0.0, precision=prec)
    KB = host(gp.kmm(kern, dev(X), dev(B), precision=prec))
    ref = [_block_dot(B[c], B[c]) / _block_dot(B[c], KB[c]) for c in range(3)]
    np.testing.assert_array_equal(r.alpha[0], ref)


@pytest.mark.parametrize("n", [131072, 131073, 262145])
def test_first_step_size_to_the_bit_with_many_partial_sums(n):
    """512 blocks' sums are added by every workgroup, more of them once before; 512 rows to a block at n = 262,145.  B holds
    signs, so that every product is exact and the FMAs are plain additions."""
    from paper_2109_09817_amd import gp
    rng = np.random.default_rng(n)
    X, B = rng.standard_normal((n, 4)), rng.choice([-1.0, 1.0], (2, n))
    kern = gp.Kernel(np.full(4, 0.5), 1.1, 0.5)
    r = gp.mbcg(kern, dev(X), dev(B), 1, 0.0, precision="bf16x3")
    KB = host(gp.kmm(kern, dev(X), dev(B), precision="bf16x3"))

    def block_sum(v):
        w = np.zeros(256)
        for i in range(0, len(v), 256):
            w[:len(v[i:i + 256])] += v[i:i + 256]
        w = w.reshape(4, 64)
        while w.shape[1] > 1:
            h = w.shape[1] // 2
            w = w[:, :h] + w[:, h:]
        return ((w[0, 0] + w[1, 0]) + w[2, 0]) + w[3, 0]
    rows = 256 if n <= 262144 else 512

    def dot(a, b):
        return block_sum(np.array([block_sum((a * b)[i:i + rows]) for i in range(0, n, rows)]))
    np.testing.assert_array_equal(r.alpha[0], [dot(B[c], B[c]) / dot(B[c], KB[c]) for c in range(2)])


@pytest.mark.parametrize("kind", [ok.MATERN52, ok.RBF])
@pytest.mark.parametrize("d", [5, 21, 48, 64, 100])
@pytest.mark.parametrize("t", [3, 20, 40, 64, 130])
def test_fp32_products_with_one_and_two_row_blocks_per_wave(t, d, kind):
    """One or two 16-row blocks per wave, by the number of workgroups (m = 1,500 rows, single rows and 300 of them differ in
    it): a row has the same bits either way.  Square product (n = 7,001) against the FP64 form or the
    oracle, bar 1e-5 of the off-diagonal part as elsewhere."""
    from paper_2109_09817_amd import gp
    rng = np.random.default_rng(d + t)
    n, m = 50000, 1500
    X, V, Z = dev(rng.standard_normal((n, d))), dev(rng.standard_normal((t, n))), rng.standard_normal((m, d))
    th = ok.Theta(rng.uniform(0.8, 1.2, d) * np.sqrt(d), 1.1, 1e-2, kind)
    got = host(gp.kmm(_gk(th), X, V, Z=dev(Z), precision="fp32"))
    for r in (0, 31, 700, 1499):
        np.testing.assert_array_equal(host(gp.kmm(_gk(th), X, V, Z=dev(Z[r:r + 1]), precision="fp32"))[:, 0], got[:, r])
    np.testing.assert_array_equal(host(gp.kmm(_gk(th), X, V, Z=dev(Z[900:1200]), precision="fp32")), got[:, 900:1200])
    X, V = X[:7001].contiguous(), V[:, :7001].contiguous()
    got = host(gp.kmm(_gk(th), X, V, precision="fp32"))
    if d <= 64:
        ref = host(gp.kmm(_gk(th), X, V, precision="fp64"))
    else:
        ref = ok.khat_matmul(host(X), th, host(V).T).T
    assert np.linalg.norm(got - ref) <= 1e-5 * np.linalg.norm(ref - 1.11 * host(V))


@pytest.mark.parametrize("kind", [ok.MATERN52, ok.RBF])
@pytest.mark.parametrize("t", [65, 68, 69, 100, 130])
def test_fp64_products_beyond_64_columns(t, kind):
    """Columns beyond whole groups of 64 in the same launch (small n) or in one of their own (n = 9,000).  Bar as for the
    other FP64 products: 1e-13 of |K| |V|.  A row of a cross product has the same bits alone and among others, which take
    more launches."""
    from paper_2109_09817_amd import gp
    rng = np.random.default_rng(t)
    for n, d in ((60, 48), (700, 20), (9000, 8)):
        X, V = rng.standard_normal((n, d)), rng.standard_normal((t, n))
        th = ok.Theta(rng.uniform(1.0, 2.0, d) * np.sqrt(d), 1.2, 1e-3, kind)
        rows = np.arange(n) if n < 1000 else np.sort(rng.choice(n, 500, replace=False))
        got = host(gp.kmm(_gk(th), dev(X), dev(V), precision="fp64"))[:, rows]
        K = ok.kernel(X[rows], X, th)
        K[np.arange(len(rows)), rows] += 1e-3
        assert np.max(np.abs(got - V @ K.T) / (np.abs(V) @ np.abs(K).T)) <= 1e-13
    Z = rng.standard_normal((40000, 8))
    th = ok.Theta(rng.uniform(2.0, 4.0, 8), 1.0, 0.0, kind)
    X, V = rng.standard_normal((900, 8)), rng.standard_normal((t, 900))
    got = host(gp.kmm(_gk(th), dev(X), dev(V), Z=dev(Z), precision="fp64"))
    for r in (0, 20001, 39999):
        one = host(gp.kmm(_gk(th), dev(X), dev(V), Z=dev(Z[r:r + 1]), precision="fp64"))
        np.testing.assert_array_equal(one[:, 0], got[:, r])


@pytest.mark.parametrize("kind", [ok.MATERN52, ok.RBF])
@pytest.mark.parametrize("n,d", [(31, 3), (64, 32), (65, 64), (700, 48)])
def test_fp64_square_and_cross_products_agree(n, d, kind):
    """A square product reads its row norms, a cross product computes them, by the same additions: without noise and with
    the same rows both forms differ in the diagonal alone, which the square one sets to s_f and the cross one gets from
    a squared distance that rounds to at most (d + 4) 2^-52 of the norms."""
    from paper_2109_09817_amd import gp
    rng = np.random.default_rng(n)
    X = rng.standard_normal((n, d))
    th = ok.Theta(rng.uniform(1.0, 2.0, d) * np.sqrt(d), 1.2, 0.0, kind)
    V = np.eye(n)[: min(n, 16)]
    square = host(gp.kmm(_gk(th), dev(X), dev(V), precision="fp64"))
    cross = host(gp.kmm(_gk(th), dev(X), dev(V), Z=dev(X), precision="fp64"))
    off = ~np.eye(len(V), n, dtype=bool)
    np.testing.assert_array_equal(square[off], cross[off])
    r2 = 2 * (d + 4) * 2.0**-52 * np.max(np.sum((X / th.ell) ** 2, axis=1))
    assert np.max(np.abs(square[~off] - cross[~off])) <= 1.2 * (5 / 3 + 0.5) * r2 + 1e-15
