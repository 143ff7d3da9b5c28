"""Edges of the tiled kernels: sizes just below, at and above the tile edges, against the FP64 oracle."""
import numpy as np
import pytest

import oracle.kernel as ok
from oracle import exact
from _helpers import dev, host

pytestmark = pytest.mark.gpu


def _gk(th):
    from paper_2109_09817_amd import gp
    return gp.Kernel(th.ell, th.sf, th.noise, "matern52" if th.kind == ok.MATERN52 else "rbf")


@pytest.mark.parametrize("n", [15, 16, 17, 33, 47, 49, 81, 193, 449])
def test_exact_gp_at_the_edges_of_the_diagonal_steps(n):
    """Diagonal blocks are factored in 16-column steps and inverted pairwise (64, 128, 256 ... rows); the bars are
    those of the dense parity cases (1e-10, well above 1e-14 kappa here)."""
    from paper_2109_09817_amd import gp
    rng = np.random.default_rng(n)
    X, y = rng.standard_normal((n, 4)), rng.standard_normal(n)
    th = ok.Theta(rng.uniform(1.0, 2.0, 4), 1.3, 1e-2, ok.MATERN52)
    r = gp.exact_mll_and_grad(_gk(th), dev(X), dev(y), with_grad=True, with_omega=True)
    o = exact.cholesky_gp(X, y, th)
    g = exact.mll_grad(X, y, th)
    assert abs(r.mll - o["mll"]) <= 1e-10 * (abs(o["quad"]) + abs(o["logdet"]) + n)
    assert np.linalg.norm(host(r.omega) - o["omega"]) <= 1e-10 * np.linalg.norm(o["omega"])
    assert np.max(np.abs(r.grad - g)) <= 1e-10 * np.max(np.abs(g)) * n


def test_exact_gp_with_128_wide_tiles_and_a_ragged_edge():
    """From 23 tile rows on the trailing updates take 128-wide tiles; n = 3,301 leaves a ragged last tile.  Bars as
    for the dense parity cases (1e-14 kappa with kappa below 1e4 here)."""
    from paper_2109_09817_amd import gp
    n = 3301
    rng = np.random.default_rng(5)
    X, y = rng.standard_normal((n, 3)), rng.standard_normal(n)
    th = ok.Theta(rng.uniform(0.3, 0.6, 3), 1.3, 1e-1, ok.MATERN52)
    r = gp.exact_mll_and_grad(_gk(th), dev(X), dev(y), with_grad=True, with_omega=True)
    o = exact.cholesky_gp(X, y, th)
    g = exact.mll_grad(X, y, th)
    assert abs(r.mll - o["mll"]) <= 1e-10 * (abs(o["quad"]) + abs(o["logdet"]) + n)
    assert np.linalg.norm(host(r.omega) - o["omega"]) <= 1e-10 * np.linalg.norm(o["omega"])
    assert np.max(np.abs(r.grad - g)) <= 1e-9 * np.max(np.abs(g))


@pytest.mark.parametrize("n,r", [(11009, 333), (700, 129)])
def test_large_rank_factor_on_both_tile_sizes(n, r):
    """E^T = L_G^{-1} L_M^{-1} K_MX against numpy: 128-wide tiles (n = 11,009, ragged both ways) and 64-wide ones.
    Rounding is amplified by cond(K_MM + delta I), below 1e4 on this data: bar 1e-11."""
    import scipy.linalg as sl
    from paper_2109_09817_amd import gp
    rng = np.random.default_rng(n)
    X = rng.standard_normal((n, 6))
    th = ok.Theta(rng.uniform(0.5, 1.0, 6), 1.0, 1e-2, ok.MATERN52)
    M = np.sort(rng.choice(n, r, replace=False))
    E = host(gp.nystrom_chol_precond(_gk(th), dev(X), M).E)
    KMX = ok.kernel(X[M], X, th)
    Lm = np.linalg.cholesky(KMX[:, M] + 1e-10 * r * np.eye(r))
    F = sl.solve_triangular(Lm, KMX, lower=True)
    ref = sl.solve_triangular(np.linalg.cholesky(F @ F.T + 1e-2 * np.eye(r)), F, lower=True)
    assert np.linalg.norm(E - ref) <= 1e-11 * np.linalg.norm(ref)


def _fp64_err(th, X, V, Z=None):
    from paper_2109_09817_amd import gp
    got = host(gp.kmm(_gk(th), dev(X), dev(V), Z=None if Z is None else dev(Z), precision="fp64"))
    mm = (lambda W: ok.khat_matmul(X, th, W.T).T) if Z is None else (lambda W: ok.cross_matmul(Z, X, th, W.T).T)
    return got, float(np.max(np.abs(got - mm(V)) / mm(np.abs(V))))


@pytest.mark.parametrize("kind", [ok.MATERN52, ok.RBF])
@pytest.mark.parametrize("n,d,t", [(100, 5, 4), (257, 16, 5), (800, 17, 17), (513, 33, 36), (600, 48, 52),
                                   (1000, 48, 63), (777, 64, 68), (320, 20, 515)])
def test_fp64_product_column_remainders_and_splits(n, d, t, kind):
    """Columns beyond a 16-wide block on the vector units (1 to 4) or in a padded block, one split and several,
    two column passes (t = 515).  Bar as for the other FP64 products: 1e-13 of |K| |V|."""
    rng = np.random.default_rng(n + t)
    X, V = rng.standard_normal((n, d)), rng.standard_normal((t, n))
    th = ok.Theta(rng.uniform(1.0, 2.0, d) * np.sqrt(d), 1.2, 1e-3, kind)
    assert _fp64_err(th, X, V)[1] <= 1e-13


def test_fp64_cross_product_in_row_slabs_and_row_independence():
    """m = 8,300 rows of 200 columns exceed one slab (4,480 rows) of partial sums; a row's result is bitwise that of a
    call with that row alone (the split of the b range depends on n only)."""
    from paper_2109_09817_amd import gp
    n, d, t, m = 3000, 8, 200, 8300
    rng = np.random.default_rng(2)
    X, V, Z = rng.standard_normal((n, d)), rng.standard_normal((t, n)), rng.standard_normal((m, d))
    th = ok.Theta(rng.uniform(2.0, 4.0, d), 1.0, 0.0, ok.MATERN52)
    got, err = _fp64_err(th, X, V, Z)
    assert err <= 1e-13
    for r in (0, 4479, 4480, 8299):
        one = host(gp.kmm(_gk(th), dev(X), dev(V), Z=dev(Z[r:r + 1]), precision="fp64"))
        np.testing.assert_array_equal(one[:, 0], got[:, r])


def test_fp64_product_without_a_workspace_matches_bitwise():
    import torch
    from paper_2109_09817_amd import gp
    n, d, t = 5000, 48, 16
    rng = np.random.default_rng(4)
    X, V = dev(rng.standard_normal((n, d))), dev(rng.standard_normal((t, n)))
    k = gp.Kernel(rng.uniform(5.0, 9.0, d), 1.0, 1e-4)
    out = torch.empty_like(V)
    gp.kmm_noalloc(k, X, V, out, precision="fp64")
    np.testing.assert_array_equal(host(out), host(gp.kmm(k, X, V, precision="fp64")))


@pytest.mark.parametrize("n,r,s", [(17, 1, 1), (33, 17, 15), (1000, 3, 16), (259, 64, 17), (4097, 65, 33),
                                   (300, 130, 50), (515, 31, 64), (65549, 20, 50), (66001, 5, 3)])
def test_tall_products_at_ragged_sizes(n, r, s):
    """sigma^{-1} V + Z^T diag(g) Z V (both tall-skinny products) on random factors, ragged rows, ranks and columns,
    16 and 32 rows per workgroup.  Bar: 1e-13 of the sums of magnitudes (two sums of at most n and r terms)."""
    from paper_2109_09817_amd import gp
    rng = np.random.default_rng(n + r + s)
    Z, g, V = rng.standard_normal((r, n)), rng.standard_normal(r), rng.standard_normal((s, n))
    pc = gp.Nystrom(dev(Z), dev(g), np.arange(r), 0.25)
    got = host(gp.nystrom_apply(pc, dev(V)))
    ref = 2.0 * V + ((V @ Z.T) * g) @ Z
    mag = 2.0 * np.abs(V) + ((np.abs(V) @ np.abs(Z).T) * np.abs(g)) @ np.abs(Z)
    assert np.max(np.abs(got - ref) / mag) <= 1e-13


def test_tall_product_in_place():
    """Y may be V itself: bitwise the result of the call with a separate output."""
    from paper_2109_09817_amd import gp
    rng = np.random.default_rng(8)
    Z, g, V = dev(rng.standard_normal((37, 70001))), dev(rng.standard_normal(37)), dev(rng.standard_normal((20, 70001)))
    pc = gp.Nystrom(Z, g, np.arange(37), 0.25)
    ref = host(gp.nystrom_apply(pc, V))
    gp.nystrom_apply(pc, V, out=V)
    np.testing.assert_array_equal(host(V), ref)


@pytest.mark.parametrize("k", [1, 63, 64, 65, 100, 127, 128, 129, 200])
def test_woodbury_solve_at_the_edges_of_the_in_lds_factor(k):
    """P^{-1} B = Z0 of an mBCG run: factors up to 128 are solved in LDS (two entries per lane), larger ones are not.
    Against the dense solve; rounding is amplified by cond(P) <= 1e5 here: bar 1e-10."""
    from paper_2109_09817_amd import gp
    n, d, s = 700, 6, 5
    rng = np.random.default_rng(k)
    X, B = rng.standard_normal((n, d)), rng.standard_normal((s, n))
    th = ok.Theta(rng.uniform(1.0, 2.0, d), 1.0, 1e-2, ok.MATERN52)
    kern = _gk(th)
    pc = gp.pivchol(kern, dev(X), k)
    r = gp.mbcg(kern, dev(X), dev(B), 2, 0.0, pc=pc, precision="fp32")
    L = host(pc.L)
    ref = np.linalg.solve(L.T @ L + 1e-2 * np.eye(n), B.T).T
    assert np.linalg.norm(host(r.Z0) - ref) <= 1e-10 * np.linalg.norm(ref)


@pytest.mark.parametrize("n,d", [(31, 3), (33, 16), (300, 17), (257, 49), (1000, 64), (513, 65), (300, 128)])
def test_mixed_product_at_every_slice_count_of_the_point_preparation(n, d):
    """Points are prepared 32 at a time in 16-feature slices (1 to 8 of them) and the centre is added over blocks of
    rows.  Bar: the mixed form's 5e-5 on the off-diagonal part (a correlated kernel, data shifted by 100 lengthscales)."""
    from paper_2109_09817_amd import gp
    rng = np.random.default_rng(n + d)
    X, V = rng.standard_normal((n, d)) + 100.0, rng.standard_normal((3, n))
    th = ok.Theta(rng.uniform(0.8, 1.2, d) * np.sqrt(d), 1.1, 1e-2, ok.MATERN52)
    got = host(gp.kmm(_gk(th), dev(X), dev(V), precision="bf16x3"))
    ref = ok.khat_matmul(X, th, V.T).T
    off = ref - (1.1 + 1e-2) * V
    assert np.linalg.norm(got - ref) <= 5e-5 * np.linalg.norm(off)


@pytest.mark.parametrize("n", [1, 63, 64, 65, 4097, 32768, 32769, 270000])
def test_pivoted_cholesky_at_the_edges_of_its_row_blocks(n):
    """64 rows to a workgroup up to n = 32,768, 256 beyond, 512 at n = 270,000.  The columns against the oracle's on the
    same pivots, each of which attains the largest residual diagonal; bars as for the pivoted Cholesky elsewhere."""
    from oracle.pivchol import pivoted_cholesky
    from paper_2109_09817_amd import gp
    rng = np.random.default_rng(n)
    X = rng.standard_normal((n, 4))
    th = ok.Theta(np.full(4, 1.5), 1.3, 1e-2, ok.MATERN52)
    k = min(n, 6)
    pc = gp.pivchol(_gk(th), dev(X), k)
    assert pc.rank == k
    piv = [int(p) for p in pc.pivots[:k]]
    Lo, _, _ = pivoted_cholesky(X, th, k, pivots=piv)
    np.testing.assert_allclose(host(pc.L).T, Lo, rtol=0, atol=1e-10)
    delta = np.full(n, th.sf)
    for m in range(k):
        assert delta[piv[m]] >= delta.max() - 1e-12 * th.sf
        delta -= Lo[:, m] ** 2


@pytest.mark.parametrize("n,prec", [(1, "bf16x3"), (255, "fp32"), (257, "bf16x3"), (257, "fp64"), (1500, "fp64"),
                                    (270000, "bf16x3")])
def test_first_step_size_from_the_products_own_dot(n, prec):
    """One iteration without a preconditioner: U = alpha B with alpha = B.B / B.(K B) per column, the dot added where the
    product is written (512 rows to a workgroup at n = 270,000).  Against gp.kmm and numpy: sums of n positive and
    negative terms in FP64, cancelling little here (K is diagonally dominated): bar 1e-11."""
    from paper_2109_09817_amd import gp
    rng = np.random.default_rng(n)
    X, B = rng.standard_normal((n, 6)), rng.standard_normal((3, n))
    B[2] = 0.0  # never active
    th = ok.Theta(np.full(6, 0.5), 1.0, 1.0, ok.MATERN52)
    kern = _gk(th)
    r = gp.mbcg(kern, dev(X), dev(B), 1, 0.0, precision=prec)
    KB = host(gp.kmm(kern, dev(X), dev(B), precision=prec))
    U = host(r.U)
    for c in range(2):
        alpha = (B[c] @ B[c]) / (B[c] @ KB[c])
        assert np.linalg.norm(U[c] - alpha * B[c]) <= 1e-11 * np.linalg.norm(alpha * B[c])
    assert not U[2].any()


@pytest.mark.parametrize("prec,bar", [("bf16x3", 5e-5), ("fp32", 1e-5)])
@pytest.mark.parametrize("d", [5, 21, 32, 48, 64, 100])
@pytest.mark.parametrize("t", [1, 17, 33, 50])
def test_square_product_at_every_width_of_the_sweeps(d, t, prec, bar):
    """One to four 16-column blocks at each K step count: rows per wave, the diagonal's chunk and the columns stored
    differ.  Off-diagonal part against the oracle; bars of the forms (5e-5, 1e-5) on a correlated kernel."""
    from paper_2109_09817_amd import gp
    n = 1003
    rng = np.random.default_rng(100 * d + t)
    X, V = rng.standard_normal((n, d)), rng.standard_normal((t, n))
    th = ok.Theta(rng.uniform(0.8, 1.2, d) * np.sqrt(d), 1.1, 1e-2, ok.MATERN52)
    got = host(gp.kmm(_gk(th), dev(X), dev(V), precision=prec))
    ref = ok.khat_matmul(X, th, V.T).T
    off = ref - (1.1 + 1e-2) * V
    assert np.linalg.norm(got - ref) <= bar * np.linalg.norm(off)


@pytest.mark.parametrize("prec,bar", [("bf16x3", 5e-5), ("fp32", 1e-5)])
@pytest.mark.parametrize("n,m", [(30001, 0), (9001, 1200)])
def test_products_with_one_and_several_windows_per_split(n, m, prec, bar):
    """n = 30,001: splits of several FP32 windows, partials in FP64; a cross product's splits are single windows, stored
    in FP32.  Against the FP64 form; bars as above."""
    from paper_2109_09817_amd import gp
    rng = np.random.default_rng(n)
    X, V = dev(rng.standard_normal((n, 21))), dev(rng.standard_normal((35, n)))
    Z = dev(rng.standard_normal((m, 21))) if m else None
    th = ok.Theta(np.full(21, 5.0), 1.1, 1e-2, ok.RBF)
    got = host(gp.kmm(_gk(th), X, V, Z=Z, precision=prec))
    ref = host(gp.kmm(_gk(th), X, V, Z=Z, precision="fp64"))
    off = ref - (0.0 if m else (1.1 + 1e-2) * host(V))
    assert np.linalg.norm(got - ref) <= bar * np.linalg.norm(off)


@pytest.mark.parametrize("n,m,t", [(3000, 1, 1), (3000, 17, 16), (2999, 33, 17), (3000, 64, 48), (3000, 65, 49),
                                   (3000, 130, 80), (3000, 40, 81), (3000, 97, 144), (3000, 16, 145), (3000, 66, 208),
                                   (3000, 50, 209), (3000, 80, 257), (3000, 31, 272), (3000, 100, 273),
                                   (2001, 48, 320), (300001, 40, 20)])
def test_wide_cross_product_at_its_column_forms(n, m, t):
    """Column blocks per wave and left over, query rows that leave row blocks empty, and splits of several windows
    (n = 300,001).  Against the FP64 form; the mixed form's bar, 5e-5."""
    from paper_2109_09817_amd import gp
    rng = np.random.default_rng(n + t)
    d = (5, 32, 48, 64)[t % 4]
    X, V = dev(rng.standard_normal((n, d))), dev(rng.standard_normal((t, n)))
    Z = dev(rng.standard_normal((m, d)))
    kern = _gk(ok.Theta(np.full(d, 3.0), 1.1, 1e-2, ok.MATERN52 if t % 2 else ok.RBF))
    got = host(gp.kmm(kern, X, V, Z=Z, precision="bf16x3"))
    ref = host(gp.kmm(kern, X, V, Z=Z, precision="fp64"))
    assert np.linalg.norm(got - ref) <= 5e-5 * np.linalg.norm(ref)


@pytest.mark.parametrize("n,r", [(700, 1), (5001, 127), (9000, 128), (5000, 129), (20011, 300), (1600, 1500)])
def test_large_rank_factor_with_its_gram_split(n, r):
    """F F^T with k split over workgroups (one to 78 tiles, ragged runs of k).  E against numpy; rounding is amplified
    by cond(K_MM + delta I), below 1e4 on this data: bar 1e-11."""
    import scipy.linalg as sl
    from paper_2109_09817_amd import gp
    rng = np.random.default_rng(n + r)
    X = rng.standard_normal((n, 6))
    th = ok.Theta(rng.uniform(0.3, 0.6, 6), 1.0, 1e-2, ok.MATERN52)
    M = np.sort(rng.choice(n, r, replace=False))
    E = host(gp.nystrom_chol_precond(_gk(th), dev(X), M).E)
    KMX = ok.kernel(X[M], X, th)
    KMM = KMX[:, M] + 1e-10 * r * np.eye(r)
    assert np.linalg.cond(KMM) < 1e4
    F = sl.solve_triangular(np.linalg.cholesky(KMM), KMX, lower=True)
    ref = sl.solve_triangular(np.linalg.cholesky(F @ F.T + 1e-2 * np.eye(r)), F, lower=True)
    assert np.linalg.norm(E - ref) <= 1e-11 * np.linalg.norm(ref)


@pytest.mark.parametrize("n", [256, 257, 320, 511, 513, 769, 1100, 3000])
def test_cholesky_with_its_trailing_update_beside_the_diagonal_blocks(n):
    """K_hat^{-1} y around the 256-wide super-panels (no, one and several shares of tiles, ragged last panels; n = 3,000:
    more than one launch of them).  Residual of K_hat omega = y in FP64: relative bar 1e-11 at cond(K_hat) below 1e4."""
    from paper_2109_09817_amd import gp
    rng = np.random.default_rng(n)
    X, y = rng.standard_normal((n, 5)), rng.standard_normal(n)
    th = ok.Theta(rng.uniform(0.5, 1.0, 5), 1.2, 0.1, ok.MATERN52)
    r = gp.exact_mll_and_grad(_gk(th), dev(X), dev(y), with_grad=False, with_omega=True)
    back = ok.khat_matmul(X, th, host(r.omega)[:, None])[:, 0]
    assert np.linalg.norm(back - y) <= 1e-11 * np.linalg.norm(y)


@pytest.mark.parametrize("n,m,d,t", [(1, 3, 5, 2), (4096, 0, 32, 9), (4097, 0, 33, 3), (4096, 33, 17, 20),
                                     (4353, 300, 64, 1), (4000, 31, 100, 65)])
def test_mixed_product_with_its_operands_prepared_together(n, m, d, t):
    """The centre from up to 16 blocks of 256 rows is added where the points are prepared, from more before; X, Z and V
    in one launch.  Data shifted by 100 lengthscales: a wrong centre loses all digits.  Against the oracle; 5e-5."""
    from paper_2109_09817_amd import gp
    rng = np.random.default_rng(n + t)
    X, V = rng.standard_normal((n, d)) + 100.0, rng.standard_normal((t, n))
    Z = rng.standard_normal((m, d)) + 100.0 if m else None
    th = ok.Theta(rng.uniform(0.8, 1.2, d) * np.sqrt(d), 1.1, 1e-2, ok.MATERN52)
    got = host(gp.kmm(_gk(th), dev(X), dev(V), Z=dev(Z) if m else None, precision="bf16x3"))
    ref = ok.cross_matmul(Z, X, th, V.T).T if m else ok.khat_matmul(X, th, V.T).T
    off = ref - (0.0 if m else (1.1 + 1e-2) * V)
    assert np.linalg.norm(got - ref) <= 5e-5 * np.linalg.norm(off)
