"""NaN and infinities through the kernels: what plain arithmetic would make NaN is never a finite number, and what it
leaves infinite or finite stays so."""
import numpy as np
import pytest

import oracle.kernel as ok
from _helpers import dev, host

pytestmark = pytest.mark.gpu


def _gk(th):
    from paper_2109_09817_amd import gp
    return gp.Kernel(th.ell, th.sf, th.noise, "matern52" if th.kind == ok.MATERN52 else "rbf")


def _fp64(th, X, V, Z=None):
    from paper_2109_09817_amd import gp
    return host(gp.kmm(_gk(th), dev(X), dev(V), Z=None if Z is None else dev(Z), precision="fp64"))


@pytest.mark.parametrize("kind", [ok.MATERN52, ok.RBF])
@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf, 1e200])
@pytest.mark.parametrize("n,d,t", [(40, 5, 3), (300, 17, 20), (2000, 48, 50)])
def test_fp64_product_with_a_coordinate_that_has_no_distance(n, d, t, bad, kind):
    """A NaN or infinite coordinate, or one whose square overflows, has no distance to the others: every product that
    involves the point is NaN (one split of the points and several, columns in blocks and left over, the bad point
    first, inside and last).  A query row touches its own result only, the others keep their bits."""
    rng = np.random.default_rng(n)
    X, V, Z = rng.standard_normal((n, d)), rng.standard_normal((t, n)), rng.standard_normal((70, d))
    th = ok.Theta(rng.uniform(1.0, 2.0, d) * np.sqrt(d), 1.2, 1e-3, kind)
    good = _fp64(th, X, V, Z)
    assert np.all(np.isfinite(good))
    for p in (0, n // 2 + 1, n - 1):
        Xb = X.copy()
        Xb[p, d // 2] = bad
        assert np.all(np.isnan(_fp64(th, Xb, V)))
        assert np.all(np.isnan(_fp64(th, Xb, V, Z)))
    for r in (0, 37, 69):
        Zb = Z.copy()
        Zb[r, 0] = bad
        got = _fp64(th, X, V, Zb)
        assert np.all(np.isnan(got[:, r]))
        keep = np.arange(70) != r
        np.testing.assert_array_equal(got[:, keep], good[:, keep])


def test_fp64_solve_on_a_nan_coordinate_stops():
    from paper_2109_09817_amd import _lib, gp
    rng = np.random.default_rng(0)
    X, B = rng.standard_normal((500, 6)), rng.standard_normal((3, 500))
    X[123, 2] = np.nan
    k = gp.Kernel(np.full(6, 3.0), 1.0, 1e-2)
    with pytest.raises(_lib.GpError) as e:
        gp.mbcg(k, dev(X), dev(B), 50, 1e-6, precision="fp64")
    assert e.value.code == _lib.GP_ENONFINITE


@pytest.mark.parametrize("prec", ["fp64", "bf16x3", "fp32"])
def test_square_product_of_one_point_is_its_exact_diagonal(prec):
    """No pair, no distance: (s_f + sigma^2) V whatever the coordinates hold."""
    from paper_2109_09817_amd import gp
    V = np.array([[3.0], [-0.5]])
    k = gp.Kernel(np.ones(2), 1.25, 0.5)
    for x in (1.0, 1e200):
        got = host(gp.kmm(k, dev(np.array([[x, 2.0]])), dev(V), precision=prec))
        np.testing.assert_array_equal(got, 1.75 * V)


@pytest.mark.parametrize("r", [1, 5, 16, 63, 100])
@pytest.mark.parametrize("s", [1, 20, 64])
def test_tall_product_keeps_infinities(r, s):
    """sigma^{-1} V + Z^T diag(g) Z V with Z > 0 > g and one entry of V infinite: that column is -inf, NaN where +inf meets
    -inf, and the other columns keep their bits, however the r terms are padded."""
    from paper_2109_09817_amd import gp
    n, i0 = 150, 77
    rng = np.random.default_rng(r + s)
    Z, g, V = rng.uniform(0.5, 1.0, (r, n)), -rng.uniform(0.5, 1.0, r), rng.standard_normal((s, n))
    pc = gp.Nystrom(dev(Z), dev(g), np.arange(r), 0.25)
    ref = host(gp.nystrom_apply(pc, dev(V)))
    V[s // 2, i0] = np.inf
    ref[s // 2] = -np.inf
    ref[s // 2, i0] = np.nan
    np.testing.assert_array_equal(host(gp.nystrom_apply(pc, dev(V))), ref)
