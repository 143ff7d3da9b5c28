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


@pytest.mark.parametrize("n", [15, 16, 17, 33, 47, 49, 81])
def test_exact_gp_at_the_edges_of_the_16_wide_diagonal_steps(n):
    """Diagonal blocks are factored in 16-column steps; the bars are those of the dense parity cases
    (1e-10, well above 1e-14 kappa here)."""
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
