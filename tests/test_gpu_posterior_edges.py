"""The fp32 posterior at the edges of its layouts: observation counts around
the 16-observation blocks, the 32-row blocks and the limits at which another
number of waves shares a tile's rows (128, 256 and 512), pools around the
64-candidate tile, every step count of the distance chain, and both ways to a
handle (packed on the host, packed on the device from its factorization).

Bounds: a K* entry is within 8 eps of itself (square root, exponential and
three operations in fp32, eps = 2^-24 relative each, doubled), the products
behind it are exact to that order, so |d mu| <= 8 eps sum |k alpha| and
|d sigma^2| <= 2 |v| 8 eps | |L^-1| k | , each doubled for the accumulation,
plus the rounding of the results."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2408_04323_amd as S  # noqa: E402
from oracle.gp import gp_fit as oracle_fit, gp_posterior, matern52  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
EPS = 2.0 ** -24

CASES = [(1, 1, 1), (2, 63, 2), (15, 64, 3), (16, 65, 6), (17, 129, 7), (31, 5, 10), (32, 64, 11), (33, 190, 14),
         (127, 70, 15), (128, 641, 16), (129, 100, 4), (255, 66, 9), (256, 300, 10), (257, 130, 12), (383, 64, 8),
         (511, 90, 5), (512, 200, 12), (513, 65, 13), (543, 64, 2), (576, 333, 16)]


@pytest.mark.parametrize("m,n,d", CASES, ids=[f"m{c[0]}-n{c[1]}-d{c[2]}" for c in CASES])
def test_posterior_edges(m, n, d):
    print("[case] posterior edges", m, n, d, flush=True)
    rng = np.random.default_rng(1000 * m + d)
    X, y = rng.random((m, d)), rng.standard_normal(m)
    ls, s2, tau2 = rng.uniform(0.3, 1.5, d), 1.3, 1e-2
    Xc = rng.random((n, d)).astype(np.float32)
    mu, sd = gp_posterior(oracle_fit(X, y, ls, s2, tau2, 0.0), Xc.astype(np.float64))
    k = matern52(X, Xc.astype(np.float64), ls, s2)
    Li = np.linalg.inv(np.linalg.cholesky(matern52(X, X, ls, s2) + tau2 * np.eye(m)))
    alpha = Li.T @ (Li @ y)
    v = Li @ k
    b_mu = 2 * 8 * EPS * (np.abs(k) * np.abs(alpha)[:, None]).sum(0) + 2 * EPS * np.abs(mu)
    b_var = 2 * 2 * 8 * EPS * np.linalg.norm(v, axis=0) * np.linalg.norm(np.abs(Li) @ k, axis=0) + 4 * EPS * s2
    pool = torch.from_numpy(Xc).to(DEV)
    for how in (S.gp_fit, S.gp_fit_device):
        gp = how(X, y, ls, s2, tau2)
        got_mu, got_sd = (t.cpu().numpy().astype(np.float64) for t in S.posterior(gp, pool))
        gp.close()
        assert np.all(np.abs(got_mu - mu) <= b_mu), np.max(np.abs(got_mu - mu) / b_mu)
        err = np.abs(got_sd ** 2 - sd ** 2)
        assert np.all(err <= b_var + 2 * EPS * sd ** 2), np.max(err / b_var)
