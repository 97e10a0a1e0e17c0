"""fp32 accuracy of the fp32 posterior in every form of its kernel (tiles of 32
and of 64 candidates, four and two waves per tile, every number of slots): the
variance and the mean against 64 bits within a limit that no form with a part
product lost or misplaced can meet (split_bound.py)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2408_04323_amd as S  # noqa: E402
from oracle.gp import matern52  # noqa: E402
from split_bound import LIMIT, factor, measure, problem, units  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

HALVES, FOUR, TWO = 256 * 32, 256 * 32 + 1, 7 * 256 * 64 + 1  # pools: the first form's last size, the others' first


@pytest.mark.parametrize("n", [HALVES, FOUR, TWO])
@pytest.mark.parametrize("m,d", [(32, 10), (100, 16), (128, 2), (129, 10), (256, 10), (250, 14), (193, 16), (257, 10),
                                 (512, 12), (385, 16), (576, 6), (543, 16)])
def test_six_part_products(m, d, n):
    print("[case] posterior accuracy", m, d, n, flush=True)
    X, y, ls, tau2 = problem(m, d)
    pool = np.random.default_rng(n).random((n, d)).astype(np.float32)
    at = np.unique(np.concatenate([np.arange(0, n, n // 1500), [n - 1]]))  # every lane and half of a tile
    Li, alpha = factor(X, y, ls, tau2)
    k = matern52(X, pool[at].astype(np.float64), ls, 1.0)
    u_q, u_mu = units(Li, alpha, k)
    q, mean = ((Li @ k) ** 2).sum(0), alpha @ k
    gp = S.gp_fit(X, y, ls, 1.0, tau2)
    mu, sd = (t.cpu().numpy()[at].astype(np.float64) for t in S.posterior(gp, torch.from_numpy(pool).to(DEV)))
    m_q, m_mu = measure((1.0 - sd * sd) - q, u_q, 2 * q), measure(mu - mean, u_mu, mean)
    print(f"[measure] {m_q:.2f} {m_mu:.2f}", flush=True)
    assert m_q < LIMIT and m_mu < LIMIT
