"""The believer's two ways to a pick: small pools are scored whole, of large ones
only what can still win.  A large pool, of which all but a few thousand
candidates are not admissible, gives the picks, the scores and the posterior of
those few by themselves."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2408_04323_amd as S  # noqa: E402

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _line(p, m, q):
    """The largest pool that is scored whole."""
    return ((72 + 5 * q // 2) << 20) // (p * ((m + 15) // 16 * 16 + 64))


# kind: distinct candidates; a coarse grid, on which many score alike; one candidate over and over; no score above zero
@pytest.mark.parametrize("kind,few", [("distinct", 3000), ("grid", 60000), ("equal", 30000), ("zero", 20000)])
@pytest.mark.parametrize("p,m,q,d,kernel,warped", [(1, 33, 2, 9, "matern52", False), (2, 130, 9, 6, "matern32", False),
                                                   (2, 200, 10, 3, "matern52", True), (3, 64, 18, 14, "matern52", False),
                                                   (2, 48, 30, 16, "matern32", False)])
def test_large_pools_pick_as_small_ones(p, m, q, d, kernel, warped, kind, few):
    n = _line(p, m, q) + 1
    print("[case] believer routes", p, m, q, d, kind, n, flush=True)
    rng = np.random.default_rng(1000 * m + q)
    X = rng.random((m, d))
    Y = np.sin(3 * X @ rng.standard_normal((d, p))) + 0.05 * rng.standard_normal((m, p))
    ref = Y.max(0) + 0.1 * (Y.max(0) - Y.min(0))
    if kind == "zero":
        ref = Y.min(0) - 100.0  # nothing improves on it
    ab = (rng.uniform(0.6, 1.6, d), rng.uniform(0.6, 1.6, d)) if warped else (None, None)
    ls = rng.uniform(0.3, 1.2, d) * np.sqrt(d / 3)
    gps = [S.gp_fit(X, Y[:, j], ls, 1.2, 1e-2, kernel=kernel, warp_a=ab[0], warp_b=ab[1]) for j in range(p)]
    pool = torch.rand((n, d), device=DEV, generator=torch.Generator(DEV).manual_seed(q))
    if kind == "grid":
        pool[:, :2] = (pool[:, :2] * 3).round() / 3
        pool[:, 2:] = 0.5
    elif kind == "equal":
        pool[:] = 0.3
    at = torch.from_numpy(np.sort(rng.choice(n, few, replace=False))).to(DEV)
    known = torch.zeros(n, dtype=torch.uint8, device=DEV)
    known[at] = 1
    mu, sd = torch.empty((p, n), device=DEV), torch.empty((p, n), device=DEV)
    picks, acq = S.suggest_kb(gps, None, pool, q, Y, ref, known=known, mu_out=mu, sigma_out=sd)
    mu1, sd1 = torch.empty((p, few), device=DEV), torch.empty((p, few), device=DEV)
    want, want_acq = S.suggest_kb(gps, None, pool[at].contiguous(), q, Y, ref, mu_out=mu1, sigma_out=sd1)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(picks, at.cpu().numpy()[want])
    # sigma^2 by other orders of rounding to float, in the scores to a power of |u| below ten
    np.testing.assert_allclose(acq, want_acq, rtol=1e-4, atol=1e-12)
    assert float((mu[:, at] - mu1).abs().max()) < 1e-5
    assert float((sd[:, at] - sd1).abs().max()) < 1e-5
