"""The Kriging believer where its rounds can go wrong: one and three
objectives, more picks than one pass over the observations takes (8 and 16),
pools smaller than the selection's list or than q, warped inputs, and a pool
of equal candidates, where every bound ties and the list outgrows what is
scored without waiting for its length.

Every pick is checked against the oracle's full refit along the same sequence:
within the acquisition's fp32 bar (1e-3 of the step's best) of the best
eligible candidate, and the last round's posterior within the fp32 bars."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2408_04323_amd as S  # noqa: E402
from oracle.believer import kriging_believer  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TINY = 2.0 ** -126  # scores below the smallest normal float may come out as zero

# p, n, m, q, d, kernel, warped
CASES = [(1, 50, 20, 20, 5, "matern52", False), (3, 700, 60, 5, 7, "matern52", False),
         (2, 40, 33, 40, 4, "matern52", False), (2, 30, 40, 64, 6, "matern32", False),
         (2, 900, 129, 18, 9, "matern32", True), (2, 3, 5, 3, 2, "matern52", False)]


@pytest.mark.parametrize("p,n,m,q,d,kernel,warped", CASES, ids=[f"p{c[0]}-n{c[1]}-m{c[2]}-q{c[3]}" for c in CASES])
def test_believer_edges(p, n, m, q, d, kernel, warped):
    print("[case] believer edges", p, n, m, q, flush=True)
    rng = np.random.default_rng(100 * n + q)
    X, Xc = rng.random((m, d)), rng.random((n, d)).astype(np.float32)
    w = rng.standard_normal((d, p))
    Y = np.sin(3 * X @ w) + 0.05 * rng.standard_normal((m, p))
    ref = Y.max(0) + 0.1 * (Y.max(0) - Y.min(0))
    hyp, gps = [], []
    for j in range(p):
        ab = (rng.uniform(0.6, 1.6, d), rng.uniform(0.6, 1.6, d)) if warped else None
        h = dict(lengthscale=rng.uniform(0.3, 1.2, d), signal_var=1.2, noise_var=1e-2, prior_mean=0.0, kernel=kernel,
                 warp=ab)
        hyp.append(h)
        gps.append(S.gp_fit(X, Y[:, j], h["lengthscale"], 1.2, 1e-2, kernel=kernel, warp_a=ab and ab[0],
                            warp_b=ab and ab[1]))
    ws = torch.empty(S.suggest_kb_workspace(gps, n, q), dtype=torch.uint8, device=DEV)
    mu = torch.empty((p, n), device=DEV)
    sd = torch.empty((p, n), device=DEV)
    pool = torch.from_numpy(Xc).to(DEV)
    picks, acq = S.suggest_kb(gps, None, pool, q, Y, ref, workspace=ws, mu_out=mu, sigma_out=sd)
    again, _ = S.suggest_kb(gps, None, pool, q, Y, ref)
    np.testing.assert_array_equal(picks, again)
    assert len(picks) == min(n, q) and len(set(picks.tolist())) == len(picks)
    steps = []
    _, _, mu_o, sd_o = kriging_believer(X, Y, hyp, Xc, np.ones(n), ref, len(picks), follow=picks, record=steps)
    for i, a, (acq_o, elig) in zip(picks, acq, steps):
        best = acq_o[elig].max()
        assert elig[i] and acq_o[i] >= best - 2e-3 * best - TINY, (i, acq_o[i], best)
        assert abs(a - acq_o[i]) <= 1e-3 * max(best, acq_o[i]) + TINY
    if len(picks) == q:  # the oracle's last posterior is the last scoring round's
        for j in range(p):
            assert np.all(np.abs(mu[j].cpu().numpy() - mu_o[:, j]) <= 1e-4 * np.abs(mu_o[:, j]).max())
            assert np.all(np.abs(sd[j].cpu().numpy() - sd_o[:, j]) <= 1e-3 * np.sqrt(1.2))


def test_believer_equal_candidates():
    n, q, d = 40000, 5, 3
    print("[case] believer equal candidates", n, flush=True)
    rng = np.random.default_rng(3)
    X, Y = rng.random((30, d)), rng.standard_normal((30, 2))
    gps = [S.gp_fit(X, Y[:, j], np.full(d, 0.5), 1.0, 1e-2) for j in range(2)]
    pool = torch.full((n, d), 0.3, device=DEV)
    picks, acq = S.suggest_kb(gps, None, pool, q, Y, Y.max(0) + 0.5)
    np.testing.assert_array_equal(picks, np.arange(q))
    assert np.all(np.diff(acq) <= 0)
