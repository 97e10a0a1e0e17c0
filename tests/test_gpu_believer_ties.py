"""The believer where many candidates score alike, so that what can still win is
most of the pool: pools far from every observation (second lists of both
lengths' forms), scores that are all zero, and scores that one pick lowers
everywhere.  Picks against the oracle's full refit along the same sequence, two
calls alike (the order in which a list fills differs from call to call), and a
call never much longer than the same call without ties."""
import time

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2408_04323_amd as S  # noqa: E402
from oracle.believer import kriging_believer  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _problem(m, d, p, seed):
    rng = np.random.default_rng(seed)
    X = rng.random((m, d))
    Y = np.stack([np.sin(4 * X[:, 0]) + X[:, -1] ** 2, np.cos(3 * X[:, 0]) - X[:, -1], X.sum(1)], 1)[:, :p]
    return rng, X, (Y - Y.mean(0)) / Y.std(0)


# p, n, m, d, lengthscale, shift: raised observations make the far field the best region
CASES = [(2, 150001, 24, 2, 0.02, 3.0), (2, 30000, 24, 2, 0.02, 3.0), (2, 150001, 24, 2, 0.02, 0.0),
         (1, 90000, 40, 3, 0.05, 0.0), (3, 70000, 20, 4, 0.03, 2.0), (2, 150001, 20, 2, 3.0, 0.0)]


@pytest.mark.parametrize("p,n,m,d,ls,shift", CASES)
def test_believer_ties(p, n, m, d, ls, shift):
    print("[case] believer ties", p, n, m, d, ls, shift, flush=True)
    rng, X, Y = _problem(m, d, p, n)
    Y = Y + shift
    ref, q = Y.max(0) + 0.1 * np.ptp(Y, 0), 10
    hyp = [dict(lengthscale=np.full(d, ls), signal_var=1.0, noise_var=1e-2, prior_mean=0.0, kernel="matern52",
                warp=None) for _ in range(p)]
    gps = [S.gp_fit(X, Y[:, j], h["lengthscale"], 1.0, 1e-2) for j, h in enumerate(hyp)]
    Xc = rng.random((n, d)).astype(np.float32)
    pool = torch.from_numpy(Xc).to(DEV)
    picks, acq = S.suggest_kb(gps, None, pool, q, Y, ref)
    again, acq2 = S.suggest_kb(gps, None, pool, q, Y, ref)
    np.testing.assert_array_equal(picks, again)
    np.testing.assert_array_equal(acq, acq2)
    assert len(set(picks.tolist())) == q
    steps = []
    kriging_believer(X, Y, hyp, Xc, np.ones(n), ref, q, follow=picks, record=steps)
    for i, a, (acq_o, elig) in zip(picks, acq, steps):
        best = acq_o[elig].max()
        assert elig[i] and acq_o[i] >= best - 2e-3 * best, (i, acq_o[i], best)
        assert abs(a - acq_o[i]) <= 1e-3 * best


def test_believer_all_zero():
    _, X, Y = _problem(30, 3, 2, 1)
    gps = [S.gp_fit(X, Y[:, j], np.full(3, 0.5), 1.0, 1e-2) for j in range(2)]
    pool = torch.rand((100003, 3), generator=torch.Generator().manual_seed(1)).to(DEV)
    picks, acq = S.suggest_kb(gps, None, pool, 6, Y, Y.min(0) - 1000.0)
    np.testing.assert_array_equal(picks, np.arange(6))
    assert np.all(acq == 0)


def test_believer_ties_take_no_longer():
    """Scoring every candidate again for every pick takes about three times the ordinary call here."""
    n, m, d, q = 1 << 18, 256, 10, 8
    rng, X, Y = _problem(m, d, 2, 4)
    pool = torch.tensor(rng.random((n, d), dtype=np.float32), device=DEV)

    def ms(ls, ref):
        gps = [S.gp_fit(X, Y[:, j], np.full(d, ls), 1.0, 1e-2) for j in range(2)]
        ws = torch.empty(S.suggest_kb_workspace(gps, n, q), dtype=torch.uint8, device=DEV)
        best = np.inf
        for _ in range(6):
            torch.cuda.synchronize()
            t = time.perf_counter()
            S.suggest_kb(gps, None, pool, q, Y, ref, workspace=ws)
            best = min(best, time.perf_counter() - t)
        return best * 1e3

    usual = ms(0.6, Y.max(0) + 0.2)
    for what, ls, ref in (("all zero", 0.6, Y.min(0) - 1000.0), ("far field", 0.02, Y.max(0) + 0.2)):
        took = ms(ls, ref)
        print("[case] believer", what, took, "ms, usual", usual, flush=True)
        assert took <= 2 * usual
