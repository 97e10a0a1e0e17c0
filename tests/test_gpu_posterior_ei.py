"""EI made by the posterior's own launch, where a workgroup has one tile and
where it has several: that of the means and deviations it has written."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2408_04323_amd as S  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,eps", [("f32", 2.0 ** -24), ("f64", 2.0 ** -53)])
@pytest.mark.parametrize("m", [5, 129, 300])
@pytest.mark.parametrize("n", [1, 31, 33, 64, 65, 8193, 300001])
def test_ei_beside_the_posterior(n, m, dtype, eps):
    print("[case] posterior ei", n, m, dtype, flush=True)
    rng = np.random.default_rng(m)
    X, y = rng.random((m, 4)), rng.standard_normal(m)
    gp = S.gp_fit(X, y, np.full(4, 0.4), 1.0, 1e-2, dtype=dtype)
    pool = torch.tensor(np.random.default_rng(n).random((n, 4), dtype=np.float32), device="cuda:0")
    best, xi = float(y.min()), 1e-4
    b = S.score_pool([gp], None, pool, 1, best_y=best, xi=xi)
    want = S.acq_ei(b.mu[0].double(), b.sigma[0].double(), best, xi)
    torch.cuda.synchronize()
    # The same formula in double from the same values, good to 8e-16 of itself either way (16 eps between two), and
    # rounded once; two of u = (c - mu) / sd lie up to two ulps apart, each of which moves it by u^2 + 1 ulps at most;
    # below the type's smallest normal number nothing is left.
    u = (best + xi - b.mu[0].double()) / b.sigma[0].double()
    tiny = 2.0 ** -126 if dtype == "f32" else 2.0 ** -1022
    assert bool(((b.acq.double() - want).abs() <= (2 * eps + 2.0 ** -53 * (20 + 4 * u * u)) * want + tiny).all())
