"""The device factorization at the edges of its schedule, against the oracle:
one block, two, three; a worker's share that just fits its registers (m = 256)
and one that does not (257, 289); partly filled last blocks; and a pivot that
fails early, late or in the last block, which is reported as NOT_PD (never as
a wait that ran out) and leaves the next evaluation sound."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2408_04323_amd as S  # noqa: E402
from oracle.mle import nll_and_grad  # noqa: E402

pytestmark = pytest.mark.gpu
D = 12


def _case(m):
    rng = np.random.default_rng(m)
    X, y = rng.random((m, D)), rng.standard_normal(m)
    return X, y, np.log(np.concatenate([rng.uniform(0.2, 0.6, D), [1.3, 0.02]]))


def _check(m):
    X, y, theta = _case(m)
    nll, g = S.gp_nll_device(X, y, theta)
    nll_o, g_o = nll_and_grad(theta, X, y, "matern52")
    # 1e-10 and 1e-8: m eps times K's condition number (below 1e4 with this noise), with room
    assert nll == pytest.approx(nll_o, rel=1e-10, abs=1e-10)
    np.testing.assert_allclose(g, g_o, rtol=1e-8, atol=1e-8)


@pytest.mark.parametrize("m", [2, 16, 32, 33, 48, 49, 97, 112, 240, 241, 257, 272, 289, 560])
def test_factor_sizes(m):
    print("[case] factor", m, flush=True)
    _check(m)


@pytest.mark.parametrize("m,bad", [(16, 3), (33, 32), (273, 1), (273, 18), (273, 130), (273, 272), (576, 575)])
def test_factor_reports_a_failing_pivot(m, bad):
    print("[case] pivot", m, bad, flush=True)
    X, y, theta = _case(m)
    X[bad] = X[0]  # the same observation twice, and no noise
    theta[-1] = -60.0
    with pytest.raises(S.ScootError) as e:
        S.gp_nll_device(X, y, theta)
    assert e.value.status == -2
    _check(m)
