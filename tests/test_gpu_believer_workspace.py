"""The believer's workspace: the size that is reported is what the parts take,
the call stays inside it wherever it starts, and a smaller one is refused."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2408_04323_amd as S  # noqa: E402

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
GUARD = 4096


# n: pools scored whole at every pick, by the narrow and the wide kernel, which keep a row per pick; larger ones,
# which keep none, eight or sixteen rows
@pytest.mark.parametrize("offset", [0, 4, 1])
@pytest.mark.parametrize("n,q,warped", [(5, 3, False), (300, 9, False), (300, 64, True), (70001, 10, False),
                                        (1048579, 9, False), (1048579, 10, False),
                                        (1048579, 18, True)])
def test_reported_size_is_what_the_call_uses(n, q, warped, offset):
    print("[case] believer workspace", n, q, warped, offset, flush=True)
    d, p, m = 3, 2, 40
    rng = np.random.default_rng(n + q)
    X, Y = rng.random((m, d)), rng.standard_normal((m, p))
    ab = np.full(d, 1.3) if warped else None
    gps = [S.gp_fit(X, Y[:, j], np.full(d, 0.4), 1.0, 1e-2, warp_a=ab, warp_b=ab) for j in range(p)]
    pool = torch.from_numpy(rng.random((n, d)).astype(np.float32)).to(DEV)
    ref = Y.max(0) + 0.2
    size = S.suggest_kb_workspace(gps, n, q)
    # per candidate; the rows; the factors of q picks; rounding to 256 bytes
    rows = q - 1 if n < 100000 else (q - 2) // 8 * 8
    most = n * (16 * p + 17 + 4 * p * rows + (4 * d * p if warped else 0))
    small = p * (q + 1) * 64 * 8 + p * q * q * 8 + 8 * q
    assert size <= most + small + 32 * 256 + 32 * p * 8
    raw = torch.full((offset + size + GUARD,), 0xA5, dtype=torch.uint8, device=DEV)
    ws = raw[offset:offset + size]
    mu, sd = torch.empty((p, n), device=DEV), torch.empty((p, n), device=DEV)
    picks, acq = S.suggest_kb(gps, None, pool, q, Y, ref, workspace=ws, mu_out=mu, sigma_out=sd)
    mu2, sd2 = torch.empty((p, n), device=DEV), torch.empty((p, n), device=DEV)
    want, want_acq = S.suggest_kb(gps, None, pool, q, Y, ref, mu_out=mu2, sigma_out=sd2)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(picks, want)
    np.testing.assert_array_equal(acq, want_acq)
    assert torch.equal(mu, mu2) and torch.equal(sd, sd2)
    assert bool((raw[:offset] == 0xA5).all()) and bool((raw[offset + size:] == 0xA5).all())
    with pytest.raises(Exception, match="workspace too small"):
        S.suggest_kb(gps, None, pool, q, Y, ref, workspace=ws[:size - 1])
