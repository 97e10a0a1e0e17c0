"""The fp64 normal partial expectation behind EI and EHVI: EI against 60-digit
arithmetic over the whole range of u = (best + xi - mu) / sigma, from where the
density underflows to where it no longer matters, either side of every end of
the approximation, and at the special values."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
mp = pytest.importorskip("mpmath")

import paper_2408_04323_amd as S  # noqa: E402

pytestmark = pytest.mark.gpu


def _ei(mu, sd, best, dtype):
    out = S.acq_ei(torch.tensor(mu, dtype=dtype, device="cuda:0"), torch.tensor(sd, dtype=dtype, device="cuda:0"),
                   best, xi=0.0)
    torch.cuda.synchronize()
    return out.cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("lo,hi", [(-37.0, -20.0), (-20.0, -5.5), (-5.5, -4.5), (-4.5, -1.0), (-1.0, 1.0), (1.0, 6.0),
                                   (6.0, 60.0)])
def test_ei_f64_relative_error(lo, hi):
    print("[case] ei", lo, hi, flush=True)
    mp.mp.dps = 400
    u = np.concatenate([np.random.default_rng(int(lo * 10) & 255).uniform(lo, hi, 301), [lo, hi, 0.5 * (lo + hi)]])
    got = _ei(-u, np.ones_like(u), 0.0, torch.float64)  # best - mu = u exactly, sd = 1
    want = [mp.mpf(v) * mp.erfc(-mp.mpf(v) / mp.sqrt(2)) / 2 + mp.exp(-mp.mpf(v) ** 2 / 2) / mp.sqrt(2 * mp.pi)
            for v in u]
    err = max(abs(float((mp.mpf(float(a)) - b) / b)) for a, b in zip(got, want))
    # polynomial, exp and four products: below ten half-ulps
    assert err < 10 * 2.0 ** -53, err


def test_ei_f64_special_values():
    print("[case] ei special", flush=True)
    inf, nan = np.inf, np.nan
    mu = np.array([0.0, -3.0, 3.0, inf, -inf, nan, 1.0, 39.0, 45.0, -45.0])
    sd = np.array([1.0, 0.0, 0.0, 1.0, 1.0, 1.0, nan, 1.0, 1.0, 1.0])
    got = _ei(mu, sd, 0.0, torch.float64)
    assert got[0] == pytest.approx(0.3989422804014327, rel=1e-15)
    assert got[1] == 3.0 and got[2] == 0.0          # sd = 0: max(0, best - mu)
    assert got[3] == 0.0 and got[4] == inf and np.isnan(got[5])
    assert got[6] == 0.0                            # a NaN sd counts as 0
    assert 0.0 <= got[7] < 1e-300 and got[8] == 0.0 and got[9] == 45.0


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("n,q", [(1, 1), (511, 3), (513, 8), (5000, 64), (261120, 5), (261121, 5), (262145, 64)])
def test_selection_beside_ehvi(n, q, dtype):
    """The picks that the fused pass makes in its EHVI kernel, with workgroups of
    eight and of sixteen waves, are those of the selection by itself."""
    print("[case] select", n, q, dtype, flush=True)
    rng = np.random.default_rng(n)
    X, Y = rng.random((24, 4)), rng.standard_normal((24, 2))
    gps = [S.gp_fit(X, Y[:, j], np.full(4, 0.4), 1.0, 1e-2, dtype=dtype) for j in range(2)]
    forest = S.forest_create(np.array([0, 0, 0], np.int32), np.array([0.7, 0, 0], np.float32),
                             np.array([1, -1, -1], np.int32), np.array([2, -1, -1], np.int32),
                             np.array([0, 65536, 0], np.int32), np.array([0, 3], np.int64), 4)
    Xc = torch.tensor(rng.random((n, 4), dtype=np.float32), device="cuda:0")
    b = S.score_pool(gps, forest, Xc, q, Y_obs=Y, ref=Y.max(0) + 0.1)
    idx, score, n_valid = S.suggest_topq(b.acq, b.mask, q)
    torch.cuda.synchronize()
    assert b.idx.tolist() == idx.tolist() and int(b.n_valid) == int(n_valid) == int(b.mask.sum())
    assert torch.equal(b.score.nan_to_num(-1), score.nan_to_num(-1))


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("m", [1, 2, 3, 4, 7, 40])
def test_ehvi_three_objectives_few_columns(m, dtype):
    """Fronts of as many columns as the workgroup has waves, fewer and more, at
    pools around a workgroup's 64 candidates, against the oracle."""
    from oracle.hypervolume import ehvi, nondominated

    rng = np.random.default_rng(m)
    Y = rng.random((m, 3))
    Y /= Y.sum(1, keepdims=True)  # every point on the front
    ref = np.full(3, 1.1)
    for n in (1, 63, 64, 65, 200):
        print("[case] ehvi3", m, n, dtype, flush=True)
        mu, sd = rng.random((n, 3)), np.abs(rng.normal(0, 0.3, (n, 3)))
        sd[0] = 0.0
        mu, sd = ([torch.tensor(v[:, j], dtype=dtype, device="cuda:0") for j in range(3)] for v in (mu, sd))
        got = S.acq_ehvi(mu, sd, Y, ref).cpu().numpy().astype(np.float64)
        held = [np.stack([v.cpu().numpy().astype(np.float64) for v in a], axis=1) for a in (mu, sd)]
        want = ehvi(held[0], held[1], nondominated(Y, ref), ref)
        eps = 2.0 ** (-24 if dtype == torch.float32 else -53)
        # three factors good to about eight eps of themselves (the float partial
        # expectation to 4e-7), whose differences telescope over at most m + 1 columns
        assert np.max(np.abs(got - want)) <= 24 * eps * (m + 3) * np.max(want)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("n,q", [(8192, 64), (8193, 64), (16385, 64), (50000, 12), (130561, 4), (131073, 4)])
def test_selection_beside_ehvi_many_keys(n, q, dtype):
    """Either side of 1024 keys for the second stage in workgroups of eight and of sixteen waves."""
    test_selection_beside_ehvi(n, q, dtype)
