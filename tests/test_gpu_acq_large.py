"""EHVI over pools whose launch would hold 2^32 threads and more: the last
candidates' scores are those of the same candidates by themselves; and the
one-wave form of large pools with small fronts."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2408_04323_amd as S  # noqa: E402

pytestmark = pytest.mark.gpu


def test_ehvi_three_objectives_beyond_2_30_candidates():
    n, tail = (1 << 30) + 65, 1000
    print("[case] ehvi3", n, flush=True)
    free, _ = torch.cuda.mem_get_info()
    if free < 16 * n:
        pytest.skip("not enough device memory")
    mu = torch.full((n,), 3.0, device="cuda:0")  # beyond the reference point
    sd = torch.full((n,), 0.1, device="cuda:0")
    rng = np.random.default_rng(0)
    for at in (0, (1 << 29) - 500, n - tail):  # ends, and across a multiple of 2^29
        mu[at:at + tail] = torch.from_numpy(rng.standard_normal(tail).astype(np.float32)).cuda()
        sd[at:at + tail] = torch.from_numpy(rng.uniform(0.1, 1.0, tail).astype(np.float32)).cuda()
    Y, ref = np.array([[0.2, -0.1, 0.3], [-0.4, 0.5, 0.1]]), np.ones(3)
    out = S.acq_ehvi([mu] * 3, [sd] * 3, Y, ref)
    for at in (0, (1 << 29) - 500, n - tail):
        m, d = mu[at:at + tail].clone(), sd[at:at + tail].clone()
        want = S.acq_ehvi([m] * 3, [d] * 3, Y, ref)
        assert float(want.max()) > 0.01
        # the columns' terms may come in another order: each good to about eight eps, three of them
        assert float((out[at:at + tail] - want).abs().max()) <= 24 * 2.0 ** -24 * 5 * float(want.max()), at


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("m,n", [(1, 8 * 256 * 64 - 63), (1, 8 * 256 * 64 - 64), (3, 16 * 256 * 64 - 63), (4, 16 * 256 * 64 - 64),
                                 (5, 16 * 256 * 64), (10, 16 * 256 * 64 + 1), (11, 300001)])
def test_ehvi_three_objectives_one_wave(m, n, dtype):
    """Large pools with small fronts take one wave per workgroup: the scores of the same candidates in a small pool."""
    print("[case] ehvi3 one wave", m, n, dtype, flush=True)
    rng = np.random.default_rng(m)
    Y = rng.random((m, 3))
    Y /= Y.sum(1, keepdims=True)  # every point on the front
    gen = torch.Generator("cuda:0").manual_seed(m)
    mu = [torch.rand(n, dtype=dtype, device="cuda:0", generator=gen) for _ in range(3)]
    sd = [0.3 * torch.rand(n, dtype=dtype, device="cuda:0", generator=gen) for _ in range(3)]
    got = S.acq_ehvi(mu, sd, Y, np.full(3, 1.1))
    for at in (0, n - 4097):
        part = [[v[at:at + 4097].clone() for v in a] for a in (mu, sd)]
        want = S.acq_ehvi(*part, Y, np.full(3, 1.1))
        eps = 2.0 ** (-24 if dtype == torch.float32 else -53)
        # the columns' terms in another order: each good to about eight eps, m + 1 of them
        assert float((got[at:at + 4097] - want).abs().max()) <= 24 * eps * (m + 3) * float(want.max())
