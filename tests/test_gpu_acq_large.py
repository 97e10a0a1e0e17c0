"""EHVI over pools whose launch would hold 2^32 threads and more: the last
candidates' scores are those of the same candidates by themselves."""
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
        assert torch.equal(out[at:at + tail], want), at
