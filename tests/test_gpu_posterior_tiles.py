"""Small pools take tiles of 32 candidates, others of 64: the same bits, either
side of the edges of both tiles and of the size where one passes to the other."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2408_04323_amd as S  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
HALVES = 256 * 32  # one tile of 32 per compute unit


@pytest.mark.parametrize("m,d", [(1, 1), (32, 10), (64, 3), (97, 12), (128, 10), (129, 6), (192, 10), (256, 16)])
def test_tiles_of_32_and_64_give_the_same_bits(m, d):
    print("[case] posterior tiles", m, d, flush=True)
    rng = np.random.default_rng(m)
    gp = S.gp_fit(rng.random((m, d)), rng.standard_normal(m), rng.uniform(0.3, 1.5, d), 1.0, 1e-2)
    pool = torch.from_numpy(rng.random((HALVES + 101, d)).astype(np.float32)).to(DEV)
    mu, sd = S.posterior(gp, pool)
    for n in (1, 31, 32, 33, 63, 65, 4097, HALVES - 1, HALVES):
        a, b = S.posterior(gp, pool[:n].contiguous())
        assert torch.equal(a, mu[:n]) and torch.equal(b, sd[:n]), n
