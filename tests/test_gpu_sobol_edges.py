"""Candidate generation at the sizes where the kernel's paths change: every
dimension count (its own instantiation, a block of 256 / d runs), pools that
start and end inside a run, rows that are not aligned to 16 bytes (stored one
float at a time), more chunks than workgroups, and grids around 2^24 levels,
where the product with 1 / (levels - 1) gives way to the division.  All of it
is integer and exactly rounded work: bits against the oracle."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2408_04323_amd as S  # noqa: E402
from oracle.sobol import known_constraints_mask, sobol_pool as oracle_pool  # noqa: E402
from workloads import sobol_table  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

LEVELS = [0, 1, 2, 3, 64, 1 << 24, (1 << 24) + 1, 8129, 3000001, 1 << 30]
CASES = [(d, 16 * (256 // d) * 2 + 5, 3 * d, d % 3) for d in range(1, 17)] + [(16, 400003, 7, 0), (12, 336, 0, 0),
                                                                            (12, 337, 0, 1), (8, 4096, 16, 0)]


@pytest.mark.parametrize("d,n,skip,shift", CASES)
def test_pool_bits(d, n, skip, shift):
    rng = np.random.default_rng(d)
    lv = [LEVELS[(d + j) % len(LEVELS)] for j in range(d)]
    r = 1 + d % 8
    A = rng.choice([-1.0, 0.0, 1.0, 0.375], size=(r, d))
    b = rng.uniform(-0.2, 0.6, r)
    poly, vinit = sobol_table(d)
    print("[case] sobol", d, n, skip, shift, flush=True)
    sys.stdout.flush()
    room = torch.full((n * d + 8,), -7.0, dtype=torch.float32, device=DEV)
    out = room[shift:shift + n * d].view(n, d)  # shift floats off the allocation's alignment
    known = torch.full((n + 1,), 9, dtype=torch.uint8, device=DEV)
    S.sobol_pool(poly, vinit, lv, n, skip=skip, A=A, b=b, out=out, known=known[:n])
    torch.cuda.synchronize()
    got, mask = out.cpu().numpy(), known[:n].cpu().numpy()
    for lo, hi in ((0, n),) if n < 10000 else ((0, 2000), (n - 2000, n)):
        want = oracle_pool(poly, vinit, lv, hi - lo, skip=skip + lo)
        np.testing.assert_array_equal(got[lo:hi].view(np.uint32), want.view(np.uint32))
        np.testing.assert_array_equal(mask[lo:hi], known_constraints_mask(want, A, b))
    rest = room.cpu().numpy()
    assert (rest[:shift] == -7.0).all() and (rest[shift + n * d:] == -7.0).all() and int(known[n]) == 9
