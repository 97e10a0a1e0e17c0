"""The limit of split_bound.py, by an emulation of the split product with exact
accumulation: the six part products pass, any five of them fail."""
import numpy as np
import pytest

from oracle.gp import matern52
from split_bound import EPS, LIMIT, factor, measure, problem, units

SIX = [(0, 0), (0, 1), (1, 0), (1, 1), (0, 2), (2, 0)]


def _parts(x):
    """Three bfloat16 values, each the nearest to what the ones before leave."""
    x, out = x.astype(np.float64), []
    for _ in range(3):
        u = x.astype(np.float32).view(np.uint32)
        u = (u + np.uint32(0x7FFF) + ((u >> np.uint32(16)) & np.uint32(1))) & np.uint32(0xFFFF0000)
        out.append(u.view(np.float32).astype(np.float64))
        x = x - out[-1]
    return out


@pytest.mark.parametrize("m,d,tau2", [(32, 10, 1e-2), (128, 2, 1e-2), (128, 10, 1e-2), (129, 3, 1e-2), (256, 10, 1e-3), (257, 7, 1e-2),
                                      (512, 12, 1e-3), (576, 16, 1e-2), (576, 3, 1e-2)])
def test_six_part_products_are_told_from_five(m, d, tau2):
    X, y, ls, tau2 = problem(m, d, tau2)
    rng = np.random.default_rng(m)
    Li, alpha = factor(X, y, ls, tau2)
    k = matern52(X, rng.random((512, d)), ls, 1.0)
    unit, _ = units(Li, alpha, k)
    q = ((Li @ k) ** 2).sum(0)
    a, b = _parts(Li), _parts((k * (1 + EPS * rng.uniform(-2, 2, k.shape))).astype(np.float32))
    terms = {ij: a[ij[0]] @ b[ij[1]] for ij in SIX}
    v = sum(terms.values())
    assert measure((v * v).sum(0) - q, unit, 2 * q) < LIMIT / 2
    for ij in SIX:
        less = v - terms[ij]
        assert measure((less * less).sum(0) - q, unit, 2 * q) > 1.5 * LIMIT, ij
