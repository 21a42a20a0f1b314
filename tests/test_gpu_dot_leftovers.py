"""Dots whose terms do not fit the FPE: exponents spread far enough that most
insertions leave something for the long accumulator, products out of the range of
twoprod, and non-finite factors in each place of the unrolled loop.  Exact dots
equal the oracle's for every FPE length, around the sizes where a workgroup's last
pass over its elements is whole, ragged or missing and where the launch shape changes."""
import numpy as np
import pytest

from gpu_util import T, H, same
from paper_2302_04180_amd import rpk

pytestmark = pytest.mark.gpu


def vectors(n, spread, seed):
    rng = np.random.default_rng(seed)
    return [np.ldexp(rng.uniform(-1, 1, n), rng.integers(-spread, spread + 1, n)) for _ in range(2)]


@pytest.mark.parametrize("n", [1, 63, 1023, 1024, 1025, 4095, 4096, 4097, 65537, 270001])
@pytest.mark.parametrize("spread", [20, 60, 480, 1000])
def test_spread_exponents(orc, n, spread):
    x, y = vectors(n, spread, n + spread)
    ref = orc.exdot(x, y)
    xd, yd = T(x), T(y)
    for fpe in (1, 2, 3, 4, 8):
        got = float(H(rpk.exdot(xd, yd, fpe=fpe)))
        assert same(got, ref), (fpe, got, ref)
    for block, grid in ((64, 1), (1024, 2), (320, 7)):
        assert same(float(H(rpk.exdot(xd, yd, block=block, grid=grid))), ref), (block, grid)


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_one_factor_is_not_finite(bad):
    x, y = vectors(8192, 60, 5)
    for at in (0, 63, 64, 1023, 1024, 3000, 4095, 4096, 8191):
        z = x.copy()
        z[at] = bad
        for n in (at + 1, 8192):
            for grid in (0, 1, 3):
                assert np.isnan(float(H(rpk.exdot(T(z[:n]), T(y[:n]), grid=grid)))), (at, n, grid)
    assert np.isfinite(float(H(rpk.exdot(T(x), T(y)))))
