"""Automatic launch shapes of the dots: exact ones equal the oracle's and
lightweight ones (nothing lost) equal them, on both sides of every size where the
shape changes."""
import numpy as np
import pytest

from gpu_util import T, H
from paper_2302_04180_amd import rpk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [4096, 4097, 65535, 65536, 66559, 66560, 262143, 262144, 1048575, 1048576])
def test_both_sides_of_each_shape(orc, n):
    rng = np.random.default_rng(n)
    x, y = rng.uniform(-1, 1, n), rng.uniform(-1, 1, n)
    ref = orc.exdot(x, y)
    assert float(H(rpk.exdot(T(x), T(y)))) == ref
    value, lost = rpk.fpedot(T(x), T(y))
    assert int(H(lost)) == 0 and float(H(value)) == ref
    # the plain sum: n products and additions of at most 1 each
    assert abs(float(H(rpk.exdot(T(x), T(y), dots=rpk.PLAIN))) - ref) <= n * n * 2.0 ** -53
