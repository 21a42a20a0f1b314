"""Row dictionary of the SpMV: a matrix whose rows are few different lists of
(column - row, value) is read through a dictionary, every other one through its
SELL copy.  The rows are compared with the oracle (exact, bit for bit) and with
a chain of fmas in entry order (plain, bit for bit) on both sides of every rule
that decides: the number of different rows, the dictionary's entries, the rows
for each different one; with unequal row lengths, ragged last slices, entries
out of column order, and rows that need the integer path."""
from fractions import Fraction

import numpy as np
import pytest

from gpu_util import T, H, same, first_diff
from paper_2302_04180_amd import rpk

pytestmark = pytest.mark.gpu


def cyclic(n, kinds, width, seed, spread=0):
    """n rows cycling through `kinds` different ones of 1..width entries around
    the diagonal (offsets modulo n would differ per row, so rows near the ends
    keep only the entries that fit); spread: binary exponents of the values."""
    rng = np.random.default_rng(seed)
    lens = 1 + np.arange(kinds) % width
    offs = [np.concatenate([[0], rng.permutation(np.r_[-40:0, 1:41])[:k - 1]]) for k in lens]
    vals = [np.ldexp(rng.uniform(1, 2, k), rng.integers(-spread, spread + 1, k)) * rng.choice([-1.0, 1.0], k)
            for k in lens]
    rp, ci, v = [0], [], []
    for r in range(n):
        o, a = offs[r % kinds], vals[r % kinds]
        order = np.random.default_rng(r % kinds).permutation(len(o))
        keep = [j for j in order if 0 <= r + o[j] < n]
        ci += [r + o[j] for j in keep]
        v += [a[j] for j in keep]
        rp.append(len(ci))
    return np.array(rp, np.int32), np.array(ci, np.int32), np.array(v, np.float64)


def fma_rows(rp, ci, v, x):
    """Rows as chains of fmas in entry order, each rounded once (rationals)."""
    out = np.zeros(rp.size - 1)
    for r in range(rp.size - 1):
        acc = 0.0
        for k in range(rp[r], rp[r + 1]):
            acc = float(Fraction(v[k]) * Fraction(x[ci[k]]) + Fraction(acc))
        out[r] = acc
    return out


# (rows, different rows, widest row): the dictionary holds 255 different rows
# and the empty one in 1,024 entries, for at least 32 rows each; ends of the
# matrix add the rows that lose entries
CASES = [(64, 1, 1), (65, 2, 2), (1000, 3, 7), (4099, 40, 3), (9000, 200, 4), (9000, 254, 1), (9001, 255, 1),
         (9001, 256, 1), (300, 10, 5), (320, 10, 1), (319, 10, 1), (5000, 90, 9), (3000, 12, 30)]


@pytest.mark.parametrize("n,kinds,width", CASES)
@pytest.mark.parametrize("spread", [0, 30, 480])
def test_dictionary_rows(orc, n, kinds, width, spread):
    A = cyclic(n, kinds, width, seed=n + kinds, spread=spread)
    rng = np.random.default_rng(7)
    x = np.ldexp(rng.uniform(-1, 1, n), rng.integers(-spread, spread + 1, n))
    x[rng.random(n) < 0.1] = 0.0
    M = rpk.Matrix(*A)
    ref = orc.exspmv(*A, x)
    y = H(rpk.exspmv(M, T(x)))
    assert same(y, ref), first_diff(y, ref)
    for block, grid in ((64, 3), (1024, 1)):
        assert same(H(rpk.exspmv(M, T(x), block=block, grid=grid, fpe=1)), ref)
    if spread < 100 and n < 2000:
        assert np.array_equal(H(rpk.exspmv(M, T(x), dots=rpk.PLAIN)), fma_rows(*A, x))
    M.close()


def test_dictionary_nonfinite_and_late_difference(orc):
    # one row that differs from its kind in the last bit of one value keeps its
    # own value, wherever it lies
    for at in (0, 63, 64, 2047, 4095):
        A = cyclic(4096, 4, 5, seed=3)
        v = A[2].copy()
        v[A[0][at]] = np.nextafter(v[A[0][at]], 2.0)
        x = np.random.default_rng(at).uniform(-1, 1, 4096)
        M = rpk.Matrix(A[0], A[1], v)
        assert same(H(rpk.exspmv(M, T(x))), orc.exspmv(A[0], A[1], v, x))
        x[100] = np.inf
        y = H(rpk.exspmv(M, T(x)))
        touched = np.array([100 in A[1][A[0][r]:A[0][r + 1]] for r in range(4096)])
        assert np.array_equal(np.isnan(y), touched)
        M.close()
