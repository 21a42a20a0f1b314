"""The certified row sum as the SpMV computes it (row_cert): pairwise twosums, an
error bound, and an exactness test from binary exponents.  Its arithmetic is
restated in IEEE double with exact rationals for the fma; every certified row
must be the correctly rounded exact sum, on the adversarial rows of the older
form's test and on rows built around the exactness test's edge."""
import math
from fractions import Fraction as F

import numpy as np
import pytest

from test_row_certificate import exact_rn, rows, tsum


def frexp_exp(v):
    return 0 if v == 0.0 or not math.isfinite(v) else math.frexp(v)[1]


def limits(values):
    """(xlo, xhi, xlsb) of a matrix with these values."""
    nz = [v for v in values if v != 0.0] or [1.0]  # a matrix has a non-zero diagonal
    lsb = []
    for v in nz:
        num, den = abs(v).as_integer_ratio()
        lsb.append((num & -num).bit_length() - 1 - (den.bit_length() - 1))
    e = [frexp_exp(v) for v in nz]
    return -966 - min(e), 989 - max(e), min(lsb) - 1


def certify(a, x, lim):
    xlo, xhi, xlsb = lim
    s = q = m = 0.0
    elo, ehi = 1 << 30, -(1 << 30)
    j0 = 0
    while j0 < len(a):
        B = 8 if len(a) - j0 > 4 else 4
        av = (list(a[j0:j0 + B]) + [0.0] * B)[:B]
        xv = (list(x[j0:j0 + B]) + [x[0]] * B)[:B]  # slots past the row repeat an operand of it
        p, qq, mm = [], [], []
        for i in range(0, B, 2):
            for k in (i, i + 1):
                elo, ehi = min(elo, frexp_exp(xv[k])), max(ehi, frexp_exp(xv[k]))
            p0, p1 = av[i] * xv[i], av[i + 1] * xv[i + 1]
            if not (math.isfinite(p0) and math.isfinite(p1)):
                return False, 0.0
            r0 = float(F(av[i]) * F(xv[i]) - F(p0))
            r1 = float(F(av[i + 1]) * F(xv[i + 1]) - F(p1))
            r, t = tsum(p0, p1)
            p.append(r)
            qq.append((r0 + r1) + t)
            mm.append((abs(r0) + abs(r1)) + abs(t))
        while len(p) > 1:
            n2 = []
            for i in range(0, len(p), 2):
                r, t = tsum(p[i], p[i + 1])
                n2.append((r, (qq[i] + qq[i + 1]) + t, (mm[i] + mm[i + 1]) + abs(t)))
            p, qq, mm = map(list, zip(*n2))
        if j0 == 0:
            s, q, m = p[0], qq[0], mm[0]
        else:
            s, t = tsum(s, p[0])
            q += qq[0] + t
            m += mm[0] + abs(t)
        j0 += B
    y = s + (q + 0.0)
    ay = abs(y)
    if not (elo >= xlo and ehi <= xhi and ay < 2.0 ** 1020):
        return False, y
    if m == 0.0 or frexp_exp(m) <= elo + xlsb:
        return True, y
    k = 2.0 * j0 + 2.0
    E = (m * (k * 2.0 ** -53)) * (1.0 + 2.0 ** -28) + k * 2.0 ** -1074
    z = y - s
    r = (s - (y - z)) + (q - z)
    up = float(np.nextafter(ay, np.inf)) - ay
    half = 0.25 * up if math.frexp(ay)[0] == 0.5 else 0.5 * up
    return ay >= 2.0 ** -960 and (abs(r) + E) * (1.0 + 2.0 ** -50) < half, y


def edge_rows(rng, count):
    """Short coefficients and operands whose sums sit on midpoints, with the
    spread of the exponents swept across the exactness test's limit."""
    for _ in range(count):
        w = int(rng.integers(2, 12))
        a = rng.choice([-1.0, 1.0, 6.0, -2.0, 1.5, 7.75], w)
        bits = int(rng.integers(1, 54))
        x = rng.integers(-(1 << bits), 1 << bits, w).astype(np.float64)
        x = np.ldexp(x, rng.integers(-60, 61, w) if rng.random() < 0.5 else int(rng.integers(-1000, 900)))
        if rng.random() < 0.3:
            x[rng.integers(0, w)] = 0.0
        if rng.random() < 0.3:  # cancel the leading part, leaving half an ulp and a far tail
            x[0] = 1.0
            x[1] = float(np.ldexp(1.0, -53)) * (1 if rng.random() < 0.5 else -1)
            x[2:] = np.ldexp(rng.integers(-3, 4, w - 2).astype(np.float64), int(rng.integers(-130, -50)))
            a[:2] = 1.0
        yield a, x


@pytest.mark.parametrize("make", [rows, edge_rows])
@pytest.mark.parametrize("seed", [1, 2, 3])
def test_certified_rows_are_correctly_rounded(make, seed):
    rng = np.random.default_rng(seed)
    certified = total = 0
    for a, x in make(rng, 1500):
        ok, y = certify(list(map(float, a)), list(map(float, x)), limits(list(map(float, a))))
        total += 1
        if ok:
            certified += 1
            ref = exact_rn(a, x)
            assert np.float64(y).view(np.uint64) == np.float64(ref).view(np.uint64), (a, x, y, ref)
    assert certified > total // 3


def test_stencil_midpoints_are_settled():
    lim = limits([6.0, -1.0])
    # midpoints of one-bit-too-long sums, which the bound alone declines, to even
    assert certify([1.0, 1.0], [1.0, 1.0 + 2.0 ** -52], limits([1.0])) == (True, 2.0)
    assert certify([1.0, 1.0], [1.0 + 2.0 ** -52, 1.0 + 2.0 ** -51], limits([1.0])) == (True, 2.0 + 2.0 ** -50)
    # 1 + 2^-53 spans more bits than the exactness test allows, and is a midpoint: declined
    assert not certify([1.0, 1.0], [1.0, 2.0 ** -53], limits([1.0]))[0]
    rng = np.random.default_rng(5)
    for _ in range(2000):
        x = rng.uniform(-1, 1, 7)
        a = [-1.0, -1.0, -1.0, 6.0, -1.0, -1.0, -1.0]
        ok, y = certify(a, list(map(float, x)), lim)
        assert ok and y == exact_rn(a, x)
    # zero rows and signed zeros give +0
    for z in (0.0, -0.0):
        ok, y = certify([6.0, -1.0], [z, z], lim)
        assert ok and y == 0.0 and math.copysign(1.0, y) == 1.0
