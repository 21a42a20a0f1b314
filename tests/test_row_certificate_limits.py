"""Limits of the certified row sum as they are held: a word for a dictionary row, a
word for a slice's range and a byte for a row's lowest bit (csrc/span.h), never looser
than the exact ones.  Rows certified under them are correctly rounded, and one entry
of many bits elsewhere in a matrix of short ones leaves its rows certified."""
import os
import subprocess

import numpy as np
import pytest

from test_row_certificate import exact_rn, rows
from test_row_certificate_exponents import certify, edge_rows, limits

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include "span.h"
int main() {
  long bad = 0;
  for (int elo = -1073; elo <= 1024; ++elo)
    for (int ehi = elo; ehi <= 1024; ehi += 1 + (ehi - elo) / 7) {
      const int lsb = elo - 1 - (ehi - elo) % 53 < -1074 ? -1074 : elo - 1 - (ehi - elo) % 53;
      const rpk::CertLim l = rpk::cert_unpack(rpk::cert_pack(elo, ehi, lsb));
      const int xlo = -966 - elo, xhi = 989 - ehi;
      bad += l.xlo < xlo || l.xlo > xlo + 3 || l.lsb1 != lsb - 1;
      bad += l.xhi > xhi || l.xhi < (xhi < 2044 ? xhi : 2044) - 3;
    }
  for (int lsb = -1074; lsb <= 1023; ++lsb) {
    const int b = rpk::cert_unpack_lsb(rpk::cert_pack_lsb(lsb));
    bad += b > lsb - 1 || b <= lsb - 1 - 16;
  }
  std::printf("bad %ld\n", bad);
  return bad != 0;
}
"""


def test_packed_limits_are_never_looser(tmp_path):
    src, exe = tmp_path / "limits.cpp", tmp_path / "limits"
    src.write_text(PROGRAM)
    subprocess.check_call(["hipcc", "-x", "hip", "--offload-host-only", "-std=c++17", "-O1",
                           "-I" + os.path.join(ROOT, "paper_2302_04180_amd", "csrc"), str(src), "-o", str(exe)])
    out = subprocess.run([str(exe)], stdout=subprocess.PIPE, timeout=60)
    assert out.returncode == 0 and b"bad 0" in out.stdout, out.stdout.decode()


def held(values, lsb_step=1, others=()):
    """Limits of a row as held: range over the row and the others of its slice, in
    steps of four, its lowest bit in steps of lsb_step."""
    xlo, xhi, _ = limits(list(values) + list(others))
    _, _, lsb1 = limits(values)
    return -(-xlo // 4) * 4, xhi // 4 * 4, lsb1 // lsb_step * lsb_step


@pytest.mark.parametrize("make", [rows, edge_rows])
@pytest.mark.parametrize("step", [1, 16])
def test_certified_rows_are_correctly_rounded(make, step):
    rng = np.random.default_rng(step)
    certified = total = 0
    for a, x in make(rng, 1500):
        a, x = list(map(float, a)), list(map(float, x))
        ok, y = certify(a, x, held(a, step, [6.0, 2.0 ** -30, 1e9]))
        total += 1
        if ok:
            certified += 1
            ref = exact_rn(a, x)
            assert np.float64(y).view(np.uint64) == np.float64(ref).view(np.uint64), (a, x, y, ref)
    assert certified > total // 3


def test_one_odd_entry_elsewhere():
    rng = np.random.default_rng(3)
    a = [-1.0, -1.0, -1.0, 6.0, -1.0, -1.0, -1.0]
    xs = [list(map(float, rng.uniform(-1, 1, 7))) for _ in range(2000)]
    for step in (1, 16):
        assert all(certify(a, x, held(a, step, [0.1, 6.1]))[0] for x in xs)
    # with the lowest bit of the whole matrix a quarter of them were not
    assert sum(certify(a, x, limits(a + [0.1]))[0] for x in xs) < 1700


def odd_matrices():
    from paper_2302_04180_amd import inputs
    import test_gpu_window as window
    rng = np.random.default_rng(9)
    yield "dictionary", inputs.poisson7(24), {}
    rp, ci, v = inputs.poisson7(24)                                     # short coefficients, all rows different
    yield "sell", (rp, ci, np.where(ci == np.repeat(np.arange(rp.size - 1), np.diff(rp)), 9.0,
                                    -rng.integers(32, 64, v.size) / 32.0)), {}
    rp, ci, v = window.scattered(40000, 1000, 1000, 20, seed=60000)
    yield "window", (rp, ci, np.round(v * 64) / 64 + (v == 0)), dict(block=1024, grid=16)


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["dictionary", "sell", "window"])
@pytest.mark.parametrize("value", [0.1, 6.1, 1e-300, 5e-324, 1e300])
def test_gpu_odd_entry_keeps_the_certificate(orc, kind, value):
    from gpu_util import T, H, same, first_diff
    from paper_2302_04180_amd import rpk
    A, launch = next((A, launch) for name, A, launch in odd_matrices() if name == kind)
    rp, ci, v = A[0], A[1], A[2].copy()
    k = rp[5] + (ci[rp[5]] == 5)                                        # an entry of row 5 beside its diagonal
    v[k] = value
    M = rpk.Matrix(rp, ci, v)
    f = M.form(**launch)
    assert f["certified"] == 1 and (f["dictionary"] > 0) == (kind == "dictionary") and (f["window"] > 0) == (kind == "window")
    rng = np.random.default_rng(4)
    for x in (rng.uniform(-1, 1, M.n), rng.integers(-8, 9, M.n) / 8.0,
              np.ldexp(rng.uniform(-1, 1, M.n), rng.integers(-300, 301, M.n))):
        y, ref = H(rpk.exspmv(M, T(x), **launch)), orc.exspmv(rp, ci, v, x)
        assert same(y, ref), first_diff(y, ref)
    M.close()
