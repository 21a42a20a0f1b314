"""Operand window of the SpMV: a matrix of scattered columns inside a band takes
its operand from LDS where the window of a workgroup's rows fits there.  Rows are
compared with the oracle (exact) and with the same kernel without a window
(plain), bit for bit: bands on both sides of the widest one, one-sided, ragged
last slices and workgroups without rows, unequal rows, and rows that need the
integer path.  Solves are compared with those of a launch shape that has no
window."""
import numpy as np
import pytest

from gpu_util import T, H, same, first_diff
from paper_2302_04180_amd import rpk

pytestmark = pytest.mark.gpu


def scattered(n, lo, hi, k, seed, spread=0, symmetric=False):
    """Rows of 2 to k entries at random columns between lo before and hi behind the
    diagonal, the outermost ones included; diagonally dominant (spread = 0)."""
    rng = np.random.default_rng(seed)
    r = np.repeat(np.arange(n), rng.integers(2, k + 1, n))
    c = r + rng.integers(-lo, hi + 1, r.size)
    r = np.concatenate([r, [lo], [n - 1 - hi]])
    c = np.concatenate([c, [0], [n - 1]])
    keep = (c >= 0) & (c < n) & (c != r)
    r, c = r[keep], c[keep]
    if symmetric:
        r, c = np.concatenate([r, c]), np.concatenate([c, r])
    key = np.unique(r * np.int64(n) + c)
    r, c = key // n, key % n
    if symmetric:
        pair = np.minimum(r, c) * np.int64(n) + np.maximum(r, c)
        v = -(1 + (pair % 1009) / 1009.0)
    else:
        v = rng.uniform(-1, 1, r.size)
    diag = np.bincount(r, weights=np.abs(v), minlength=n) + 1.0
    if spread:
        v = np.ldexp(v, rng.integers(-spread, spread + 1, v.size))
    r, c, v = np.concatenate([r, np.arange(n)]), np.concatenate([c, np.arange(n)]), np.concatenate([v, diag])
    order = np.lexsort((c, r))
    rp = np.zeros(n + 1, np.int64)
    np.cumsum(np.bincount(r, minlength=n), out=rp[1:])
    return rp.astype(np.int32), c[order].astype(np.int32), v[order]


# (rows, band before, band behind, entries, workgroup, workgroups); the band may
# be 16,384 columns wide, and none of them has a window in 512 workgroups of 512
CASES = [(40000, 1000, 1000, 20, 1024, 16), (40001, 700, 0, 16, 512, 25), (39937, 0, 900, 18, 256, 40),
         (70000, 8192, 8192, 30, 256, 31), (70000, 8192, 8193, 30, 256, 31), (66000, 9000, 3000, 24, 1024, 37),
         (5000, 64, 64, 16, 64, 200), (5063, 100, 200, 40, 128, 7)]


@pytest.mark.parametrize("n,lo,hi,k,block,grid", CASES)
@pytest.mark.parametrize("spread", [0, 480])
def test_rows(orc, n, lo, hi, k, block, grid, spread):
    A = scattered(n, lo, hi, k, seed=n + k, spread=spread)
    M = rpk.Matrix(*A)
    rng = np.random.default_rng(3)
    x = np.ldexp(rng.uniform(-1, 1, n), rng.integers(-spread, spread + 1, n))
    y = H(rpk.exspmv(M, T(x), block=block, grid=grid))
    ref = orc.exspmv(*A, x)
    assert same(y, ref), first_diff(y, ref)
    assert same(H(rpk.exspmv(M, T(x), block=block, grid=grid, fpe=1)), ref)
    plain = H(rpk.exspmv(M, T(x), block=512, grid=512, dots=rpk.PLAIN))
    assert same(H(rpk.exspmv(M, T(x), block=block, grid=grid, dots=rpk.PLAIN)), plain)
    x[lo] = np.inf                       # only the rows that hold it, as without a window
    assert same(H(rpk.exspmv(M, T(x), block=block, grid=grid)), H(rpk.exspmv(M, T(x), block=512, grid=512)))
    M.close()


@pytest.mark.parametrize("variant,symmetric", [(rpk.STD, False), (rpk.PIPELINED, False), (rpk.PCG, True)])
@pytest.mark.parametrize("n,lo,hi,k,block,grid", [CASES[0], CASES[2], CASES[5]])
@pytest.mark.parametrize("dots", [rpk.EXACT, rpk.FPE])
def test_solves(n, lo, hi, k, block, grid, variant, symmetric, dots):
    A = scattered(n, lo, hi, k, seed=5, symmetric=symmetric)
    M = rpk.Matrix(*A)
    b = T(np.random.default_rng(4).uniform(-1, 1, n))
    out = [rpk.solve(M, b, tol=1e-10, maxit=40, variant=variant, dots=dots, block=B, grid=G, record=True)
           for B, G in ((block, grid), (512, 512))]
    (x, i), (x1, i1) = out
    assert i["status"] == i1["status"] and i["iters"] == i1["iters"] > 3
    assert same(H(x), H(x1)), first_diff(H(x), H(x1))
    assert same(H(i["hist"]), H(i1["hist"])) and same(i["true_res"], i1["true_res"])
    M.close()
