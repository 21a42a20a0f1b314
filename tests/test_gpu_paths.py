"""The tests of the row dictionary, the operand window and the shorter standard loops
compare bits, which every path gives: here that the matrices they use take the path
they are there for, on both sides of each rule."""
import numpy as np
import pytest

from paper_2302_04180_amd import inputs, rpk
import test_gpu_dictionary as dictionary
import test_gpu_std_loops as loops
import test_gpu_window as window

pytestmark = pytest.mark.gpu


def form(A, **launch):
    M = rpk.Matrix(*A)
    f = M.form(**launch)
    M.close()
    return f


def distinct_rows(rp, ci, v):
    return len({(tuple((ci[a:b] - r).tolist()), v[a:b].tobytes()) for r, (a, b) in enumerate(zip(rp[:-1], rp[1:]))})


@pytest.mark.parametrize("n,kinds,width", dictionary.CASES)
def test_dictionaries(n, kinds, width):
    A = dictionary.cyclic(n, kinds, width, seed=n + kinds)
    rows, wide = distinct_rows(*A), int(np.diff(A[0]).max())
    # 255 rows and the empty one, in 1,024 entries, for 32 rows each at least
    fits = rows <= 255 and (rows + 1) * (-(-wide // 4) * 4 + 1) <= 1024 and n >= 32 * rows
    assert form(A)["dictionary"] == (rows if fits else 0)


def test_both_sides_are_there():
    got = [form(dictionary.cyclic(n, k, w, seed=n + k))["dictionary"] > 0 for n, k, w in dictionary.CASES]
    assert any(got) and not all(got)


@pytest.mark.parametrize("n,lo,hi,k,block,grid", window.CASES)
def test_windows(n, lo, hi, k, block, grid):
    A = window.scattered(n, lo, hi, k, seed=n + k)
    f = form(A, block=block, grid=grid)
    chunk = -(--(-n // grid) // 64) * 64
    assert f["dictionary"] == 0 and f["window"] == (chunk + lo + hi if lo + hi <= 16384 else 0)
    assert form(A, block=512, grid=512)["window"] == 0


@pytest.mark.parametrize("kind,edge,how", loops.CASES)
def test_loops(kind, edge, how):
    A = getattr(inputs, kind)(edge)
    n, nnz = A[0].size - 1, A[2].size
    want = 3 if nnz <= 3000000 else 4 if nnz <= 8000000 + 9 * n else 5
    assert form(A)["std_kernels"] == want and form(loops.without_dictionary(A))["std_kernels"] == 5
    M = rpk.Matrix(*A)
    b = rpk.torch.ones(n, dtype=rpk.torch.float64, device="cuda")
    _, info = rpk.solve(M, b, tol=0.0, maxit=2, timing=True, **how)
    M.close()
    launched = sum(1 for k in info["phase_launches"][:5] if k)
    assert launched == (5 if how.get("dots") == rpk.FPE else want)


def test_every_loop_is_there():
    assert {form(getattr(inputs, kind)(edge))["std_kernels"] for kind, edge, _ in loops.CASES} == {3, 4, 5}


def test_certified_rows():
    assert form(inputs.poisson7(20))["certified"] == 1 and form(inputs.poisson27_etype(20))["certified"] == 1
