"""Standard loop in three, four and five kernels: the shorter loops, taken by
matrices with a row dictionary and a uniform Jacobi vector, form p and q at the
gathers.  Each solve is compared bit for bit (scalars, iterates, residual) with
the five-kernel one of the same matrix that explicit zero entries, which change
no sum, keep out of the dictionary; on both sides of each rule that chooses, with
each kind of dots, odd launch shapes, and stopped and resumed after every number
of iterations in which the buffers of p and s differ."""
import numpy as np
import pytest

from gpu_util import T, H, same, first_diff, say
from paper_2302_04180_amd import inputs, rpk

pytestmark = pytest.mark.gpu


def without_dictionary(A):
    """The matrix with one explicit zero in each of its first 400 rows, every one
    at another distance from the diagonal: more different rows than fit."""
    rp, ci, v = A
    rows = np.arange(min(400, (rp.size - 1) // 2))
    at = rp[rows + 1]
    cols = (2 * rows + 200) % (rp.size - 1)
    out = rp.astype(np.int64).copy()
    out[1:rows.size + 1] += rows + 1
    out[rows.size + 1:] += rows.size
    return out.astype(np.int32), np.insert(ci, at, cols).astype(np.int32), np.insert(v, at, 0.0)


# 7 points: 2.99M entries in three kernels, 3.05M in four; 27 points: three, four,
# and at 13.5M entries five
CASES = [("poisson7", 17, {}), ("convdiff7", 30, dict(dots=rpk.PLAIN)), ("convdiff7", 31, dict(dots=rpk.FPE)),
         ("convdiff7", 33, dict(block=192, grid=77, fpe=2)), ("poisson7", 40, dict(block=1024, grid=256, fpe=4)),
         ("poisson7", 75, {}), ("poisson7", 76, {}), ("convdiff7", 77, dict(dots=rpk.PLAIN)),
         ("convdiff7", 78, dict(block=320, grid=301, fpe=1)), ("poisson27_etype", 21, {}),
         ("poisson27_etype", 50, {}), ("poisson27_etype", 80, {})]


@pytest.mark.parametrize("kind,edge,how", CASES)
def test_same_bits_as_five_kernels(kind, edge, how):
    A = getattr(inputs, kind)(edge)
    M, M5 = rpk.Matrix(*A), rpk.Matrix(*without_dictionary(A))
    b = T(inputs.uniform(edge ** 3, 7))
    x0 = T(inputs.uniform(edge ** 3, 8))
    maxit = 9
    x5, i5 = rpk.solve(M5, b, x0=x0, tol=0.0, maxit=maxit, record=True, record_xr=edge < 40, **how)
    x, i = rpk.solve(M, b, x0=x0, tol=0.0, maxit=maxit, record=True, record_xr=edge < 40, **how)
    say(kind, edge, how, i["status"], i["iters"])
    assert same(H(x), H(x5)), first_diff(H(x), H(x5))
    assert same(H(i["hist"]), H(i5["hist"])), first_diff(H(i["hist"]), H(i5["hist"]))
    if edge < 40:
        assert same(H(i["xr"]), H(i5["xr"]))
    for k in ("status", "iters", "tau", "tau0", "true_res"):
        assert same(i[k], i5[k]) if isinstance(i[k], float) else i[k] == i5[k], k


@pytest.mark.parametrize("kind,edge,how", [c for c in CASES if c[1] < 77 and c[2].get("dots") != rpk.FPE])
def test_resumed_after_each_limit(kind, edge, how):
    import torch
    A = getattr(inputs, kind)(edge)
    M = rpk.Matrix(*A)
    b = T(inputs.uniform(edge ** 3, 7))
    xu, iu = rpk.solve(M, b, tol=0.0, maxit=9, **how)
    nb = rpk.solve_workspace_bytes(M, **how)
    ws = torch.zeros(nb, dtype=torch.uint8, device="cuda")
    x, info = rpk.solve(M, b, tol=0.0, maxit=0, workspace=ws, **how)
    assert info["status"] == "NOT_CONVERGED" and info["iters"] == 0
    for m in (0, 1, 2, 5, 5, 9):
        x, info = rpk.solve(M, b, x0=x, tol=0.0, maxit=m, workspace=ws, resume=True, **how)
        say("resumed to", m, info["status"], info["iters"])
        assert info["status"] == "NOT_CONVERGED" and info["iters"] == m
    assert same(H(x), H(xu)) and same(info["tau"], iu["tau"]) and same(info["true_res"], iu["true_res"])
