"""Exact reductions in workgroups of few wavefronts: dots equal the oracle's and
batches in small tiles equal the systems alone, from one wavefront to five."""
import numpy as np
import pytest

from gpu_util import T, H, same
from paper_2302_04180_amd import inputs, rpk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("block", [64, 128, 192, 256, 320])
@pytest.mark.parametrize("n,grid", [(1, 1), (65, 1), (1000, 2), (20001, 9), (50000, 70)])
def test_dots(orc, block, n, grid):
    rng = np.random.default_rng(n + block)
    for spread in (0, 40):
        x, y = (np.ldexp(rng.uniform(-1, 1, n), rng.integers(-spread, spread + 1, n)) for _ in range(2))
        ref = orc.exdot(x, y)
        for fpe in (1, 3, 8):
            assert same(float(H(rpk.exdot(T(x), T(y), block=block, grid=grid, fpe=fpe))), ref), fpe


@pytest.mark.parametrize("variant", [rpk.STD, rpk.PIPELINED, rpk.PCG])
@pytest.mark.parametrize("block,tile", [(64, 64), (128, 64), (192, 320), (256, 128)])
def test_batches(variant, block, tile):
    Ms = [rpk.Matrix(*A) for A in (inputs.poisson7(9), inputs.poisson7_vardiag(11), inputs.poisson7(4))]
    bs = [T(inputs.uniform(M.n, 30 + k)) for k, M in enumerate(Ms)]
    xs, infos = rpk.solve_batched(Ms, bs, tol=1e-9, maxit=80, variant=variant, block=block, tile=tile)
    for M, b, x, info in zip(Ms, bs, xs, infos):
        x1, i1 = rpk.solve(M, b, tol=1e-9, maxit=80, variant=variant)
        assert info["status"] == i1["status"] == "OK" and info["iters"] == i1["iters"] and same(H(x), H(x1))
        M.close()
