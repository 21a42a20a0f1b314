"""A limit on the workgroups of a batch's launches: the tiles are covered in at most
four launches a phase, and every system keeps its bits."""
import pytest

from gpu_util import T, H, same
from paper_2302_04180_amd import inputs, rpk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant", [rpk.STD, rpk.PIPELINED, rpk.PCG])
@pytest.mark.parametrize("grid", [1, 8, 40, 1000])
def test_capped_launches(variant, grid):
    Ms = [rpk.Matrix(*inputs.poisson7(e)) for e in (13, 6, 17)]
    bs = [T(inputs.uniform(M.n, 50 + k)) for k, M in enumerate(Ms)]
    xs, infos = rpk.solve_batched(Ms, bs, tol=1e-9, maxit=60, variant=variant, tile=64, block=64, grid=grid)
    tiles = sum(-(-M.n // 64) for M in Ms)
    got = infos[0]["used"]["grid"]
    assert 4 * got >= tiles and got >= min(grid, tiles)
    for M, b, x, info in zip(Ms, bs, xs, infos):
        x1, i1 = rpk.solve(M, b, tol=1e-9, maxit=60, variant=variant)
        assert info["iters"] == i1["iters"] and same(H(x), H(x1))
        M.close()
