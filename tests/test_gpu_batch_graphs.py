"""Batches of equal shape on one workspace: a captured iteration graph serves only
batches that take the same kernels.  Systems with a uniform Jacobi vector and
systems of the same sizes without one follow each other, and the tiles of a
capped grid take several launches."""
import pytest
import torch

from gpu_util import H, same, say
from paper_2302_04180_amd import inputs, rpk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant", [rpk.STD, rpk.PIPELINED, rpk.PCG])
@pytest.mark.parametrize("grid", [0, 8])
def test_uniform_and_varying_diagonals_in_turn(variant, grid):
    edges = (9, 17, 12)
    kinds = [[inputs.poisson7(e) for e in edges], [inputs.poisson7_vardiag(e) for e in edges]]
    Ms = [[rpk.Matrix(*a) for a in As] for As in kinds]
    for turn in (0, 1, 0, 1):
        bs = [rpk.exspmv(m, torch.linspace(-1.0, 1.0, m.n, dtype=torch.float64, device="cuda")) for m in Ms[turn]]
        say("variant", variant, "grid", grid, "turn", turn)
        xs, infos = rpk.solve_batched(Ms[turn], bs, tol=1e-9, maxit=300, variant=variant, tile=512, grid=grid)
        for m, b, x, info in zip(Ms[turn], bs, xs, infos):
            xa, ia = rpk.solve(m, b, tol=1e-9, maxit=300, variant=variant)
            assert info["status"] == ia["status"] == "OK" and info["iters"] == ia["iters"]
            assert same(H(x), H(xa))
    for m in Ms[0] + Ms[1]:
        m.close()
