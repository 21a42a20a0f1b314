"""Pipelined loop with none, six and thirteen of its vectors streamed past the
Infinity Cache: one to four copies of a 96^3 system, stopped after a few
iterations, give the bits of the system solved alone (whose vectors all fit)."""
import pytest

from gpu_util import T, H, same, first_diff
from paper_2302_04180_amd import inputs, rpk

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", params=["convdiff7", "poisson7_vardiag"])
def system(request):
    M = rpk.Matrix(*getattr(inputs, request.param)(96))
    b = T(inputs.uniform(96 ** 3, 41))
    yield M, b, rpk.solve(M, b, tol=0.0, maxit=12, variant=rpk.PIPELINED)
    M.close()


# rows: 1.8M (all fit), 2.7M (eleven fit), 3.5M
@pytest.mark.parametrize("copies,streamed", [(2, False), (3, False), (4, True)])
def test_same_bits(system, copies, streamed):
    M, b, (x1, i1) = system
    xs, infos = rpk.solve_batched([M] * copies, [b] * copies, tol=0.0, maxit=12, variant=rpk.PIPELINED)
    for x, i in zip(xs, infos):
        assert i["streamed"] == streamed and i["iters"] == i1["iters"] == 12
        assert same(H(x), H(x1)), first_diff(H(x), H(x1))
        assert same(i["tau"], i1["tau"]) and same(i["true_res"], i1["true_res"])
