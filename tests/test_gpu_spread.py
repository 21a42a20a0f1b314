"""Batches and server rounds in which a system has more than its share of tiles
and is cut over several XCDs: every solve keeps the bits of that system alone."""
import numpy as np
import pytest

from gpu_util import T, H, same
from paper_2302_04180_amd import inputs, rpk

pytestmark = pytest.mark.gpu

# one large system; two large ones around small ones; nearly even ones, of which
# one is cut by a single tile
MIXES = [(40,), (9, 40, 12, 30, 4), (17, 17, 17, 17, 17, 17, 17, 17, 17)]


def systems(edges):
    As = [(inputs.poisson7 if k % 2 else inputs.convdiff7)(e) for k, e in enumerate(edges)]
    return [rpk.Matrix(*A) for A in As], [T(inputs.uniform(e ** 3, 60 + k)) for k, e in enumerate(edges)]


def check(Ms, bs, xs, infos, variant, maxit):
    for M, b, x, info in zip(Ms, bs, xs, infos):
        x1, i1 = rpk.solve(M, b, tol=1e-9, maxit=maxit, variant=variant)
        assert info["status"] == i1["status"] and info["iters"] == i1["iters"]
        assert same(H(x), H(x1)) and same(info["tau"], i1["tau"]) and same(info["true_res"], i1["true_res"])


@pytest.mark.parametrize("edges", MIXES)
@pytest.mark.parametrize("variant", [rpk.STD, rpk.PIPELINED])
def test_batch(edges, variant):
    Ms, bs = systems(edges)
    tiles = [-(-e ** 3 // 256) for e in edges]
    whole = rpk.plan_tiles([e ** 3 for e in edges], 256)
    assert 16 * (len(whole) // 8) > 17 * -(-sum(tiles) // 8)    # the systems are cut
    xs, infos = rpk.solve_batched(Ms, bs, tol=1e-9, maxit=60, variant=variant, tile=256, block=128)
    check(Ms, bs, xs, infos, variant, 60)


@pytest.mark.parametrize("edges", MIXES)
def test_server(edges):
    Ms, bs = systems(edges)
    srv = rpk.Server(hbm_budget=1 << 28, max_slots=16, chunk=4, tol=1e-9, maxit=60, variant=rpk.PIPELINED,
                     tile=256, block=128)
    xs = [T(np.zeros(b.numel())) for b in bs]
    tickets = [srv.submit(M, b, x) for M, b, x in zip(Ms, bs, xs)]
    check(Ms, bs, xs, [srv.wait(t) for t in tickets], rpk.PIPELINED, 60)
