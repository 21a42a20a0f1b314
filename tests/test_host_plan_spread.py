"""The tile table that batches and the server run (on the CPU, no device call): every
row of every system once, in 64-row-aligned tiles numbered 0..G-1 inside each system,
within the length the workspace has room for; where whole systems would leave XCDs
idle, cut into contiguous ranges that fill the XCDs evenly, else the uncut table."""
import numpy as np
import pytest

from paper_2302_04180_amd import rpk


@pytest.fixture(scope="module", autouse=True)
def lib():
    import torch  # noqa: F401  (one HIP runtime shared with torch)
    rpk.load()


def check(sizes, tile):
    t = rpk.plan_tiles(sizes, tile, spread=True)
    whole = rpk.plan_tiles(sizes, tile)
    G = [max(1, -(-n // tile)) for n in sizes]
    assert len(t) % 8 == 0 and len(t) <= 8 * (-(-sum(G) // 8) + max(G))
    real = t[t[:, 0] >= 0]
    real = real[np.lexsort((real[:, 3], real[:, 0]))]
    assert len(real) == sum(G) and np.all(t[t[:, 0] < 0] == [-1, 0, 0, 0])
    at = 0
    for k, n in enumerate(sizes):
        mine = real[at:at + G[k]]
        at += G[k]
        assert np.all(mine[:, 0] == k) and np.array_equal(mine[:, 3], np.arange(G[k]))
        lo, hi = mine[:, 1], mine[:, 2]
        assert lo[0] == 0 and hi[-1] == n and np.array_equal(lo[1:], hi[:-1])
        assert np.all(lo % 64 == 0) and np.all(hi > lo) and np.all(hi - lo <= tile)
    share = -(-sum(G) // 8)
    cut = 16 * (len(whole) // 8) > 17 * share
    assert len(t) == (8 * share if cut else len(whole))
    if not cut:
        assert np.array_equal(t, whole)
        return False
    for x in range(8):  # an XCD's list: runs of consecutive tiles of one system, no padding inside
        mine = t[x::8]
        mine = mine[mine[:, 0] >= 0]
        assert len(mine) <= share and np.all(t[x::8][:len(mine), 0] >= 0)
        same = mine[1:, 0] == mine[:-1, 0]
        assert np.all(mine[1:, 3][same] == mine[:-1, 3][same] + 1)
        assert np.sum(~same) + 1 == len(set(mine[:, 0].tolist())) or not len(mine)
    return True


def test_random_mixes():
    rng = np.random.default_rng(11)
    cuts = 0
    for k in range(300):
        count = int(rng.integers(1, 40))
        sizes = np.exp(rng.uniform(0, np.log(2e6 if k % 3 else 2e4), count)).astype(np.int64) + 1
        cuts += check([int(n) for n in sizes], int(rng.choice([64, 128, 512, 1024, 4096, 16384])))
    assert 30 < cuts < 270


@pytest.mark.parametrize("sizes,tile,cut", [
    ([1], 64, False), ([64 * 8], 64, True), ([64] * 8, 64, False), ([64] * 9, 64, False), ([64 * 17] * 9, 64, True),
    ([2 ** 31 - 1], 1 << 16, True), ([2 ** 31 - 1, 1, 1], 1 << 20, True), ([10 ** 6] * 8, 4096, False),
    ([10 ** 6] * 7, 4096, True), ([10 ** 6] + [1] * 500, 4096, True), ([5] * 1000, 1024, False)])
def test_extreme_mixes(sizes, tile, cut):
    assert check(sizes, tile) == cut


def test_the_served_mix_is_cut():
    edges = [18, 119, 36, 57, 21, 100, 33, 64, 18, 27, 89, 46, 41, 75, 24, 30]
    assert check([e ** 3 for e in edges], 4096)
