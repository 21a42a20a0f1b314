"""Workspaces of the asynchronous dots: one for each stream, so that dots that
overlap share no counters and accumulators, and one for each captured dot."""
import types

import numpy as np
import pytest
import torch

from paper_2302_04180_amd import rpk


class FakeLibrary:
    """Takes the place of the C library on the CPU: notes the workspaces it is given."""

    def __init__(self):
        self.ws = []

    def rpk_exdot_workspace_bytes(self, n, launch, out):
        out._obj.value = 4096 + 8 * (n // 1000)
        return 0

    def rpk_exdot(self, n, x, y, out, dots, launch, ws, ws_bytes, stream):
        self.ws.append((stream, ws, ws_bytes))
        return 0

    def rpk_fpedot(self, n, x, y, out, lost, launch, ws, ws_bytes, stream):
        self.ws.append((stream, ws.value, ws_bytes))
        return 0


@pytest.fixture
def fake(monkeypatch):
    now = types.SimpleNamespace(lib=FakeLibrary(), stream=0, capturing=False, made=[])
    zeros = torch.zeros

    def cpu_zeros(*size, device=None, **kw):
        now.made.append(zeros(*size, **kw))  # kept, so that no address is used twice
        return now.made[-1]

    monkeypatch.setattr(rpk, "_lib", now.lib)
    monkeypatch.setattr(rpk, "_dev", lambda t: t)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 0, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda dev: now.stream, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_isCurrentStreamCapturing", lambda: now.capturing, raising=False)
    monkeypatch.setattr(torch, "zeros", cpu_zeros)
    for cache in ("_ws_cache", "_dot_ws"):
        monkeypatch.setattr(rpk, cache, {}, raising=False)
    rpk._dot_bytes.cache_clear()
    yield now
    rpk._dot_bytes.cache_clear()


def both(n):
    x = torch.empty(n, dtype=torch.float64)
    rpk.exdot(x, x)
    rpk.fpedot(x, x)


def test_a_workspace_for_each_stream(fake):
    for stream in (0, 7, 0, 9, 7):
        fake.stream = stream
        both(5000)
    of = {s: {w for t, w, _ in fake.lib.ws if t == s} for s in (0, 7, 9)}
    assert all(len(w) == 1 for w in of.values())                 # kept and shared in a stream
    assert len(set.union(*of.values())) == 3                     # by no two streams
    fake.stream = 7
    both(5000000)                                                # a larger one for one of them
    assert fake.lib.ws[-1][1] not in set.union(*of.values())
    fake.stream = 9
    both(5000)
    assert {fake.lib.ws[-1][1]} == of[9]


def test_captured_dots_have_their_own(fake):
    both(5000)
    eager = fake.lib.ws[-1][1]
    fake.capturing = True
    for _ in range(3):
        both(5000)
    fake.capturing = False
    both(5000)
    captured = [w for _, w, _ in fake.lib.ws[2:8]]
    assert len(set(captured)) == 6 and eager not in captured
    assert fake.lib.ws[-1][1] == eager


def test_the_number_kept_is_bounded(fake):
    for stream in range(3 * rpk._DOT_STREAMS):
        fake.stream = stream
        both(2000)
    assert len(rpk._dot_ws) == rpk._DOT_STREAMS
    assert (0, 3 * rpk._DOT_STREAMS - 1) in rpk._dot_ws


@pytest.mark.gpu
def test_dots_on_two_streams(orc):
    sizes = (70000, 300001, 1500000, 9000)
    rng = np.random.default_rng(17)
    data = [(rng.uniform(-1, 1, n), rng.uniform(-1, 1, n)) for n in sizes]
    ref = [orc.exdot(x, y) for x, y in data]
    dev = [(torch.tensor(x, device="cuda"), torch.tensor(y, device="cuda")) for x, y in data]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(3)]
    got = [[], [], []]
    for turn in range(40):
        for k, s in enumerate(streams):
            with torch.cuda.stream(s):
                x, y = dev[(turn + k) % len(sizes)]
                got[k].append((rpk.exdot(x, y), *rpk.fpedot(x, y)))
    torch.cuda.synchronize()
    for k in range(3):
        for turn, (e, f, lost) in enumerate(got[k]):
            want = ref[(turn + k) % len(sizes)]
            assert float(e) == want and float(f) == want and int(lost) == 0, (k, turn)


@pytest.mark.gpu
def test_replayed_dots_beside_eager_ones(orc):
    rng = np.random.default_rng(18)
    n = 400000
    x, y = (torch.tensor(rng.uniform(-1, 1, n), device="cuda") for _ in range(2))
    rpk.exdot(x, y)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        a, (b, lost) = rpk.exdot(x, y), rpk.fpedot(x, y)
    side = torch.cuda.Stream()
    for turn in range(4):
        x.copy_(torch.tensor(rng.uniform(-1, 1, n), device="cuda"))
        want = orc.exdot(x.cpu().numpy(), y.cpu().numpy())
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            g.replay()
        eager = [rpk.exdot(x, y) for _ in range(5)]
        torch.cuda.synchronize()
        assert float(a) == want and float(b) == want and int(lost) == 0, turn
        assert all(float(e) == want for e in eager)
