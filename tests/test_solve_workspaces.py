"""The cached workspace of solves and batches under several threads (on the CPU, the
C library replaced): no solve gets a workspace whose zero fill, queued on the stream
of the thread that made it, may still be pending."""
import threading
import time
import types

import pytest
import torch

from paper_2302_04180_amd import rpk


class FakeLibrary:
    def __init__(self):
        self.filling = {}  # workspace -> thread whose stream fills it, until its solve has waited for it
        self.early = []

    def rpk_solve_workspace_bytes(self, A, o, out):
        out._obj.value = 1 << 16
        return 0

    def rpk_solve_batched_workspace_bytes(self, ns, A, o, out):
        out._obj.value = 1 << 16
        return 0

    def _run(self, ws):
        me = threading.get_ident()
        if self.filling.get(ws.value, me) != me:
            self.early.append(ws.value)
        time.sleep(0.02)
        self.filling.pop(ws.value, None)
        return 0

    def rpk_solve(self, A, b, x, o, ws, ws_bytes, stream, info):
        return self._run(ws)

    def rpk_solve_batched(self, ns, A, b, x, o, ws, ws_bytes, stream, infos):
        return self._run(ws)


@pytest.mark.parametrize("batched", [False, True])
def test_two_threads_and_a_new_workspace(monkeypatch, batched):
    import ctypes
    lib = FakeLibrary()
    zeros = torch.zeros
    second = threading.Event()

    def slow_zeros(*size, device=None, **kw):
        t = zeros(*size, **kw)
        if kw.get("dtype") == torch.uint8:
            lib.filling[t.data_ptr()] = threading.get_ident()
        return t

    look_up = rpk._workspace

    def look_up_and_wait(nbytes, key):  # lets the other thread go on between the look-up and the solve
        t = look_up(nbytes, key)
        if threading.current_thread() is first:
            second.set()
            time.sleep(0.1)
        return t

    monkeypatch.setattr(rpk, "_lib", lib)
    monkeypatch.setattr(rpk, "_dev", lambda t: t)
    monkeypatch.setattr(rpk, "_stream", lambda: ctypes.c_void_p(0))
    monkeypatch.setattr(rpk, "_ws_cache", {})
    monkeypatch.setattr(rpk, "_workspace", look_up_and_wait)
    monkeypatch.setattr(torch, "zeros", slow_zeros)
    A = types.SimpleNamespace(n=8, handle=ctypes.c_void_p(8))
    b = torch.empty(8, dtype=torch.float64)

    def call():
        rpk.solve_batched([A], [b]) if batched else rpk.solve(A, b)

    first = threading.Thread(target=call)
    first.start()
    assert second.wait(10)
    call()
    first.join(10)
    assert not lib.early
