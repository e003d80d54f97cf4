"""The torch layer's cache of prepared workspaces under threads that share a
stream, with a stub in place of the library: CPU tensors, no kernel runs.

A stub call checks what a launch needs: the memory behind its workspace
pointer still belongs to a live tensor when the call is made."""
import collections
import threading
import time
import weakref

import pytest

torch = pytest.importorskip("torch")
from paper_2402_09900_amd import binding as mb  # noqa: E402

WAIT = 0.5


class _TrackingTorch:
    """torch, remembering the workspaces (uint8) it makes by their pointer."""

    def __init__(self):
        self.live = {}

    def __getattr__(self, name):
        return getattr(torch, name)

    def empty(self, *shape, **kw):
        t = torch.empty(*shape, **kw)
        if kw.get("dtype") is torch.uint8:
            self.live[t.data_ptr()] = weakref.ref(t)
        return t

    def alive(self, pointer):
        ref = self.live.get(pointer)
        return ref is not None and ref() is not None


class _StubLibrary:
    """Library whose `prepare` and `launch` are callbacks of the test."""

    def __init__(self, prepare, launch):
        self.memoroid_workspace_prepare = lambda p, n, s: prepare(p) or mb.OK
        self.memoroid_discount_workspace_bytes = lambda B, T: 4096
        # (r, start, gamma, G, B, T, workspace, bytes, stream)
        self.memoroid_discounted_return_prepared = lambda *a: launch(a[5], a[6]) or mb.OK


@pytest.fixture
def layer(monkeypatch):
    """Install a stub; returns (install, call): call(T) is one torch-layer call of length T."""
    track = _TrackingTorch()
    mb._torch()
    monkeypatch.setattr(mb, "_T", track)
    monkeypatch.setattr(mb, "_raw_stream", lambda index: 7)
    monkeypatch.setattr(mb, "_check_cuda", lambda *ts: torch.device("cpu"))
    monkeypatch.setattr(mb, "_PREPARED", collections.OrderedDict())

    def install(prepare=lambda p: None, launch=lambda T, p: None):
        stub = _StubLibrary(prepare, launch)
        monkeypatch.setattr(mb, "lib", lambda: stub)
        return track

    def call(T):
        mb.discounted_return(torch.zeros(1, T), torch.zeros(1, T, dtype=torch.uint8), 0.9)

    return install, call


def _run(targets):
    errors = []

    def guarded(f):
        try:
            f()
        except BaseException as e:      # noqa: BLE001 - reported by the test
            errors.append(e)

    ts = [threading.Thread(target=guarded, args=(f,)) for f in targets]
    for t in ts:
        t.start()
    for t in ts:
        t.join(30)
    assert not errors, errors


def _meet(barrier):
    try:
        barrier.wait(WAIT)
    except threading.BrokenBarrierError:
        pass


def test_two_first_calls_keep_their_workspaces(layer):
    """Both threads find no workspace and prepare one; each pointer must be
    alive at its launch, after both have gone through the cache."""
    install, call = layer
    preparing, launching = threading.Barrier(2), threading.Barrier(2)
    seen = []

    def launch(T, pointer):
        _meet(launching)
        seen.append(track.alive(pointer))

    track = install(lambda p: _meet(preparing), launch)
    _run([lambda: call(64)] * 2)
    assert seen == [True, True]
    assert len(mb._PREPARED) == 1


def test_eviction_by_other_calls_keeps_the_workspace(layer):
    """A workspace dropped from the full cache between a thread's lookup and
    its launch stays alive until that launch is done."""
    install, call = layer
    inside, dropped = threading.Event(), threading.Event()
    seen = []

    def launch(T, pointer):
        if T == 64 and call_no[0] == 2:
            inside.set()
            dropped.wait(10)
            seen.append(track.alive(pointer))

    track = install(launch=launch)
    call_no = [1]
    call(64)
    call_no[0] = 2

    def others():
        assert inside.wait(10)
        for i in range(mb._PREPARED_MAX + 1):
            call(100 + i)
        dropped.set()

    _run([lambda: call(64), others])
    assert seen == [True]
    assert len(mb._PREPARED) == mb._PREPARED_MAX


def test_calls_on_one_workspace_do_not_interleave(layer):
    """A call may launch several kernels that hand values on in its workspace:
    another thread's call on that workspace waits until it has returned."""
    install, call = layer
    inside = [0]
    most = [0]

    def launch(T, pointer):
        inside[0] += 1
        most[0] = max(most[0], inside[0])
        time.sleep(0.1)
        inside[0] -= 1

    install(launch=launch)
    call(64)
    _run([lambda: call(64)] * 3)
    assert most[0] == 1
