"""Which stream a context's calls go to and what they wait for, on a model of streams (no GPU).

A model stream knows the calls that are ordered before its next one; waiting for another stream
adds what that one knows.  Every eager call of a context shares its level buffers with the
calls before it, so it must know all of them, whatever streams they ran on."""
import threading

import pytest

torch = pytest.importorskip("torch")

from paper_2205_05840_amd import _lib, solver  # noqa: E402


class Stream:
    """torch numbers its own streams; one made elsewhere is numbered by its handle."""

    def __init__(self, world, handle, external=False):
        self.world, self.cuda_stream = world, handle
        self.stream_id = handle if external else len(world.streams)
        self.known, self.alive = set(), True
        world.streams[handle] = self

    def wait_stream(self, other):
        assert self.alive and other.alive, "a destroyed stream"
        self.known |= other.known

    def synchronize(self):
        assert self.alive, "a destroyed stream"


class OnDevice:
    def __init__(self, world, index):
        self.world, self.index = world, index

    def __enter__(self):
        self.before, self.world.device = self.world.device, self.index

    def __exit__(self, *exc):
        self.world.device = self.before


class World:
    """The streams, the caller's current one, the library's bound one and the calls made."""

    def __init__(self, monkeypatch):
        self.streams, self.calls, self.capturing = {}, [], None
        self.device = 0   # the current device
        self.current = Stream(self, 0)
        mp = monkeypatch
        mp.setattr(torch.cuda, "Stream", lambda device=None: Stream(self, 1000 + len(self.streams)))
        self.mine = threading.local()   # a thread's own current stream
        mp.setattr(torch.cuda, "current_stream", lambda device=None: getattr(self.mine, "stream", self.current))
        mp.setattr(torch.cuda, "is_current_stream_capturing", lambda: self.capturing is self.current)
        mp.setattr(torch.cuda, "current_device", lambda: self.device)
        mp.setattr(torch.cuda, "device", lambda d: OnDevice(self, torch.device(d).index))
        mp.setattr(_lib, "ndmg_set_stream", self.set_stream)
        empty = torch.empty
        mp.setattr(torch, "empty", lambda *a, device=None, **k: empty(*a, **k))
        self.ctx = solver._Context()
        self.ctx._alloc(16, "cuda:0")
        self.ctx.ctx = 1
        self.bound = self.ctx.stream   # (setup passes the context's own stream)

    def set_stream(self, ctx, handle):
        self.bound = self.streams[handle]

    def fn(self, ctx, name):
        """A library call: its name goes into what its stream knows."""
        st = self.bound
        assert st.alive, "a destroyed stream"
        if not self.capturing:
            self.calls.append((name, st, set(st.known)))
            st.known.add(name)
        return name

    def eager_calls_are_ordered(self):
        for i, (name, _, known) in enumerate(self.calls):
            missing = {n for n, _, _ in self.calls[:i]} - known
            assert not missing, (name, missing)


@pytest.fixture
def world(monkeypatch):
    w = World(monkeypatch)
    yield w
    w.ctx.ctx = None   # (no library context behind it)


def test_steps_and_solves_follow_each_other(world):
    a, b = Stream(world, 11), Stream(world, 13)
    for i, (s, solve) in enumerate([(a, 0), (b, 0), (b, 1), (a, 0), (a, 0), (b, 1), (b, 0)]):
        world.current = s
        (world.ctx._run if solve else world.ctx._step)(world.fn, f"call {i}")
        assert world.calls[-1][1] is (world.ctx.stream if solve else s)
    world.eager_calls_are_ordered()


@pytest.mark.parametrize("after", ["step", "solve"])
def test_work_before_a_capture_is_waited_for_after_it(world, after):
    a, b, c = Stream(world, 11), Stream(world, 13), Stream(world, 17)
    world.current = a
    world.ctx._step(world.fn, "before")
    world.current = world.capturing = b   # (a raw capture: nothing has waited for a)
    world.ctx._step(world.fn, "captured")
    world.capturing, world.current = None, c
    (world.ctx._step if after == "step" else world.ctx._run)(world.fn, "after")
    world.eager_calls_are_ordered()


def test_a_stream_of_the_caller_may_end_after_its_work(world):
    ext = Stream(world, 4096, external=True)
    world.current = ext
    world.ctx._step(world.fn, "first")
    assert "first" in ext.known   # what the caller does next on it follows the step
    ext.alive = False             # synchronised and destroyed by the caller
    world.current = Stream(world, 11)
    world.ctx._step(world.fn, "second")
    world.ctx._run(world.fn, "third")
    world.eager_calls_are_ordered()
    world.ctx._last.synchronize()   # (as closing the context does)


@pytest.mark.parametrize("call", ["_step", "_run"])
def test_calls_run_on_the_context_s_device(world, call):
    """(the default stream's handle, 0, names the current device's: a launch there must find the
    context's device current)"""
    world.ctx.device = torch.device("cuda:1")
    at = []

    def fn(ctx):
        at.append(world.device)

    for current in (0, 1):
        world.device = current
        getattr(world.ctx, call)(fn)
        assert world.device == current
    assert at == [1, 1]


def test_calls_from_two_threads_keep_their_streams(world):
    """A second thread's step, let in between the first one's choice of stream and its launch
    (if the context lets it), must not take the stream from under it."""
    a, b = Stream(world, 11), Stream(world, 13)
    bind, between, done = world.set_stream, threading.Event(), threading.Event()

    def set_stream(ctx, handle):
        bind(ctx, handle)
        if handle == a.cuda_stream:
            between.set()
            done.wait(0.5)   # (a context that makes the second thread wait lets this time out)

    _lib.ndmg_set_stream = set_stream   # (restored by the fixture)

    def second():
        world.mine.stream = b
        between.wait(5)
        world.ctx._step(world.fn, "second")
        done.set()

    t = threading.Thread(target=second)
    t.start()
    world.mine.stream = a
    world.ctx._step(world.fn, "first")
    t.join(5)
    assert not t.is_alive()
    assert {name: st for name, st, _ in world.calls} == {"first": a, "second": b}
    world.eager_calls_are_ordered()
