"""What the binding does around the library's calls, with a stand-in for the library and for torch's streams: which call comes
after which, and which work is ordered behind which."""
import gc

import pytest
import torch

from paper_1810_08403_amd import binding as B


class Stream:
    """`seen`: the operations that are done before anything enqueued from now on starts."""
    def __init__(self, handle):
        self.cuda_stream, self.seen = handle, set()

    def enqueue(self, what):
        self.seen.add(what)

    def wait_stream(self, other):
        self.seen |= other.seen


class Library:
    """Every graph_create is a piece of work on the context's stream; `behind[i]`: what was done before the i-th started."""
    def __init__(self, streams):
        self.streams, self.current, self.made = streams, None, Stream("the library's own")
        self.log, self.behind, self.alive = [], [], set()

    def saga_create(self, out, device, stream, budget):
        out._obj.value = 77
        self.alive.add(77)
        self.current = self.streams[stream.value] if stream.value else self.made
        return 0

    def saga_set_stream(self, ctx, stream, ordered):
        to = self.streams[stream or 0]
        if ordered:
            to.wait_stream(self.current)
        self.current = to
        return 0

    def saga_graph_create_csc(self, ctx, n, nnz, col_ptr, row_idx, where, out):
        assert 77 in self.alive
        self.behind.append(set(self.current.seen))
        self.current.enqueue(("call", len(self.behind) - 1))
        out._obj.value = 1000 + len(self.behind)
        self.alive.add(out._obj.value)
        return 0

    def saga_graph_destroy(self, g):
        g = getattr(g, "value", g)
        self.log.append("graph_destroy" if 77 in self.alive else "graph_destroy after its context")
        self.alive.remove(g)
        return 0

    def saga_destroy(self, ctx):
        self.alive.remove(77)
        self.log.append("destroy")
        return 0

    def saga_last_error(self, ctx):
        return b""


@pytest.fixture
def fake(monkeypatch):
    """(library, streams by handle, what torch's current stream is): handle 0 is the default stream."""
    streams = {0: Stream(0)}
    state = {"current": streams[0], "capturing": False, "device": 0, "capturing_on": 0}

    def new_stream(device=None):
        s = Stream(len(streams))
        streams[s.cuda_stream] = s
        return s

    lib = Library(streams)
    monkeypatch.setattr(B, "load_library", lambda: lib)
    monkeypatch.setattr(torch.cuda, "is_available", lambda: True)
    monkeypatch.setattr(torch.cuda, "Stream", new_stream)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: state["current"])
    monkeypatch.setattr(torch.cuda, "default_stream", lambda device=None: streams[0])
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: state["capturing"] and state["device"] == state["capturing_on"])

    class Device:
        def __init__(self, device):
            self.device = device

        def __enter__(self):
            self.before, state["device"] = state["device"], self.device

        def __exit__(self, *exc):
            state["device"] = self.before

    monkeypatch.setattr(torch.cuda, "device", Device)
    return lib, streams, state


def _graph(ctx):
    return ctx.graph_create_csc(1, torch.zeros(2, dtype=torch.int64), torch.zeros(0, dtype=torch.int32))


@pytest.mark.parametrize("context_first", [True, False])
def test_a_context_and_its_graphs_collected_together(fake, context_first):
    """The collector clears weak references before it calls finalisers, and calls them in any order."""
    lib = fake[0]
    gc.collect()
    ctx = B.Context(0)
    graphs = [_graph(ctx), _graph(ctx)]
    if context_first:
        ctx.cycle = graphs           # (and a graph refers to its context)
    else:
        cell = [graphs, ctx]
        cell.append(cell)
        del cell
    del ctx, graphs
    gc.collect()
    assert lib.log == ["graph_destroy", "graph_destroy", "destroy"] and not lib.alive


def test_graphs_outlive_their_destroyed_context_as_empty_handles(fake):
    lib = fake[0]
    ctx = B.Context(0)
    g, other = _graph(ctx), _graph(ctx)
    other.destroy()
    ctx.destroy()
    assert lib.log == ["graph_destroy", "graph_destroy", "destroy"] and not g._h
    g.destroy()
    ctx.destroy()
    assert len(lib.log) == 3


def _call(lib, ctx, streams, under):
    """One call with torch's current stream `under`, after work of the program there; the call's number."""
    under.enqueue(("before", len(lib.behind)))
    _graph(ctx)
    i = len(lib.behind) - 1
    assert ("before", i) in lib.behind[i], "the call does not wait for what the program enqueued before it"
    assert ("call", i) in under.seen, "what the program enqueues after the call does not wait for it"
    return i


@pytest.mark.parametrize("given", ["none", "a stream", "the default stream"])
def test_calls_are_ordered_like_torch_operations(fake, given):
    """Whichever stream the context was given and whichever is current, also in turn: behind the program's earlier work there,
    ahead of its later work, and behind the call before (the workspaces are shared)."""
    lib, streams, state = fake
    stream = {"none": None, "a stream": torch.cuda.Stream(), "the default stream": streams[0]}[given]
    ctx = B.Context(0, stream=stream)
    side = torch.cuda.Stream()
    for k, under in enumerate([streams[0], streams[0], side, streams[0], side, side, stream or streams[0], streams[0]]):
        state["current"] = under
        i = _call(lib, ctx, streams, under)
        assert k == 0 or ("call", i - 1) in lib.behind[i]
    ctx.destroy()


def test_the_stream_attribute_orders_what_waits_for_it(fake):
    """`stream` was the stream all calls run on, and programs wait on it: with the context following the default stream, what
    waits on `stream` still waits for the calls, read after them, read before them and kept, or read twice."""
    lib, streams, state = fake
    ctx = B.Context(0)
    waiting = torch.cuda.Stream()
    i = _call(lib, ctx, streams, streams[0])
    assert lib.current is streams[0]           # nobody asked: the call runs on the default stream itself
    kept = ctx.stream
    assert kept.cuda_stream != 0               # a stream that can be captured from
    waiting.wait_stream(kept)
    assert ("call", i) in waiting.seen
    for under in (streams[0], waiting, streams[0], kept):
        state["current"] = under
        i = _call(lib, ctx, streams, under)
        later = torch.cuda.Stream()
        later.wait_stream(kept)
        assert ("call", i) in later.seen and ctx.stream is kept
    ctx.destroy()
    assert ctx.stream is kept

    given = torch.cuda.Stream()
    assert B.Context(0, stream=given).stream is given
    assert B.Context(0, stream=streams[0]).stream is streams[0]


def test_the_stream_attribute_read_during_a_capture(fake):
    """No event from outside may enter a capture: the order is made by the first call after it."""
    lib, streams, state = fake
    ctx = B.Context(0)
    i = _call(lib, ctx, streams, streams[0])
    state["current"], state["capturing"] = torch.cuda.Stream(), True
    kept = ctx.stream
    assert not kept.seen
    state["current"], state["capturing"] = streams[0], False
    j = _call(lib, ctx, streams, streams[0])
    assert ("call", i) in lib.behind[j] and ("call", j) in kept.seen
    ctx.destroy()


def test_a_capture_on_the_context_s_device_is_seen_from_another_device(fake):
    """Which device is current has no say in it: streams are asked for on the context's."""
    lib, streams, state = fake
    ctx = B.Context(1)
    i = _call(lib, ctx, streams, streams[0])
    capture = torch.cuda.Stream()
    state.update(current=capture, capturing=True, capturing_on=1, device=0)
    _graph(ctx)
    assert ("call", i) not in lib.behind[-1]     # no event from outside enters the capture, and
    assert lib.current is streams[0]             # the context is back on the default stream after the call
    ctx.destroy()
