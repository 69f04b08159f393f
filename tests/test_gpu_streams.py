"""Calls follow torch's current stream: the library runs on the default stream itself, and on a stream of its own, joined by
events, under any other. Its workspaces are shared by all calls of a context, so switching must keep calls in order."""
import pytest
import torch

import saga_inputs as si

pytestmark = pytest.mark.gpu


# the library's own choice of stream, a stream given at creation, the default stream given at creation (which records no graph)
@pytest.mark.parametrize("given", [False, True, "default"])
def test_alternating_streams_without_host_waits(given):
    import paper_1810_08403_amd as saga
    wl = si.workload(2, scale=13, f_in=96, f_out=40)
    n = wl.graph.n
    side, other = torch.cuda.Stream(), torch.cuda.Stream()
    if given == "default":
        other = torch.cuda.default_stream()
    ctx = saga.Context(0, stream=other) if given else saga.Context(0)
    h = ctx.graph_create_csc(n, wl.graph.col_ptr.cuda(), wl.graph.row_idx.cuda())
    w, W = wl.edge_weight.cuda(), wl.W.cuda()
    layer = lambda x, y: ctx.layer_forward(h, x, y, edge_op="mul_weight", edge_weight=w, W=W, act="relu")
    X = [torch.randn(n, 96, device="cuda") for _ in range(12)]
    want = []
    for x in X:
        want.append(torch.empty(n, 40, device="cuda"))
        layer(x, want[-1])
        torch.cuda.synchronize()
    got = [torch.full((n, 40), float("nan"), device="cuda") for _ in X]
    graphs = []
    main = torch.cuda.current_stream()
    for i, (x, y) in enumerate(zip(X, got)):
        if i % 3 == 0:                                # default stream, input made just before
            layer(x + 0.0, y)
        elif i % 3 == 1 or given == "default":        # a side stream that does not wait for the call before
            with torch.cuda.stream(side):
                layer(x, y)
        else:                                         # recorded in between: runs at its replay
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g):
                layer(x, y)
            graphs.append(g)
    main.wait_stream(side)
    for k in range(3):
        for g in graphs:
            g.replay()
        layer(X[0], got[0])
    ctx.synchronize()
    torch.cuda.synchronize()
    for i in range(len(X)):
        assert torch.equal(got[i], want[i]), f"call {i} differs"
    ctx.destroy()


@pytest.mark.parametrize("given", [False, True, "default"])
def test_workspaces_that_grow_from_stream_to_stream(given):
    """Every call needs more workspace than the one before and is made under another stream, with no host wait of the test's own
    between them: a workspace is not given back while a call on the stream before still uses it."""
    import paper_1810_08403_amd as saga
    wl = si.workload(2, scale=14, f_in=128, f_out=8)
    n = wl.graph.n
    side = torch.cuda.Stream()
    stream = {False: None, True: torch.cuda.Stream(), "default": torch.cuda.default_stream()}[given]
    sizes = [(66, 8), (80, 40), (100, 150), (128, 300)]    # one work list: bands of 2,048 rows for all of these widths
    X = [torch.randn(n, f, device="cuda") for f, _ in sizes]
    W = [torch.randn(f, fo, device="cuda") for f, fo in sizes]
    w = wl.edge_weight.cuda()
    want = []
    for x, m in zip(X, W):                                 # each with workspaces of its own
        c = saga.Context(0, stream=stream)
        want.append(torch.empty(n, m.shape[1], device="cuda"))
        c.layer_forward(c.graph_create_csc(n, wl.graph.col_ptr.cuda(), wl.graph.row_idx.cuda()), x, want[-1], edge_op="mul_weight", edge_weight=w, W=m)
        torch.cuda.synchronize()
        c.destroy()
    got = [torch.full_like(y, float("nan")) for y in want]
    torch.cuda.synchronize()
    ctx = saga.Context(0, stream=stream)
    h = ctx.graph_create_csc(n, wl.graph.col_ptr.cuda(), wl.graph.row_idx.cuda())
    for i, (x, m) in enumerate(zip(X, W)):
        with torch.cuda.stream(side if i % 2 else torch.cuda.default_stream()):
            ctx.layer_forward(h, x, got[i], edge_op="mul_weight", edge_weight=w, W=m)
    ctx.synchronize()
    torch.cuda.synchronize()
    for i in range(len(X)):
        assert torch.equal(got[i], want[i]), f"call {i} differs"
    ctx.destroy()


def test_waiting_on_the_stream_attribute():
    """A side stream that waits on `ctx.stream` alone sees a call made under the default stream, and a graph is captured on it."""
    import paper_1810_08403_amd as saga
    wl = si.workload(2, scale=15, f_in=128, f_out=128)
    n = wl.graph.n
    side = torch.cuda.Stream()
    ctx = saga.Context(0)
    h = ctx.graph_create_csc(n, wl.graph.col_ptr.cuda(), wl.graph.row_idx.cuda())
    w, W, X = wl.edge_weight.cuda(), torch.randn(128, 128, device="cuda"), torch.randn(n, 128, device="cuda")
    layer = lambda y: ctx.layer_forward(h, X, y, edge_op="mul_weight", edge_weight=w, W=W)
    want, got, graphed = (torch.full((n, 128), float("nan"), device="cuda") for _ in range(3))
    layer(want)
    torch.cuda.synchronize()
    seen = torch.full_like(got, float("nan"))
    for _ in range(20):
        layer(got)
    side.wait_stream(ctx.stream)
    with torch.cuda.stream(side):
        seen.copy_(got)
    torch.cuda.synchronize()
    assert torch.equal(seen, want)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=ctx.stream):
        layer(graphed)
    for _ in range(3):
        graphed.fill_(float("nan"))
        g.replay()
        layer(got)
        torch.cuda.synchronize()
        assert torch.equal(graphed, want) and torch.equal(got, want)
    ctx.destroy()
