"""saga_layer_forward_noalloc (the entry point for callers that must not allocate) against saga_layer_forward, through
the C ABI on the GPU: same bits, on two calls in a row of which the second is smaller, so that what the first call left
in the shared static scratch array would show if the second read any of it."""
import numpy as np
import pytest
import torch

import saga_inputs as si

pytestmark = pytest.mark.gpu


def _graph(rng, n, m, hub):
    edges = set(zip(rng.integers(n, size=m).tolist(), rng.integers(n, size=m).tolist()))
    if hub:
        edges |= {(u, 5) for u in range(n)}        # a column long enough to be cut into pieces: partial rows in the scratch
    return si.csc_from_lists(n, sorted(edges))


@pytest.mark.parametrize("op,agg,dtype", [("mul_weight", "sum", torch.float32), ("copy", "max", torch.float32),
                                          ("mul_weight", "sum", torch.bfloat16), ("gated", "sum", torch.float32),
                                          ("pool", "max", torch.float32)])
@pytest.mark.parametrize("small_layer", [0, 1])   # 0: the second call, too, is several launches with rows and weights in the scratch
def test_no_alloc_matches_the_ordinary_call(op, agg, dtype, small_layer):
    import paper_1810_08403_amd as saga
    rng = np.random.default_rng(21)
    t = lambda *shape, s=1.0: torch.as_tensor((rng.standard_normal(shape) * s).astype(np.float32)).cuda()
    ctx = saga.Context(0)
    ctx.set_option("small_layer", small_layer)
    for n, m, hub, F, Fo in ((6000, 90000, True, 128, 64), (700, 5000, False, 64, 16)):   # the second call is the smaller one
        g = _graph(rng, n, m, hub)
        h = ctx.graph_create_csc(n, g.col_ptr.cuda(), g.row_idx.cuda())
        X, W, bias = t(n, F).to(dtype), t(F, Fo, s=0.3).to(dtype), t(Fo, s=0.2)
        kw = {}
        if op == "mul_weight":
            kw["edge_weight"] = t(g.nnz)
        if op == "gated":
            kw.update(W_gate=t(F, 2 * F, s=0.2), b_gate=t(F, s=0.2), W_msg=t(F, F, s=0.2))
        if op == "pool":
            kw.update(W_pool=t(F, F, s=0.2), b_pool=t(F, s=0.2))
        args = dict(edge_op=op, agg=agg, W=W, bias=bias, act="relu", **kw)
        Y0, A0 = torch.full((n, Fo), float("nan"), device="cuda", dtype=dtype), torch.full((n, F), float("nan"), device="cuda")
        Y1, A1 = torch.full_like(Y0, float("nan")), torch.full_like(A0, float("nan"))
        ctx.layer_forward(h, X, Y0, accum_out=A0, **args)             # the ordinary call also builds the work list for this width
        ctx.layer_forward(h, X, Y1, accum_out=A1, no_alloc=True, **args)
        torch.cuda.synchronize()
        what = f"{op} {agg} {dtype} n={n} F={F}->{Fo}"
        assert not torch.isnan(Y1.float()).any() and not torch.isnan(A1).any(), what
        assert torch.equal(Y0, Y1), what + ": Y differs from saga_layer_forward"
        assert torch.equal(A0, A1), what + ": the Gather output differs from saga_layer_forward"
        assert h.info()["n_split_vertices"] > 0 or not hub, what
        h.destroy()
    ctx.destroy()


def test_no_alloc_refusals():
    import paper_1810_08403_amd as saga
    rng = np.random.default_rng(22)
    ctx = saga.Context(0)
    n = 9000
    g = si.csc_from_lists(n, [(i, (i * 7) % n) for i in range(n)])
    h = ctx.graph_create_csc(n, g.col_ptr.cuda(), g.row_idx.cuda())
    X = torch.zeros(n, 2048, device="cuda")
    W = torch.zeros(2048, 4, device="cuda")
    Y = torch.empty(n, 4, device="cuda")
    with pytest.raises(saga.SagaError) as e:                          # no work list for this row width yet
        ctx.layer_forward(h, X, Y, edge_op="copy", W=W, no_alloc=True)
    assert e.value.status == 3
    ctx.layer_forward(h, X, Y, edge_op="copy", W=W)
    with pytest.raises(saga.SagaError) as e:                          # 9000 x 2048 x 4 bytes of Gather output: beyond 64 MiB
        ctx.layer_forward(h, X, Y, edge_op="copy", W=W, no_alloc=True)
    assert e.value.status == 4 and "scratch" in str(e.value)
    Xs, Ws, Ys = X[:, :256].contiguous(), W[:256].contiguous(), torch.full((n, 4), float("nan"), device="cuda")
    ctx.layer_forward(h, Xs, Y, edge_op="copy", W=Ws)
    ctx.layer_forward(h, Xs, Ys, edge_op="copy", W=Ws, no_alloc=True)   # and a layer that fits goes through afterwards
    torch.cuda.synchronize()
    assert torch.equal(Y, Ys)
    h.destroy()
    ctx.destroy()


# layers whose fp32 matrices fit the 64 MiB and whose packed weights (K padded to 32, three bf16 parts a value) do not: packed
# and multiplied some columns at a time; one product, the second of two, two operands
@pytest.mark.parametrize("op,F,Fm,Fo,with_self", [("copy", 16, 16, 800000, False), ("pool", 98560, 16, 786560, False), ("copy", 3, 3, 400001, True)])
def test_no_alloc_with_more_packed_weights_than_scratch(op, F, Fm, Fo, with_self):
    import paper_1810_08403_amd as saga
    n = 70
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    t = lambda *shape: torch.randn(*shape, generator=g, device="cuda")
    ctx = saga.Context(0)
    h = ctx.graph_create_csc(n, torch.arange(n + 1, device="cuda"), torch.arange(n, dtype=torch.int32, device="cuda"))
    X = t(n, F)
    kw = dict(edge_op=op, W=t(Fm, Fo), bias=t(Fo))
    if op == "pool":
        kw.update(W_pool=t(Fm, F) * 0.01, b_pool=t(Fm), agg="max")
    if with_self:
        kw["W_self"] = t(F, Fo)
    Y0, Y1 = torch.full((n, Fo), float("nan"), device="cuda"), torch.full((n, Fo), float("nan"), device="cuda")
    A = torch.full((n, Fm), float("nan"), device="cuda")
    ctx.layer_forward(h, X, Y0, accum_out=A, **kw)
    ctx.layer_forward(h, X, Y1, no_alloc=True, **kw)
    torch.cuda.synchronize()
    assert torch.equal(Y0, Y1) and not torch.isnan(Y1).any()
    ref, scale = A.double() @ kw["W"].double() + kw["bias"].double(), A.double().abs() @ kw["W"].double().abs() + kw["bias"].double().abs()
    if with_self:
        ref, scale = ref + X.double() @ kw["W_self"].double(), scale + X.double().abs() @ kw["W_self"].double().abs()
    assert ((Y1.double() - ref).abs() / scale).max().item() <= 1e-5
    h.destroy()
    ctx.destroy()


@pytest.mark.parametrize("first,then", [(dict(F=128), dict(F=64)), (dict(F=128), dict(F=128, mma=1))])
def test_no_alloc_takes_a_list_built_for_another_width_or_without_mma(first, then):
    """Without bands the work list is the same for every width, and it is the same with and without the matrix unit: the
    call without allocations takes it (items that four wavefronts share are in it) and gives the ordinary call's bits."""
    import paper_1810_08403_amd as saga
    rng = np.random.default_rng(3)
    n = 6000
    g = _graph(rng, n, 90000, True)
    ctx = saga.Context(0)
    ctx.set_option("stripe_kb", 0)
    ctx.set_option("cut_degree", 1 << 20)                     # the hub is one long item
    h = ctx.graph_create_csc(n, g.col_ptr.cuda(), g.row_idx.cuda())
    X = torch.as_tensor(rng.standard_normal((n, 128)).astype(np.float32)).cuda().bfloat16()
    out = lambda F: torch.full((n, F), float("nan"), device="cuda")
    Y = lambda F: torch.empty(n, F, device="cuda", dtype=torch.bfloat16)
    run = lambda F, A, **kw: ctx.layer_forward(h, X[:, :F].contiguous(), Y(F), edge_op="copy", accum_out=A, **kw)
    run(first["F"], out(first["F"]))
    ctx.set_option("mma", then.get("mma", 0))
    F = then["F"]
    A0, A1 = out(F), out(F)
    run(F, A0, no_alloc=True)
    run(F, A1)
    torch.cuda.synchronize()
    assert not torch.isnan(A0).any() and torch.equal(A0, A1)
    dst, msg = torch.repeat_interleave(torch.arange(n), g.col_ptr.diff()).cuda(), X[g.row_idx.long().cuda(), :F].double()
    ref, scale = (torch.zeros(n, F, dtype=torch.float64, device="cuda").index_add_(0, dst, v) for v in (msg, msg.abs()))
    # at most 6,000 additions of exact messages, each off by a unit in the last place at most (the matrix unit truncates)
    assert ((A0.double() - ref).abs() <= 6000 * 2.0 ** -23 * scale).all()
    ctx.destroy()
