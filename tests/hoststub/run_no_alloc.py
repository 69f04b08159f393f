"""saga_layer_forward_noalloc on the CPU stand-in of the HIP runtime: the call must reach no allocator (the stand-in
counts hipMalloc / hipFree / hipHostMalloc / hipHostFree and stream and event creations), must give the bits of the
ordinary call, must refuse a row width whose work list has not been built and a layer that does not fit the scratch array.

  python tests/hoststub/run_no_alloc.py <library>"""
import os
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
TESTS = os.path.dirname(HERE)
sys.path[:0] = [os.path.dirname(TESTS), TESTS, HERE]

import numpy as np
import torch

import saga_inputs as si
from paper_1810_08403_amd import binding as B
from stub_binding import StubContext, dev


def dense_blocks_near_the_limit(lib, rng):
    """bf16 sums whose dense blocks, in chunks of the length that is taken by their number, write more partial rows than the
    scratch array holds, and in longer chunks do not: accepted, in those chunks, while the ordinary call keeps the short ones; and in a
    context with a budget, no more partial rows than the longest chunks write."""
    src, dst = si.rmat_edges(9, 40 << 9, 909)
    g = si.build_csc(1 << 9, src, dst, symmetrise=True, self_loops=True)

    def context(budget=0, **options):
        ctx = StubContext(lib, budget)
        for k, v in dict(dense_min_edges=8, dense_tile_gain=0, stripe_kb=0, **options).items():  # (no bands: the same pieces for every width)
            ctx.set_option(k, v)
        ctx.set_profiling(True)
        return ctx, ctx.graph_create_csc(g.n, dev(g.col_ptr), dev(g.row_idx))

    def layer(F, Fo):
        X = dev(torch.as_tensor(rng.standard_normal((g.n, F)).astype(np.float32)).to(torch.bfloat16))
        kw = dict(W=dev(torch.full((F, Fo), 0.01).to(torch.bfloat16))) if Fo else {}

        def call(ctx, h, no_alloc=False):
            Y = dev(torch.full((g.n, Fo or F), float("nan"), dtype=torch.bfloat16))
            before = ctx.lib.stub_allocator_calls()
            ctx.layer_forward(h, X, Y, edge_op="copy", no_alloc=no_alloc, **kw)
            calls = ctx.lib.stub_allocator_calls() - before
            ctx.synchronize()
            assert not torch.isnan(Y.t.float()).any() and not (no_alloc and calls)
            return Y.t, calls, ctx.get_timings()["n_partial_rows"]
        return call

    rows = {}
    for chunk in (5, 10, 128):
        ctx, h = context(dense_chunk=chunk)
        rows[chunk] = layer(128, 0)(ctx, h)[2]
        h.destroy()
        ctx.destroy()
    mib = lambda n_rows, F: n_rows * F * 4 / 2 ** 20
    wide, narrow = 11008, 128
    beside = 2 * wide * (512 + 128) / 2 ** 20     # bf16 rows before the product, and weights of up to 128 columns
    assert mib(rows[128], wide) < mib(rows[10], wide) + beside < 64 < mib(rows[5], wide) + beside and mib(rows[5], wide) < 64, rows
    assert mib(rows[5], 16384) > 64 > mib(rows[10], 16384)
    checked = 0
    # the ordinary call's chunks, those of the call that must not allocate
    for F, Fo, budget, length, fits in ((wide, 3, 0, 5, 10), (16384, 0, 0, 5, 10), (narrow, 3, 0, 5, 5), (narrow, 3, 1 << 30, 128, 128)):
        ctx, h = context(budget)
        call = layer(F, Fo)
        Y0, _, n0 = call(ctx, h)
        Y1, _, n1 = call(ctx, h, no_alloc=True)
        Y2, calls, n2 = call(ctx, h)
        assert n0 == n2 == rows[length] and n1 == rows[fits] and calls == 0, (F, Fo, budget, n0, n1, n2, rows)
        assert torch.equal(Y0, Y2)
        if length == fits:
            assert torch.equal(Y0, Y1)
        else:   # other groups of the same fp32 sums, rounded to bf16 before the product and behind it
            assert float((Y0.double() - Y1.double()).norm() / Y0.double().norm()) < 2.0 ** -8
        h.destroy()
        ctx.destroy()
        checked += 1
    # two layers of one width, of which one fits with the shortest chunks and the other does not: made at the ordinary call that needs
    # them, but not while its stream is captured; a call that must not allocate takes the shortest that are there and fit
    ctx, h = context()
    with_w, without = layer(wide, 3), layer(wide, 0)
    first = without(ctx, h)[0]
    assert torch.equal(without(ctx, h, no_alloc=True)[0], first)
    try:
        with_w(ctx, h, no_alloc=True)
        raise AssertionError("chunks that nothing has made yet were taken")
    except B.SagaError as e:
        assert e.status == 4, e
    large = layer(wide, 3)
    large(ctx, h)                                  # (grows the workspaces, and makes the longer chunks)
    h.destroy()
    h = ctx.graph_create_csc(g.n, dev(g.col_ptr), dev(g.row_idx))
    without(ctx, h)
    ctx.lib.stub_set_capturing(1)
    _, calls, n = with_w(ctx, h)
    assert calls == 0 and n == rows[5], "a plan was built while a stream was captured"
    ctx.lib.stub_set_capturing(0)
    _, calls, n = with_w(ctx, h)
    assert calls > 0 and n == rows[5]
    assert with_w(ctx, h, no_alloc=True)[2] == rows[10]
    assert without(ctx, h, no_alloc=True)[2] == rows[5]
    assert with_w(ctx, h)[1] == without(ctx, h)[1] == 0, "a plan that was there is built again"
    h.destroy()
    ctx.destroy()
    return checked + 1


def main():
    lib = sys.argv[1]
    rng = np.random.default_rng(11)
    t = lambda *shape, s=1.0: torch.as_tensor((rng.standard_normal(shape) * s).astype(np.float32))
    ctx = StubContext(lib)
    ctx.set_mode(2, 5)
    checked = 0
    for n, m, hub in ((700, 9000, True), (150, 900, False)):          # the second graph is smaller: stale scratch contents must not show
        edges = set(zip(rng.integers(n, size=m).tolist(), rng.integers(n, size=m).tolist()))
        if hub:
            edges |= {(u, 3) for u in range(n)}                        # a column that is cut into pieces: partial rows in the scratch
        g = si.csc_from_lists(n, sorted(edges))
        h = ctx.graph_create_csc(n, dev(g.col_ptr), dev(g.row_idx))
        w = t(g.nnz)
        for op, F, Fo, agg in (("mul_weight", 24, 8, "sum"), ("copy", 24, 5, "max"), ("gated", 8, 4, "sum"), ("pool", 12, 4, "max")):
            X, W, bias = t(n, F), t(F, Fo, s=0.3), t(Fo, s=0.2)
            kw = {}
            if op == "mul_weight":
                kw["edge_weight"] = dev(w)
            if op == "gated":
                kw.update(W_gate=dev(t(F, 2 * F, s=0.3)), b_gate=dev(t(F, s=0.2)))
            if op == "pool":
                kw.update(W_pool=dev(t(F, F, s=0.3)), b_pool=dev(t(F, s=0.2)))
            args = dict(edge_op=op, agg=agg, W=dev(W), bias=dev(bias), act="relu", **kw)
            Y0, A0 = dev(torch.full((n, Fo), float("nan"))), dev(torch.full((n, F), float("nan")))
            Y1, A1 = dev(torch.full((n, Fo), float("nan"))), dev(torch.full((n, F), float("nan")))
            ctx.layer_forward(h, dev(X), Y0, accum_out=A0, **args)                # builds the work list for this row width
            before = ctx.lib.stub_allocator_calls()
            ctx.layer_forward(h, dev(X), Y1, accum_out=A1, no_alloc=True, **args)
            assert ctx.lib.stub_allocator_calls() == before, f"{op}: the no-allocation call reached an allocator"
            ctx.synchronize()                                                       # resident calls return after enqueueing
            assert torch.equal(Y0.t, Y1.t) and torch.equal(A0.t, A1.t), f"{op} n={n}: results differ from the ordinary call"
            assert not torch.isnan(Y1.t).any()
            checked += 1
        # a row width nobody has run yet: refused, not built
        try:
            ctx.layer_forward(h, dev(t(n, 200)), dev(torch.empty(n, 200)), edge_op="copy", no_alloc=True)
            raise AssertionError("a missing work list was accepted")
        except B.SagaError as e:
            assert e.status == 3, e
        h.destroy()
    # a layer that does not fit the 64 MiB: refused with SAGA_ERR_BUDGET, and the next call still works
    n, F = 9000, 2048
    g = si.csc_from_lists(n, [(i, (i * 7) % n) for i in range(n)])
    h = ctx.graph_create_csc(n, dev(g.col_ptr), dev(g.row_idx))
    X, W = torch.zeros(n, F), torch.zeros(F, 4)
    Y = dev(torch.empty(n, 4))
    ctx.layer_forward(h, dev(X), Y, edge_op="copy", W=dev(W))
    try:
        ctx.layer_forward(h, dev(X), Y, edge_op="copy", W=dev(W), no_alloc=True)
        raise AssertionError("a layer beyond the scratch size was accepted")
    except B.SagaError as e:
        assert e.status == 4, e
    ctx.layer_forward(h, dev(X), Y, edge_op="copy", W=dev(W))
    h.destroy()
    # layers whose fp32 matrices fit the 64 MiB and whose packed weights (K padded to 32, three bf16 parts a value) do not: one
    # product of 50 MiB, the same after a per-vertex product that was counted with a little more, a second operand, and a gated
    # layer whose gap between the packed columns must not count
    n = 5
    h = ctx.graph_create_csc(n, dev(torch.arange(n + 1, dtype=torch.int64)), dev(torch.arange(n, dtype=torch.int32)))
    for op, F, Fm, Fo, with_self in (("copy", 16, 16, 800000, False), ("pool", 98560, 16, 786560, False), ("copy", 3, 3, 400001, True),
                                     ("gated", 2000, 2000, 3, False)):
        X, W = t(n, F), t(Fm, Fo, s=0.3)
        kw = dict(edge_op=op, W=dev(W), bias=dev(t(Fo)))
        if op == "pool":
            kw.update(W_pool=dev(t(Fm, F, s=0.01)), b_pool=dev(t(Fm)), agg="max")
        if op == "gated":
            kw.update(W_gate=dev(t(F, 2 * F, s=0.01)), b_gate=dev(t(F)))
        if with_self:
            kw["W_self"] = dev(t(F, Fo))
        Y0, Y1 = dev(torch.full((n, Fo), float("nan"))), dev(torch.full((n, Fo), float("nan")))
        ctx.layer_forward(h, dev(X), Y0, **kw)
        before = ctx.lib.stub_allocator_calls()
        ctx.layer_forward(h, dev(X), Y1, no_alloc=True, **kw)
        assert ctx.lib.stub_allocator_calls() == before
        ctx.synchronize()
        assert torch.equal(Y0.t, Y1.t) and not torch.isnan(Y1.t).any(), f"{op} {F} {Fm} {Fo}"
        checked += 1
    h.destroy()
    ctx.destroy()
    checked += dense_blocks_near_the_limit(lib, rng)
    print(f"ok: {checked} layers, no allocator reached", flush=True)


if __name__ == "__main__":
    main()
