"""Which layers go out in one launch, and their results, on the CPU stand-in: inside the rule, at its borders, and where outputs
share memory with each other or with something that is read.

  python tests/hoststub/run_small_layers.py <library>"""
import ctypes
import os
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
TESTS = os.path.dirname(HERE)
sys.path[:0] = [os.path.dirname(TESTS), TESTS, HERE]

import numpy as np
import torch

import oracle
from helpers import assert_sum_close
from stub_binding import Dev, StubContext, dev


def regular(n, deg):
    """Every column with `deg` sources, the first with one edge more."""
    rows = [np.sort((v * 7 + np.arange(deg + (v == 0)) * 3) % n) for v in range(n)]
    return torch.from_numpy(np.concatenate([[0], np.cumsum([len(r) for r in rows])])), torch.from_numpy(np.concatenate(rows).astype(np.int32))


def main():
    lib = sys.argv[1]
    rng = np.random.default_rng(3)
    t = lambda *s: torch.as_tensor(rng.standard_normal(s).astype(np.float32))
    ctx = StubContext(lib)
    ctx.lib.stub_small_launches.restype = ctypes.c_int64
    checked = 0

    def graph(n, deg):
        cp, ri = regular(n, deg)
        return n, cp, ri, ctx.graph_create_csc(n, dev(cp), dev(ri))

    def layer(g, F, N, one_launch, place=None, op="copy", agg="sum", act="relu", self_=False):
        nonlocal checked
        n, cp, ri, h = g
        X, W, bias = t(n, F), t(F, N), t(N)
        w = t(ri.numel())
        # (views keep their strides as Dev tensors of their own)
        mem = torch.full((n, F + N), float("nan"))
        Xd, Wd, bd, wd = dev(X), dev(W), dev(bias), dev(w)
        Yd, Ad = dev(torch.full((n, N), float("nan"))), dev(torch.full((n, F), float("nan")))

        def view(x):
            d = Dev(torch.empty(0))
            d.t = x
            return d
        if place == "Y in X":
            Xd, Yd = view(mem[:, :F]), view(mem[:, :N])
            Xd.t.copy_(X)
        elif place == "A in Y":
            Yd, Ad = view(mem[:, :N]), view(mem[:, 1:1 + F])
        elif place == "A in W":
            Wd = view(mem.view(-1)[F:F + F * N].view(F, N))
            Wd.t.copy_(W)
            Ad = view(mem.view(-1)[:n * F].view(n, F))
        elif place == "A in bias":
            bd = view(mem.view(-1)[F:F + N])
            bd.t.copy_(bias)
            Ad = view(mem.view(-1)[:n * F].view(n, F))
        elif place == "no A":
            Ad = None
        kw = dict(W=Wd, bias=bd, act=act, agg=agg, edge_op=op, accum_out=Ad)
        if op == "mul_weight":
            kw["edge_weight"] = wd
        if self_:
            kw["W_self"] = dev(t(F, N))
        before = ctx.lib.stub_small_launches()
        ctx.layer_forward(h, Xd, Yd, **kw)
        ctx.synchronize()
        took = ctx.lib.stub_small_launches() - before
        assert took == int(one_launch), (n, F, N, place, op, agg, took)
        ref = oracle.layer(cp.numpy(), ri.numpy(), X.numpy(), op, w.numpy() if op == "mul_weight" else None, agg=agg, W=W.numpy(), bias=bias.numpy(), act=act)
        if place in (None, "no A", "Y in X") and not self_:
            assert_sum_close(Yd.t.numpy(), ref["Y"], ref["Y_abs"], 1e-5, f"{n} {F} {N} {place}")
            if Ad is not None:
                assert_sum_close(Ad.t.numpy(), ref["A"], ref["A_abs"], 1e-5, f"{n} {F} {N} {place} A")
        checked += 1

    g = graph(700, 8)
    for op in ("copy", "mul_weight"):
        for agg in ("sum", "max"):
            layer(g, 64, 64, True, op=op, agg=agg)
            layer(g, 64, 64, True, op=op, agg=agg, place="no A", act="sigmoid")
    for F, N, one in ((12, 16, False), (13, 16, True), (128, 16, True), (129, 16, False), (64, 256, True), (64, 257, False), (96, 160, True), (96, 161, False)):
        layer(g, F, N, one)
    layer(g, 64, 64, False, self_=True)
    for place in ("Y in X", "A in Y", "A in W", "A in bias"):
        layer(g, 64, 64, False, place=place)
    long = graph(300, 95)
    layer(long, 64, 64, True)                     # the first column has 96 edges
    longer = graph(300, 96)
    layer(longer, 64, 64, False)                   # 97
    ctx.set_option("small_layer", 0)
    layer(g, 64, 64, False)
    ctx.set_option("small_layer", 1)
    # 32,768 columns of at most 16 edges: sums of rows of eight fragments are k_gather_light's in separate launches, which adds them in
    # another order
    light = graph(32768, 2)
    for F, agg, one in ((28, "sum", True), (29, "sum", False), (32, "sum", False), (32, "max", True), (33, "sum", True)):
        layer(light, F, 8, one, agg=agg, place="no A")
    # as many steps in a row as are faster than several launches, of the longest column and the average one: two passes of rows of more
    # than 64 values, up to 260, 200 and 150 with one or two, up to four and more tiles of 32 outputs
    for deg, F, N, one in ((64, 128, 16, True), (65, 128, 16, False), (65, 64, 16, True), (49, 65, 65, True), (50, 65, 65, False),
                           (74, 64, 160, True), (75, 64, 160, False)):
        x = graph(300, deg)
        layer(x, F, N, one)
        x[3].destroy()
    # no limit where the rows are a workgroup per compute unit; two to a unit, three and four, and not more than LDS holds
    for n, deg, cases in ((2049, 94, ((128, 128, True), (64, 256, True))),
                          (8193, 45, ((64, 32, True), (64, 128, True), (16, 128, True), (16, 129, False), (64, 129, False), (128, 16, False), (65, 33, True),
                                      (97, 65, False))),
                          (12289, 45, ((128, 16, True),)),
                          (16385, 24, ((33, 16, True), (64, 16, True), (65, 16, False), (65, 64, True), (33, 96, True), (33, 97, False))),
                          (24577, 14, ((64, 64, True), (65, 16, False), (32, 96, True), (33, 96, False), (32, 160, False))),
                          (24577, 31, ((64, 64, False), (32, 64, True), (32, 96, False)))):
        x = graph(n, deg)
        for F, N, one in cases:
            layer(x, F, N, one, place="no A")
        x[3].destroy()
    for x in (g, long, longer, light):
        x[3].destroy()
    ctx.destroy()
    # no memory for rows that stay in the kernel
    n, cp, ri = 700, *regular(700, 8)
    peak = []
    for small in (0, 1):
        ctx = StubContext(lib)
        ctx.set_option("small_layer", small)
        h = ctx.graph_create_csc(n, dev(cp), dev(ri))
        at = ctx.peak_device_bytes()
        ctx.layer_forward(h, dev(t(n, 64)), dev(torch.empty(n, 64)), edge_op="copy", W=dev(t(64, 64)))
        ctx.synchronize()
        peak.append(ctx.peak_device_bytes() - at)
        h.destroy()
        ctx.destroy()
    assert peak[1] < n * 64 * 4 < peak[0], peak
    print(f"ok: {checked} layers", flush=True)


if __name__ == "__main__":
    main()
