"""The work lists of resident propagations, as the kernels get them: items that four wavefronts share are those past 128
edges where a band holds 4,096 rows, past 256 where it holds 32,768, past 1,024 otherwise, and the first of the list, and
there are none where no item of narrow rows is far above the average; light columns end it,
and lie behind it once more in order of length; every edge is in one item; forwards and backwards (edges by source), with and without bands, lists kept for another
width among them, on the CPU stand-in.

  python tests/hoststub/run_shared_items.py <library>"""
import ctypes
import os
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
TESTS = os.path.dirname(HERE)
sys.path[:0] = [os.path.dirname(TESTS), TESTS, HERE]

import numpy as np
import torch

import oracle
import saga_inputs as si
from helpers import assert_sum_close
from stub_binding import StubContext, dev


def last_list(ctx, capacity):
    items, by_length, counts = np.full((capacity, 4), -1, np.int32), np.full((capacity, 4), -1, np.int32), (ctypes.c_int64 * 4)()
    ctx.lib.stub_last_work_list(items.ctypes.data_as(ctypes.c_void_p), by_length.ctypes.data_as(ctypes.c_void_p), ctypes.c_int64(capacity), counts)
    n, team, light, light_edges = counts
    assert n <= capacity
    return items[:n].astype(np.int64), by_length[:light].astype(np.int64), team, light, light_edges


def check(ctx, col_ptr, long_edges, expect_long, expect_light):
    nnz, n = int(col_ptr[-1]), len(col_ptr) - 1
    items, by_length, team, light, light_edges = last_list(ctx, nnz + n)
    v, e0, e1, slot = items.T
    length = e1 - e0
    cover = np.zeros(nnz + 1, np.int64)
    np.add.at(cover, e0, 1)
    np.add.at(cover, e1, -1)
    assert (np.cumsum(cover)[:-1] == 1).all(), "an edge in no item or in two"
    assert (e0 >= col_ptr[v]).all() and (e1 <= col_ptr[v + 1]).all()
    if expect_long is not None:
        assert set(np.flatnonzero(length > long_edges)) == set(range(team)), (team, int((length > long_edges).sum()))
        assert (team > 0) == expect_long, team
    else:
        assert team == 0 and (length > long_edges).all()
    # the light columns end the list, in column order; their copy has the longest first within every 1,024
    is_light = (slot < 0) & (length <= 16)
    n_light = int(is_light.sum())
    assert is_light[len(items) - n_light:].all() and (np.diff(v[is_light]) > 0).all()
    assert light == (n_light if expect_light else 0)
    if light:
        assert light_edges == length[is_light].sum()
    for i in range(0, light, 1024):
        part = by_length[i:i + 1024]
        assert (np.diff((16 - (part[:, 2] - part[:, 1])) * n + part[:, 0]) > 0).all()
        assert np.array_equal(part[np.argsort(part[:, 0])], items[is_light][i:i + 1024])
    pieces = slot >= 0
    assert sorted(slot[pieces].tolist()) == list(range(int(pieces.sum())))


def main():
    lib = sys.argv[1]
    rng = np.random.default_rng(11)
    n = 6000
    deg = rng.integers(0, 30, n)
    deg[[7, 70, 700]] = [5200, 129, 128]
    pairs = {(v, int(u)) for v in range(n) for u in rng.choice(n, deg[v], replace=False)}
    pairs |= {(v, 9) for v in range(0, n, 2)}              # a hub in the edges by source
    g = si.csc_from_lists(n, sorted((u, v) for v, u in pairs))
    cp, ri = g.col_ptr.numpy(), g.row_idx.numpy()
    out_deg = np.bincount(ri, minlength=n)
    cp_out = np.concatenate([[0], np.cumsum(out_deg)])
    t = lambda *s: torch.as_tensor((rng.standard_normal(s) * 0.3).astype(np.float32))
    for opts in (dict(), dict(cut_degree=1 << 20), dict(stripe_kb=0, cut_degree=1 << 20), dict(split=16, cut_degree=40)):
        ctx = StubContext(lib)
        for k, x in opts.items():
            ctx.set_option(k, x)
        h = ctx.graph_create_csc(n, dev(g.col_ptr), dev(g.row_idx))
        for F in (16, 128, 16):
            X, W = t(n, F), t(F, 4)
            # bands of 1 MiB: 16,384 rows of 64 bytes, 65,536 of 16, 2,048 of 512 (or no bands)
            long_edges = 128 if "stripe_kb" not in opts and F == 16 else 1024
            Y, A = dev(torch.full((n, 4), float("nan"))), dev(torch.full((n, F), float("nan")))
            ctx.layer_forward(h, dev(X), Y, edge_op="copy", W=dev(W), accum_out=A)
            ctx.synchronize()
            # cut at band ends, rows of 128 features make pieces of 2,048 sources at most; uncut, the hub is one item
            hub_piece = int((ri[cp[7]:cp[7 + 1]] < 2048).sum())
            check(ctx, cp, long_edges, True if long_edges == 128 or "cut_degree" in opts and opts["cut_degree"] > 5200 else hub_piece > 1024, True)
            ref = oracle.layer(cp, ri, X.numpy(), "copy", None, agg="sum", W=W.numpy())
            assert_sum_close(Y.t.numpy(), ref["Y"], ref["Y_abs"], 1e-4, f"{opts} F {F}")
            dX, dW = dev(torch.full((n, F), float("nan"))), dev(torch.full((F, 4), float("nan")))
            ctx.layer_backward(h, A, dev(t(n, 4)), dev(W), dW, X=dev(X), edge_op="copy", dX=dX)
            ctx.synchronize()
            width = min(F, 4)                                    # what travels back is the gradient of the narrower side
            assert width == 4
            check(ctx, cp_out, 256 if "stripe_kb" not in opts else 1024, True, True)
        h.destroy()
        ctx.destroy()
    # every column past the limit: shared where a band holds 4,096 rows, not where it holds more of them
    n, d = 800, 600
    g = si.csc_from_lists(n, sorted((int(u), v) for v in range(n) for u in rng.choice(n, d, replace=False)))
    cp = g.col_ptr.numpy()
    ctx = StubContext(lib)
    h = ctx.graph_create_csc(n, dev(g.col_ptr), dev(g.row_idx))
    for F, long_edges, expect_long in ((16, 128, None), (64, 128, True)):
        ctx.layer_forward(h, dev(t(n, F)), dev(torch.empty(n, F)), edge_op="copy")
        ctx.synchronize()
        check(ctx, cp, long_edges, expect_long, False)
    h.destroy()
    ctx.destroy()
    print("ok: work lists of resident propagations", flush=True)


if __name__ == "__main__":
    main()
