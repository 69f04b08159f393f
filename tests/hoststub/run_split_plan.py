"""The split workspace of streamed backward calls on the CPU stand-in: parts of a matrix whose own plan has more splits than
the plan of all its rows, which sized the workspace.

  python tests/hoststub/run_split_plan.py <library>"""
import ctypes
import os
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
TESTS = os.path.dirname(HERE)
sys.path[:0] = [os.path.dirname(TESTS), TESTS, HERE]

import torch

from stub_binding import StubContext, dev


def plan(lib, n, FP, FQ, room=1024):
    rows, splits = ctypes.c_int64(), ctypes.c_int32()
    lib.stub_tn_plan(n, FP, FQ, room, ctypes.byref(rows), ctypes.byref(splits))
    assert rows.value % 16 == 0 and splits.value >= 1 and (splits.value - 1) * rows.value < max(n, 1) <= splits.value * rows.value
    return splits.value


def main():
    ctx = StubContext(sys.argv[1])
    ctx.lib.stub_tn_plan.argtypes = [ctypes.c_int64, ctypes.c_int32, ctypes.c_int32, ctypes.c_int64, ctypes.c_void_p, ctypes.c_void_p]
    ctx.lib.stub_tn_plan.restype = None
    more = 0
    for FP, FQ in ((256, 256), (128, 128), (8, 3000), (602, 41), (1, 1), (640, 640), (64, 64)):
        for n in (65537, 172034, 262145, 21505, 300, 16385):
            room = plan(ctx.lib, n, FP, FQ)
            for m in {n // 2, n - n // 2, n // 3, n - 2 * (n // 3), 32768, 10752, 4096, 256, 16, 1} - {0}:
                if m <= n:
                    more += plan(ctx.lib, m, FP, FQ) > room
                    assert plan(ctx.lib, m, FP, FQ, room) <= room, (n, m, FP, FQ)
    # where the workspace may not grow (streamed calls, contexts with a budget) the splits are those of eight wavefronts per compute
    # unit: fewer are longer sums, whose error is larger
    for n, FP, FQ, splits in ((131072, 320, 130, 85), (131072, 640, 300, 34), (262144, 384, 128, 169), (65536, 640, 640, 20)):
        assert plan(ctx.lib, n, FP, FQ) == splits, (n, FP, FQ, plan(ctx.lib, n, FP, FQ))
    assert more >= 3, "no part here has more splits than the whole: the cases test nothing"
    # 21,505 rows: 41 splits; the second of two source intervals, 10,752 rows: 42
    n, F, Fo = 21505, 8, 3000
    assert plan(ctx.lib, n, F, Fo) < plan(ctx.lib, n // 2, F, Fo)
    gen = torch.Generator().manual_seed(1)
    A, dY, W = torch.randn(n, F, generator=gen), torch.randn(n, Fo, generator=gen), torch.randn(F, Fo, generator=gen) * 0.05
    ctx.set_option("dst_intervals", 1)
    ctx.set_option("src_intervals", 2)
    ids = torch.arange(n, dtype=torch.int32)
    h = ctx.graph_create_csc(n, torch.arange(n + 1, dtype=torch.int64), ids)
    dW, dX = torch.full((F, Fo), float("nan")), torch.full((n, F), float("nan"))
    dWd = dev(dW)
    ctx.layer_backward(h, A, dY, dev(W), dWd, edge_op="copy", dX=dX)
    ctx.synchronize()
    for got, ref, scale in ((dWd.t, A.double().T @ dY.double(), A.double().abs().T @ dY.double().abs()),
                            (dX, dY.double() @ W.double().T, dY.double().abs() @ W.double().abs().T)):
        assert ((got.double() - ref).abs() / scale).max().item() <= 1e-5
    h.destroy()
    ctx.destroy()
    print(f"ok: {more} parts with more splits than the whole", flush=True)


if __name__ == "__main__":
    main()
