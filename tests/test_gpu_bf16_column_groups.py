"""ApplyVertex products of bf16 rows (Figure 10) whose wavefronts take three, four and five column tiles: the bits of the same product
taken 32 columns at a time, and float64 within what bf16 results allow."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,K,N,with_self", [(65536, 300, 130, False),    # five tiles, the last of two columns
                                             (65505, 65, 96, False),      # three, a last row tile of one row
                                             (65600, 128, 127, True),     # four, two operand pairs
                                             (70001, 301, 300, False),    # two groups of five, odd widths
                                             (65536, 384, 129, False),    # the largest K whose five tiles fit
                                             (65536, 385, 129, False),    # past it: two tiles
                                             (65504, 300, 130, False)])   # one row tile too few
def test_columns_together_and_apart(n, K, N, with_self):
    import paper_1810_08403_amd as saga
    gen = torch.Generator(device="cuda")
    gen.manual_seed(K * N)
    bf = torch.bfloat16
    rand = lambda *shape: torch.randn(*shape, device="cuda", generator=gen).to(bf)
    ctx = saga.Context(0)
    ids = torch.arange(n + 1, device="cuda")
    g = ctx.graph_create_csc(n, ids, ids[:-1].to(torch.int32))   # every vertex gathers itself: the product's rows are X
    X, W, bias = rand(n, K), rand(K, N), torch.randn(N, device="cuda", generator=gen)
    Ws = rand(K, N) if with_self else None

    def layer(c0, c1):
        Y = torch.full((n, c1 - c0), float("nan"), device="cuda", dtype=bf)
        kw = dict(W_self=Ws[:, c0:c1].contiguous()) if with_self else {}
        ctx.layer_forward(g, X, Y, W=W[:, c0:c1].contiguous(), bias=bias[c0:c1].contiguous(), act="relu", edge_op="copy", agg="sum", **kw)
        return Y

    Y = layer(0, N)
    assert torch.equal(Y, torch.cat([layer(c, min(c + 32, N)) for c in range(0, N, 32)], 1))
    ref = (X.double() @ (W.double() + (Ws.double() if with_self else 0)) + bias.double()).clamp(min=0)
    # half a unit of bf16 per result, and fp32 sums of K products
    assert bool(((Y.double() - ref).abs() <= ref * 2.0 ** -8 + 2.0 ** -16 * K).all())
    g.destroy()
