"""Parameter gradients of backward-ApplyVertex (Section 2.2) whose vertex range is divided over as many splits as the chip holds in one
round, in two, and in neither (few rows a split, or a workspace that may not grow), against float64."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,f_in,f_out,budget", [
    (40001, 640, 640, 0),        # 100 wavefronts a split: two rounds
    (40001, 640, 640, 1 << 32),  # the same under a budget: the division it always had
    (20479, 640, 640, 0),        # one row too few a split for either
    (174080, 384, 128, 0),       # 12: one round of 168
    (90117, 320, 130, 1 << 32),  # 24 under a budget: the division it always had
    (90117, 320, 130, 0),        # two rounds
    (35000, 64, 1000, 0)])       # a wide Q
def test_dw_against_float64(n, f_in, f_out, budget):
    import paper_1810_08403_amd as saga
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n + f_in)
    ctx = saga.Context(0, hbm_budget_bytes=budget)
    ids = torch.arange(n + 1, device="cuda")
    g = ctx.graph_create_csc(n, ids, ids[:-1].to(torch.int32))
    A, dY = torch.randn(n, f_in, device="cuda", generator=gen), torch.randn(n, f_out, device="cuda", generator=gen)
    dW = torch.full((f_in, f_out), float("nan"), device="cuda")
    ctx.layer_backward(g, A, dY, torch.zeros(f_in, f_out, device="cuda"), dW, act="none", edge_op="copy", agg="sum")
    ref = A.double().T @ dY.double()
    # a sum of n products in fp32, rounded at every 16th: far below sqrt(n / 16) half units of the last place of its largest value
    assert float((dW.double() - ref).norm() / ref.norm()) < 2.0 ** -24 * (n / 16) ** 0.5
    g.destroy()
