"""Columns of few edges, several side by side in one wavefront: widths at the edges of its lane groups and batches, columns
just below and above the most edges they may have, empty ones, every edge function, against float64 sums; and beside them
columns of so many edges that four wavefronts share one."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _graph(n, heavy, seed, lanes):
    """Degrees 0 to 16, the edges among them, in turn, for rows of more than 8 fragments with four short columns to each, since
    the kernel takes such rows where columns are short (and, with `heavy`, some of 17 and 300, and four at or past the
    lengths from which four wavefronts share an item: 129 edges at up to 256 bytes a row, 257 at up to 32, 1,025 at
    more)."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    pattern = [0, 1, 7, 8, 15, 16, 3, 13] + ([1, 0, 2, 1, 1, 0, 1, 2] * 4 if lanes > 8 else [])
    deg = torch.tensor(pattern, device=DEV).repeat(-(-n // len(pattern)))[:n].clone()
    if heavy:
        deg[97::97] = 17
        deg[5::4001] = 300
        deg[3], deg[11], deg[19], deg[27] = 128, 129, 5000, 1900
    dst = torch.repeat_interleave(torch.arange(n, device=DEV), deg)
    src = torch.randint(1, n - 1, (dst.numel(),), generator=g, device=DEV)   # nothing reads the first and the last row
    if heavy:
        src[dst == 27] = torch.randint(1, 2046, (1900,), generator=g, device=DEV)   # some 1,240 of one band
    key = torch.unique(dst * n + src)
    dst = key // n
    col_ptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(torch.bincount(dst, minlength=n), 0, out=col_ptr[1:])
    return col_ptr, (key - dst * n).int(), dst, g


def _ctx(n, col_ptr, row_idx):
    import paper_1810_08403_amd as saga
    ctx = saga.Context(0)
    return ctx, ctx.graph_create_csc(n, col_ptr, row_idx)


@pytest.mark.parametrize("F,pad", [(1, 0), (2, 1), (3, 0), (4, 0), (5, 0), (8, 0), (12, 4), (13, 0), (16, 0), (28, 0), (31, 2), (32, 0), (41, 0), (64, 0), (100, 0),
                                   (127, 1), (128, 0)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("heavy", [False, True])
def test_linear_messages(F, pad, dtype, heavy):
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    Fx = F if dtype == "f32" else 2 * F - (F & 1)   # up to 32 fragments in either type, odd widths kept
    vec = 4 if dtype == "f32" else 8
    lanes = -(-Fx // vec) if Fx >= vec else Fx
    n = (64 // lanes) * 4 * (17000 if heavy else 4200) // 3   # past the count from which the kernel is used
    col_ptr, row_idx, dst, g = _graph(n, heavy, F, lanes)
    ctx, h = _ctx(n, col_ptr, row_idx)
    big = torch.randn(n, Fx + pad, generator=g, device=DEV).to(tdt)
    big[0], big[n - 1] = float("nan"), float("inf")
    X = big[:, :Fx]
    w = torch.randn(row_idx.numel(), generator=g, device=DEV)
    for agg in ("sum", "max"):
        for weight in (w, None):
            A = torch.full((n, Fx), float("nan"), device=DEV)
            Y = torch.empty(n, Fx, device=DEV, dtype=tdt)
            kw = dict(edge_op="mul_weight", edge_weight=weight) if weight is not None else dict(edge_op="copy")
            ctx.layer_forward(h, X, Y, agg=agg, accum_out=None if dtype == "f32" else A, **kw)
            if dtype == "f32":
                A = Y
            msg = X[row_idx.long()].float()
            if weight is not None:
                msg = weight[:, None] * msg
            if agg == "max":
                ref = torch.full((n, Fx), float("-inf"), device=DEV).index_reduce_(0, dst, msg, "amax")
                ref[ref == float("-inf")] = 0
                assert torch.equal(A, ref), (F, dtype, agg)
                continue
            prod = X[row_idx.long()].double() * (1 if weight is None else weight[:, None].double())
            ref = torch.zeros(n, Fx, dtype=torch.float64, device=DEV).index_add_(0, dst, prod)
            scale = torch.zeros(n, Fx, dtype=torch.float64, device=DEV).index_add_(0, dst, prod.abs())
            # at most as many fp32 additions of rounded (fused) products as the column has edges, 5,000
            assert ((A.double() - ref).abs() <= 5010 * 2.0 ** -24 * scale).all(), (F, dtype, agg)
            assert ((A.double() - ref).norm() <= 1e-6 * ref.norm()), (F, dtype, agg)
            A2 = torch.full_like(A, float("nan"))
            ctx.layer_forward(h, X, A2 if dtype == "f32" else Y, agg=agg, accum_out=None if dtype == "f32" else A2, **kw)
            assert torch.equal(A, A2), "sums are reproducible"
    ctx.destroy()


@pytest.mark.parametrize("agg", ["sum", "max"])
@pytest.mark.parametrize("F", [3, 8, 20, 64, 128])
@pytest.mark.parametrize("heavy", [False, True])
def test_gated_and_pooled_layers_both_ways(F, agg, heavy):
    """Forward and backward against float64 autograd (dense per edge), degrees and widths as above; a vertex without in-edges whose
    own row is not finite keeps an empty sum, and a vertex without edges keeps its rows to itself. With `heavy`, light columns,
    shared long items and the pieces of cut columns lie in one propagation."""
    lanes = -(-F // 4) if F >= 4 else F
    n = (64 // lanes) * 4 * (17000 if heavy else 4200) // 3
    col_ptr, row_idx, dst, g = _graph(n, heavy, F, lanes)
    ctx, h = _ctx(n, col_ptr, row_idx)
    src = row_idx.long()
    t = lambda *s: torch.randn(*s, generator=g, device=DEV) * 0.3
    X, W, dY = t(n, F), t(F, 5), t(n, 5)
    X[0] = float("inf")                                    # no edge starts or ends here
    dX, dW, A, Y = torch.empty_like(X), torch.empty_like(W), torch.empty(n, F, device=DEV), torch.empty(n, 5, device=DEV)
    Xd = X.double()
    Xd[0] = 0
    for op in ("gated", "pool"):
        if op == "gated":
            kw = dict(W_gate=t(F, 2 * F), b_gate=t(F), W_msg=t(F, F))
            grads = dict(dW_gate=torch.empty(F, 2 * F, device=DEV), db_gate=torch.empty(F, device=DEV), dW_msg=torch.empty(F, F, device=DEV))
        else:
            kw = dict(W_pool=t(F, F), b_pool=t(F))
            grads = dict(dW_pool=torch.empty(F, F, device=DEV), db_pool=torch.empty(F, device=DEV))
        X[0] = float("inf")
        ctx.layer_forward(h, X, Y, edge_op=op, agg=agg, W=W, accum_out=A, **kw)
        X[0] = 0                                           # (the parameter gradients read every row of X)
        ctx.layer_backward(h, A, dY, W, dW, X=X, Y=Y, edge_op=op, agg=agg, dX=dX, **kw, **grads)
        leaf = {k: v.double().requires_grad_() for k, v in kw.items()}
        x = Xd.clone().requires_grad_()
        if op == "gated":
            wg = leaf["W_gate"]
            z = (x @ wg[:, :F].T)[src] + (x @ wg[:, F:].T + leaf["b_gate"])[dst]
            msg = torch.sigmoid(z) * (x @ leaf["W_msg"].T)[src]
        else:
            msg = torch.sigmoid(x @ leaf["W_pool"].T + leaf["b_pool"])[src]
        if agg == "sum":
            acc = torch.zeros(n, F, dtype=torch.float64, device=DEV).index_add(0, dst, msg)
        else:
            with torch.no_grad():
                top = torch.full((n, F), float("-inf"), dtype=torch.float64, device=DEV).index_reduce_(0, dst, msg, "amax")
                pick = (msg == top[dst]).double()          # no ties in continuous data
            acc = torch.zeros(n, F, dtype=torch.float64, device=DEV).index_add(0, dst, msg * pick)
        (acc @ W.double() * dY.double()).sum().backward()
        rel = lambda got, want: ((got.double() - want).norm() / want.norm()).item()
        assert rel(A, acc.detach()) <= 1e-5 and bool((A[col_ptr[1:] == col_ptr[:-1]] == 0).all()), (op, agg, F)
        assert rel(dW, (acc.detach().T @ dY.double())) <= 1e-5
        # a maximum may go to another edge where two messages are equal in fp32: its whole gradient moves
        bound = 1e-5 if agg == "sum" else 2e-2
        assert rel(dX, x.grad) <= bound, (op, agg, F)
        for k, v in grads.items():
            assert rel(v, leaf[k[1:]].grad) <= bound, (op, agg, F, k)
    ctx.destroy()


@pytest.mark.parametrize("F,dtype", [(36, "f32"), (41, "f32"), (52, "f32"), (61, "f32"), (64, "f32"), (68, "f32"), (69, "f32"), (100, "f32"), (127, "f32"),
                                     (128, "f32"), (72, "bf16"), (100, "bf16"), (128, "bf16"), (136, "bf16"), (150, "bf16"), (256, "bf16")])
def test_rows_of_9_to_32_fragments_keep_the_order_of_the_other_kernel(F, dtype):
    """Two such rows (from 17 fragments on) or four lie side by side in a wavefront of the kernel for columns of any length: each
    lane group adds up every second or fourth edge. Several short columns side by side give the same bits, whichever kernel
    takes them."""
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    lanes = -(-F // (4 if dtype == "f32" else 8))
    C = 4 if lanes <= 16 else 2
    n = (64 // lanes) * 4 * 4200
    g = torch.Generator(device=DEV)
    g.manual_seed(F)
    # lengths up to the longest such column, and short ones between them: 3.6 edges a column
    deg = torch.tensor([0, 1, 7, 1, 2, 16, 1, 0, 15, 2, 1, 3, 1, 8, 0, 1, 2, 13, 0, 1, 5, 2, 1, 4], device=DEV).repeat(n // 24)
    n = deg.numel()
    dst = torch.repeat_interleave(torch.arange(n, device=DEV), deg)
    key = torch.unique(dst * n + torch.randint(0, n, (dst.numel(),), generator=g, device=DEV))
    dst = key // n
    deg = torch.bincount(dst, minlength=n)
    col_ptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(deg, 0, out=col_ptr[1:])
    row_idx = (key - dst * n).int()
    ctx, h = _ctx(n, col_ptr, row_idx)
    X = torch.randn(n, F, generator=g, device=DEV).to(tdt)
    # powers of two: a fused multiply-add rounds like the addition of the product
    w = 2.0 ** torch.randint(-2, 3, (row_idx.numel(),), generator=g, device=DEV)
    for weight in (None, w):
        A = torch.full((n, F), float("nan"), device=DEV)
        kw = dict(edge_op="mul_weight", edge_weight=weight) if weight is not None else dict(edge_op="copy")
        if dtype == "f32":
            ctx.layer_forward(h, X, A, **kw)
        else:
            ctx.layer_forward(h, X, torch.empty_like(X), accum_out=A, **kw)
        chains = [torch.zeros(n, F, device=DEV) for _ in range(C)]
        for k in range(16):
            v = torch.nonzero(deg > k).flatten()
            e = col_ptr[v] + k
            msg = X[row_idx[e].long()].float()
            chains[k % C][v] += msg if weight is None else weight[e][:, None] * msg
        want = chains[0] + chains[1]
        if C == 4:
            want += chains[2] + chains[3]
        assert torch.equal(A, want), (F, dtype, weight is not None)
    ctx.destroy()
