"""PNA's transform by the rows' degrees (gas_pna_linear and its backward calls) against 64 bits, and the executor's passes by
degree against its passes without."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _rows(n, most, gen):
    d = torch.randint(0, most + 1, (n,), generator=gen)
    d[: min(n, 3)] = torch.tensor([most, 0, most])[: min(n, 3)]
    return d, torch.cat([torch.zeros(1, dtype=torch.long), d.cumsum(0)]).int().cuda()


# one row; a tile and a slab and their neighbours; degrees that no row has; widths of one tile and of several, that nothing divides
@pytest.mark.parametrize("n,most", [(1, 0), (1, 5), (127, 0), (129, 0), (513, 1), (1025, 63), (5000, 12)])
@pytest.mark.parametrize("f,f1,n_out", [(8, 8, 8), (64, 16, 64), (33, 11, 47), (256, 64, 256)])
def test_products_by_degree(n, most, f, f1, n_out):
    import paper_2106_05609_amd as gas
    from paper_2106_05609_amd import binding as B
    gen = torch.Generator().manual_seed(n + f)
    d, ptr = _rows(n, most, gen)
    delta = 1.7
    x = torch.randn(n, f + 9 * f1, generator=gen)
    x[d == 0, f:] = 0.0                                        # a row without entries has zero aggregates
    w, g = torch.randn(f + 9 * f1, n_out, generator=gen), torch.randn(n, n_out, generator=gen)
    s = torch.log(d.double() + 1.0)[:, None] / delta
    inv = torch.where(d[:, None] > 0, 1.0 / s, torch.zeros_like(s))
    a = x[:, f:f + 3 * f1].double()
    full = torch.cat([x[:, :f].double(), a, s * a, inv * a], 1)
    mag = full.abs() @ w.double().abs()
    groups = B.gas_pna_groups(ptr, most)
    X, W, G = x.cuda(), w.cuda(), g.cuda()
    hist, ids = torch.zeros(2 * n, n_out, device="cuda"), torch.randperm(2 * n, generator=gen)[:n].int().cuda()
    for relu in (False, True):
        y = torch.full((n, n_out), 5.0, device="cuda")
        B.gas_pna_linear(groups, most, X, W, f1, delta, y, relu=relu, idx=ids if relu else None, hist=hist if relu else None)
        want = full @ w.double()
        # a rounding per term of the sum, of the scaled blocks and of the scaler itself
        err = (y.cpu().double() - (want.clamp(min=0) if relu else want)).abs()
        assert (err <= 32 * 2.0 ** -24 * mag).all()
    assert torch.equal(hist[ids.long()], y) and hist.count_nonzero() == y.count_nonzero()
    gx = torch.full((n, f + 3 * f1), 5.0, device="cuda")
    B.gas_pna_linear_bwd_input(groups, most, G, W, f1, delta, gx)
    nine = g.double() @ w.double().t()
    cut = [nine[:, f + 3 * f1 * k:f + 3 * f1 * (k + 1)] for k in range(3)]
    nine_abs = g.double().abs() @ w.double().abs().t()
    cut_abs = [nine_abs[:, f + 3 * f1 * k:f + 3 * f1 * (k + 1)] for k in range(3)]
    want = torch.cat([nine[:, :f], cut[0] + s * cut[1] + inv * cut[2]], 1)
    bound = torch.cat([nine_abs[:, :f], cut_abs[0] + s * cut_abs[1] + inv * cut_abs[2]], 1)
    assert ((gx.cpu().double() - want).abs() <= 32 * 2.0 ** -24 * bound).all()
    dw = torch.full((f + 9 * f1, n_out), 5.0, device="cuda")
    B.gas_pna_linear_bwd_weight(groups, most, X, G, f1, delta, dw)
    bound = full.abs().t() @ g.double().abs()
    assert ((dw.cpu().double() - full.t() @ g.double()).abs() <= (32 + n ** 0.5) * 2.0 ** -24 * bound).all()


def test_infinite_and_tiny_values_by_degree():
    """A non-finite value takes its block by the fp32 instruction, a tiny one its tile scaled: what fp32 arithmetic gives."""
    from paper_2106_05609_amd import binding as B
    gen = torch.Generator().manual_seed(5)
    n, f, f1, n_out = 700, 64, 16, 64
    d, ptr = _rows(n, 4, gen)
    d = d.clamp(min=0)
    x, w = torch.randn(n, f + 9 * f1, generator=gen), torch.randn(f + 9 * f1, n_out, generator=gen)
    x[d == 0, f:] = 0.0
    x[11] *= 2.0 ** -120
    x[500, 3] = float("inf")
    groups, y = B.gas_pna_groups(ptr, 4), torch.empty(n, n_out, device="cuda")
    B.gas_pna_linear(groups, 4, x.cuda(), w.cuda(), f1, 1.3, y)
    s = torch.log(d.double() + 1.0)[:, None] / 1.3
    a = x[:, f:f + 3 * f1].double()
    full = torch.cat([x[:, :f].double(), a, s * a, torch.where(d[:, None] > 0, a / s, torch.zeros_like(a))], 1)
    want, got = full @ w.double(), y.cpu().double()
    fine = torch.isfinite(want).all(1)
    assert not fine[500] and fine.sum() == n - 1 and torch.equal(got[500].sign(), want[500].sign()) and got[500].isinf().all()
    err = ((got - want)[fine]).abs()
    assert (err <= 32 * 2.0 ** -24 * (full.abs() @ w.double().abs())[fine]).all()


@pytest.mark.parametrize("f,hidden", [(40, 64), (64, 96)])
def test_passes_by_degree_agree_with_passes_without(f, hidden, monkeypatch):
    from gas_inputs import batches, graphs
    from paper_2106_05609_amd import binding as B, executor
    dev = torch.device("cuda")
    g = graphs.sbm_partners(40_000, 6, 6.0, 0.85, 3, dev)
    sg = batches.batch_subgraph(g, batches.split(g, 2, 0)[0], self_loops=False)
    gen = torch.Generator(device=dev).manual_seed(1)
    normal = lambda *shape: torch.randn(*shape, generator=gen, device=dev)
    widths = [f, hidden, hidden]
    ws = [(normal(2 * i, max(8, o // 4)) / i ** 0.5, normal(i + 9 * max(8, o // 4), o) / (3 * i) ** 0.5) for i, o in zip(widths, widths[1:])]
    x, table, grad = normal(40_000, f), normal(40_000, hidden).clamp_(min=0), normal(sg.nb, hidden)
    out = []
    monkeypatch.setattr(executor, "PNA_GROUPED_TERMS", 0)
    for least in (10_000, 1 << 40):
        monkeypatch.setattr(executor, "PNA_GROUPED_ROWS", least)
        bg = executor.BatchGraph(sg.nb, sg.n_id, sg.rowptr, sg.col, g.deg, sg.colptr, sg.row, max_F=256, normalise=False, csc_pos=sg.csc_perm)
        assert bg.max_row <= B.PNA_MAX_DEGREE
        h = [table.clone()]
        y = executor.pna_forward_batch(ws, 2.0, bg, x, h)
        assert (bg._groups is not None) == (least < 1 << 40)
        h2 = [table.clone()]
        y2, grads, kept = executor.pna_train_batch(ws, 2.0, bg, x, h2, grad)
        out.append([y, y2, h[0], h2[0]] + [t for pair in (grads[l] for l in range(2)) for t in pair] + [kept[0][2], kept[1][2]])
    for a, b in zip(*out):
        # gradients: a hidden unit within rounding of zero, or a tie for an extreme, may fall on either side
        assert (a - b).norm() <= (1e-5 if a is out[0][0] or a is out[0][1] else 4e-3) * b.norm()


@pytest.mark.parametrize("n,most", [(1, 0), (1, 63), (1023, 0), (1024, 5), (1025, 63), (5000, 12), (200_000, 26)])
def test_rows_by_degree(n, most):
    """Counts, tiles of 128 rows, slabs and the row ids, ascending for every degree, where one row, a workgroup's share of rows and
    many shares are listed; slabs of 512 rows, and of more from 65,537 rows on."""
    from paper_2106_05609_amd import binding as B
    d, ptr = _rows(n, most, torch.Generator().manual_seed(n + most))
    got = B.gas_pna_groups(ptr, most).cpu().view(torch.int32)
    count = torch.bincount(d, minlength=most + 1)
    assert torch.equal(got[2:3 + most].long(), count)
    n_tiles, n_slabs, slabs_at = int(got[0]), int(got[1]), 68 + 4 * (n // 128 + most + 1)
    slab = 512 * max(1, -(-n // 65_536))
    n_slabs_most = n // slab + most + 1
    rows_at = slabs_at + 4 * n_slabs_most
    assert torch.equal(got[rows_at:rows_at + n].long(), torch.argsort(d, stable=True)) and n_slabs <= n_slabs_most
    for parts, step in ((got[68:68 + 4 * n_tiles].view(-1, 4), 128), (got[slabs_at:slabs_at + 4 * n_slabs].view(-1, 4), slab)):
        want, at = [], 0
        for k, c in enumerate(count.tolist()):
            want += [(k, at + i, min(step, c - i)) for i in range(0, c, step)]
            at += c
        assert [tuple(p[:3]) for p in parts.tolist()] == want


def _pna_batch(f, hidden, layers, monkeypatch):
    from gas_inputs import batches, graphs
    from paper_2106_05609_amd import executor
    dev = torch.device("cuda")
    monkeypatch.setattr(executor, "PNA_GROUPED_TERMS", 0)
    monkeypatch.setattr(executor, "PNA_GROUPED_ROWS", 10_000)
    g = graphs.sbm_partners(40_000, 6, 6.0, 0.85, 3, dev)
    sg = batches.batch_subgraph(g, batches.split(g, 2, 0)[0], self_loops=False)
    gen = torch.Generator(device=dev).manual_seed(1)
    normal = lambda *shape: torch.randn(*shape, generator=gen, device=dev)
    widths = [f] + [hidden] * layers
    ws = [(normal(2 * i, max(8, o // 4)) / i ** 0.5, normal(i + 9 * max(8, o // 4), o) / (3 * i) ** 0.5) for i, o in zip(widths, widths[1:])]
    batch = lambda: executor.BatchGraph(sg.nb, sg.n_id, sg.rowptr, sg.col, g.deg, sg.colptr, sg.row, max_F=256, normalise=False, csc_pos=sg.csc_perm)
    tables = [normal(40_000, hidden).clamp_(min=0) for _ in range(layers - 1)]
    return batch, ws, normal(40_000, f), tables, normal(sg.nb, hidden)


@pytest.mark.parametrize("train", [False, True])
def test_a_captured_first_pass_goes_by_degree_too(train, monkeypatch):
    """A pass over a new batch that is captured before any eager one has the eager pass's bits, in every replay, and leaves the
    batch to later eager passes as it was."""
    from paper_2106_05609_amd import executor
    batch, ws, x, tables, grad = _pna_batch(40, 64, 2, monkeypatch)

    def run(bg):
        if not train:
            return [executor.pna_forward_batch(ws, 2.0, bg, x, tables)]
        y, grads, _ = executor.pna_train_batch(ws, 2.0, bg, x, tables, grad)
        return [y] + [t for l in range(2) for t in grads[l]]
    eager, captured = batch(), batch()
    want = [t.clone() for t in run(eager) + tables]
    for bg in (eager, captured):
        bg.plan_t_all
    assert eager._groups is not None and captured._groups is None
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        got = run(captured) + tables
    assert captured._groups is None
    for _ in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, want))
        assert all(torch.equal(a, b) for a, b in zip(run(captured), want))
        torch.cuda.synchronize()


def test_groups_are_built_without_a_wait_of_the_host(monkeypatch):
    """The host runs ahead of a busy stream, and another stream that asks in the meantime finds the lists complete."""
    batch, ws, x, tables, _ = _pna_batch(40, 64, 1, monkeypatch)
    from paper_2106_05609_amd import executor
    want = executor.pna_forward_batch(ws, 2.0, batch(), x, tables)
    bg, other, busy = batch(), torch.cuda.Stream(), torch.cuda.Event()
    torch.cuda.synchronize()
    torch.cuda._sleep(100_000_000)
    busy.record()
    bg.groups
    assert not busy.query()
    with torch.cuda.stream(other):
        got = executor.pna_forward_batch(ws, 2.0, bg, x, tables)
    torch.cuda.synchronize()
    assert torch.equal(got, want)
    assert bg.groups is bg.groups


def test_weight_gradient_by_long_slabs():
    """300,000 rows: slabs of 2,560, of which the longest degree has many and the rare ones less than one."""
    from paper_2106_05609_amd import binding as B
    gen = torch.Generator().manual_seed(9)
    n, most, f, f1, n_out, delta = 300_000, 20, 24, 8, 40, 1.7
    d = torch.where(torch.rand(n, generator=gen) < 0.7, torch.tensor(7), torch.randint(0, 4, (n,), generator=gen))
    d[100:400] = torch.arange(300) % (most + 1)
    ptr = torch.cat([torch.zeros(1, dtype=torch.long), d.cumsum(0)]).int().cuda()
    x, g = torch.randn(n, f + 9 * f1, generator=gen), torch.randn(n, n_out, generator=gen)
    x[d == 0, f:] = 0.0
    s = torch.log(d.double() + 1.0)[:, None] / delta
    a = x[:, f:f + 3 * f1].double()
    full = torch.cat([x[:, :f].double(), a, s * a, torch.where(d[:, None] > 0, a / s, torch.zeros_like(a))], 1)
    dw = torch.empty(f + 9 * f1, n_out, device="cuda")
    B.gas_pna_linear_bwd_weight(B.gas_pna_groups(ptr, most), most, x.cuda(), g.cuda(), f1, delta, dw)
    bound = full.abs().t() @ g.double().abs()
    assert ((dw.cpu().double() - full.t() @ g.double()).abs() <= (32 + n ** 0.5) * 2.0 ** -24 * bound).all()


@pytest.mark.parametrize("by_degree", [True, False])
def test_gradients_in_64_bits_from_the_pass_own_decisions(by_degree, monkeypatch):
    """A hidden unit within rounding of zero, or a neighbour within rounding of an extreme, may fall on either side, and takes its
    whole share of a gradient with it.  With the pass's own decisions (its activations' signs, the first extreme of its
    messages) differentiation in 64 bits gives its gradients to rounding: six products and sums in a chain, each within
    3e-7 of 64 bits in norm."""
    from paper_2106_05609_amd import executor
    batch, ws, x, tables, grad = _pna_batch(40, 64, 2, monkeypatch)
    if not by_degree:
        monkeypatch.setattr(executor, "PNA_GROUPED_ROWS", 1 << 40)
    bg, delta = batch(), 2.0
    stored = [t.double() for t in tables]
    y, grads, kept = executor.pna_train_batch(ws, delta, bg, x, tables, grad)
    assert (bg._groups is not None) == by_degree
    nb, d, col, ids = bg.nb, (bg.rowptr[1:] - bg.rowptr[:-1]).long(), bg.col.long(), bg.n_id.long()
    row, nnz = torch.repeat_interleave(torch.arange(nb, device="cuda"), d), col.numel()
    s = torch.log(d.double() + 1.0)[:, None] / delta
    some = (d > 0)[:, None]
    params, h = [[w.double().requires_grad_() for w in pair] for pair in ws], x[ids].double()
    for l, (w1, w2) in enumerate(params):
        f, f1 = h.shape[1], w1.shape[1]
        messages, index = (h @ w1[f:])[col], row[:, None].expand(-1, f1)
        mine = kept[l][1][col]                                          # the pass's own messages

        def first(how):
            best = torch.zeros(nb, f1, device="cuda").scatter_reduce_(0, index, mine, how, include_self=False)
            at = torch.where(mine == best[row], torch.arange(nnz, device="cuda")[:, None].expand(-1, f1), nnz)
            return messages.gather(0, torch.full((nb, f1), nnz, device="cuda").scatter_reduce_(0, index, at, "amin").clamp(max=nnz - 1))
        mean = torch.zeros(nb, f1, dtype=torch.float64, device="cuda").index_add(0, row, messages) / d.clamp(min=1)[:, None]
        blocks = [torch.where(some, t + h[:nb] @ w1[:f], 0.0) for t in (mean, first("amin"), first("amax"))]
        scaled = [s * t for t in blocks] + [t / torch.where(some, s, 1.0) for t in blocks]
        out = torch.cat([h[:nb]] + blocks + scaled, 1) @ w2
        if l == 0:
            out = out * (kept[l][3] > 0)
            h = torch.cat([out, stored[0][ids[nb:]]])
    want = torch.autograd.grad(out, [w for pair in params for w in pair], grad.double())
    assert (y - out).norm() <= 1.8e-6 * out.norm()
    for got, exact in zip([t for l in range(2) for t in grads[l]], want):
        assert (got - exact).norm() <= 1.8e-6 * exact.norm()
