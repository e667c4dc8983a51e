"""Aggregation of feature rows that are no whole number of 16-byte units or not 16-byte aligned: the widths around a unit,
a team and a panel, tables whose rows start at odd addresses, light rows and rows that are cut into chunks."""
import numpy as np
import pytest
import torch

from gas_inputs import rng
from oracle import ops as oops
from tests.util import node_rel_err, to_np

pytestmark = pytest.mark.gpu

TOL = {torch.float32: 1e-5, torch.bfloat16: 2e-2}         # of the aggregation's other parity tests


def _pattern(n_rows, n_cols, long_row):
    """Rows of 0 to 70 entries and one of long_row, columns in order."""
    lens = np.array([(7 * i) % 71 for i in range(n_rows)])
    lens[n_rows // 2] = long_row
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    col = np.concatenate([np.sort((np.arange(k) * 7919 + 13 * i) % n_cols) for i, k in enumerate(lens)]).astype(np.int32)
    return ptr, col


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("F", [1, 3, 4, 5, 7, 8, 9, 33, 63, 65, 129, 250, 257, 511, 1023, 1027, 1433, 2051])
def test_aggregation_of_odd_rows(F, dtype):
    import paper_2106_05609_amd as gas
    nb, nh, n_table = 60, 40, 300
    ptr, col = _pattern(nb, nb + nh, 1500)
    n_id = to_np(rng.permutation(3, 800, n_table)[:nb + nh].to(torch.int32))
    val = to_np(rng.normal(3, 801, 0, col.size))
    # rows of X start at one element past a 16-byte boundary, the table's rows have an odd stride
    x = torch.empty(nb, F + 3, dtype=dtype, device="cuda")[:, 1:F + 1]
    x.copy_(rng.normal_matrix(3, 802, nb, F, dtype=dtype))
    hist = rng.normal_matrix(3, 803, n_table, F, dtype=dtype).cuda()
    d_ptr, d_col, d_val = (torch.from_numpy(a).cuda() for a in (ptr, col, val))
    src = torch.from_numpy(np.where(col < nb, col, -1 - n_id[col]).astype(np.int32)).cuda()
    plan = gas.gas_plan_create(d_ptr, col.size, F, ind=d_col)
    pad = torch.full((nb + 1, F + 2), 7.0, dtype=dtype, device="cuda")
    z = pad[:nb, 1:F + 1]
    gas.gas_spmm_hist(plan, d_ptr, src, d_val, x, hist, z, diag=0.5, r=x, s_res=0.25)
    torch.cuda.synchronize()
    xo = np.concatenate([to_np(x), oops.pull(to_np(hist), n_id[nb:])])
    want = oops.spmm(ptr, col, val, xo, diag=0.5, r=to_np(x), s_res=0.25)
    assert node_rel_err(to_np(z), want) <= TOL[dtype]
    assert bool((pad[:, 0] == 7.0).all()) and bool((pad[:, F + 1] == 7.0).all()) and bool((pad[nb] == 7.0).all())
    # the same pattern as a backward aggregation (one source, no residual)
    z2 = torch.full((nb, F), float("nan"), dtype=dtype, device="cuda")
    xfull = torch.from_numpy(xo.view(np.int16) if dtype == torch.bfloat16 else xo)
    xfull = (xfull.view(torch.bfloat16) if dtype == torch.bfloat16 else xfull).cuda()
    gas.gas_spmm_t(plan, d_ptr, d_col, d_val, xfull, z2)
    assert node_rel_err(to_np(z2), oops.spmm(ptr, col, val, xo)) <= TOL[dtype]


# rows, input and output width: several k steps with a remainder, one and several column tiles with a tail
PRODUCTS = [(1, 1, 1), (300, 81, 256), (129, 1433, 47), (257, 131, 129), (200, 70, 300), (5000, 250, 33)]


@pytest.mark.parametrize("views", [False, True])
@pytest.mark.parametrize("what", ["linear", "input", "weight"])
@pytest.mark.parametrize("m,k,n", PRODUCTS)
def test_bf16_products_of_odd_widths(what, m, k, n, views):
    """views: rows start one element past a 16-byte boundary and have an odd stride, the output lies between guard columns."""
    import paper_2106_05609_amd as gas

    def operand(stream, rows, cols):
        t = rng.normal_matrix(3, stream, rows, cols, dtype=torch.bfloat16).cuda()
        return torch.nn.functional.pad(t, (1, 2 + cols % 2))[:, 1:cols + 1] if views else t

    z, g, w = operand(820, m, k), operand(821, m, n), rng.normal_matrix(3, 822, k, n, dtype=torch.bfloat16).cuda()
    z64, g64, w64 = z.double(), g.double(), w.double()
    if what == "weight":
        out = torch.full((k, n), float("nan"), device="cuda")
        ws = torch.empty(max(1, gas.gas_linear_bwd_weight_workspace(m, k, n)), dtype=torch.uint8, device="cuda")
        gas.gas_linear_bwd_weight(z, g, out, ws)
        want, size, terms, stored = z64.t() @ g64, z64.t().abs() @ g64.abs(), m, 0.0
    else:
        cols = n if what == "linear" else k
        pad = torch.full((m, cols + 3), 7.0, dtype=torch.bfloat16, device="cuda")
        out = pad[:, 1:cols + 1] if views else torch.full((m, cols), float("nan"), dtype=torch.bfloat16, device="cuda")
        if what == "linear":
            gas.gas_linear(z, w, out)
            want, size, terms = z64 @ w64, z64.abs() @ w64.abs(), k
        else:
            gas.gas_linear_bwd_input(g, w, out)
            want, size, terms = g64 @ w64.t(), g64.abs() @ w64.t().abs(), n
        stored = 2.0 ** -8                 # the output's rounding to bf16: eight significant bits, half a unit of the last
        if views:
            assert bool((pad[:, 0] == 7.0).all()) and bool((pad[:, cols + 1:] == 7.0).all())
    # products of bf16 numbers are exact in fp32; every addition rounds a partial sum of at most `size`
    assert bool(((out.double() - want).abs() <= stored * want.abs() + (terms + 2) * 2.0 ** -24 * size * (1 + stored)).all())


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("F", [7, 33, 250, 256])
def test_push_of_odd_rows_to_host_memory(F, dtype):
    """From the transform's call and by itself: the rows named, and no byte of their neighbours."""
    import paper_2106_05609_amd as gas
    m, n_table = 300, 1001
    z, w = rng.normal_matrix(3, 830, m, 40, dtype=dtype).cuda(), rng.normal_matrix(3, 831, 40, F, dtype=dtype).cuda()
    w2 = rng.normal_matrix(3, 832, F, F, dtype=dtype).cuda()
    idx = rng.permutation(3, 833, n_table)[:m].to(torch.int32).cuda()
    y, h = (torch.empty(m, F, dtype=dtype, device="cuda") for _ in range(2))
    for call in (lambda t: gas.gas_linear_push(z, w, y, idx, t), lambda t: gas.gas_mlp2_push(z, w, w2, y, idx, t),
                 lambda t: gas.gas_mlp2_keep(z, w, w2, y, h, idx=idx, hist=t), lambda t: gas.gas_push(y, idx, t)):
        rows = torch.full((n_table, F), 7.0, dtype=dtype).pin_memory()
        call(gas.HostTable(rows))
        torch.cuda.synchronize()
        want = torch.full((n_table, F), 7.0, dtype=dtype)
        want[idx.cpu().long()] = y.cpu()
        assert torch.equal(rows, want)


# around a tile of 64 and 128 rows and columns, a step of 64 and a word of two
@pytest.mark.parametrize("m,k,h,n", [(1, 1, 1, 1), (63, 65, 63, 64), (64, 63, 65, 127), (65, 129, 255, 257), (129, 64, 256, 3), (16600, 9, 33, 129)])
def test_bf16_mlp_and_masks_of_odd_widths(m, k, h, n):
    """The fused MLP and the masked input gradient with an infinite row among finite ones, which no other row may see."""
    import paper_2106_05609_amd as gas
    z, w1, w2, g = (rng.normal_matrix(3, 840 + i, *s, dtype=torch.bfloat16).cuda() for i, s in
                    enumerate(((m, k), (k, h), (h, n), (m, h))))
    if m > 1:
        z[m // 2] = float("inf")
    b1, b2 = (rng.normal_matrix(3, 850 + i, 1, s, dtype=torch.bfloat16).cuda()[0] for i, s in enumerate((h, n)))
    y = torch.full((m, n + 1), 7.0, dtype=torch.bfloat16, device="cuda")
    gas.gas_mlp2(z, w1, w2, y[:, :n], b1=b1, b2=b2)
    rows = torch.arange(m, device="cuda") != m // 2 if m > 1 else torch.ones(1, dtype=torch.bool, device="cuda")
    z64 = z[rows].double()
    hid, hid_size = (z64 @ w1.double() + b1.double()).clamp_min(0), z64.abs() @ w1.double().abs() + b1.double().abs()
    # the hidden row is rounded to bf16 (2^-8 of it) after k + 1 fp32 sums; the output after h + 1 more
    hid_err = 2.0 ** -8 * hid + (k + 2) * 2.0 ** -24 * hid_size * (1 + 2.0 ** -8)
    want, size = hid @ w2.double() + b2.double(), hid @ w2.double().abs() + b2.double().abs()
    bound = 2.0 ** -8 * want.abs() + (hid_err @ w2.double().abs() + (h + 2) * 2.0 ** -24 * (size + hid_err @ w2.double().abs())) * (1 + 2.0 ** -8)
    assert bool(((y[rows, :n].double() - want).abs() <= bound).all()) and bool((y[:, n] == 7.0).all())
    gz = torch.full((m, k + 1), 7.0, dtype=torch.bfloat16, device="cuda")
    mask = rng.normal_matrix(3, 860, m, k, dtype=torch.bfloat16).cuda()
    gas.gas_linear_bwd_input(g, w1, gz[:, :k], mask=mask)
    want, size = g.double() @ w1.double().t(), g.double().abs() @ w1.double().t().abs()
    want, size = want * (mask > 0), size * (mask > 0)
    bound = 2.0 ** -8 * want.abs() + (h + 2) * 2.0 ** -24 * size * (1 + 2.0 ** -8)
    assert bool(((gz[:, :k].double() - want).abs() <= bound).all()) and bool((gz[:, k] == 7.0).all())


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("m,k,n", [(300, 81, 256), (129, 745, 47), (70, 64, 64), (1, 1, 1), (15, 31, 63), (17, 33, 64), (513, 32, 65),
                                   (16385, 33, 15), (8200, 65, 130), (33000, 31, 1)])
def test_products_in_order(m, k, n, dtype):
    """Odd bf16 widths: the bits of fp32 fused multiply-adds in the order of k (exact products, so one rounding a step: formed here in
    64 bits, rounded to fp32 each time); elsewhere gas_linear's."""
    import paper_2106_05609_amd as gas
    z, w = rng.normal_matrix(3, 870, m, k, dtype=dtype).cuda(), rng.normal_matrix(3, 871, k, n, dtype=dtype).cuda()
    y, want = (torch.full((m, n), float("nan"), dtype=dtype, device="cuda") for _ in range(2))
    gas.gas_linear_in_order(z, w, y)
    if dtype == torch.float32 or (k % 8 == 0 and n % 8 == 0):
        gas.gas_linear(z, w, want)
        assert torch.equal(y, want)
        return
    s = torch.zeros(m, n, device="cuda")
    for i in range(k):
        s = (s.double() + z[:, i:i + 1].double() * w[i:i + 1].double()).float()
    assert torch.equal(y, s.to(dtype))


@pytest.mark.parametrize("f_in,f,heads,stride", [(75, 64, 2, 75), (64, 36, 4, 64), (64, 64, 1, 67), (64, 64, 1, 64)])
def test_gat_passes_agree_in_bf16(f_in, f, heads, stride):
    """Inference and training of the same weights give the same rows and push the same rows, also where widths or rows take no
    16-byte pieces."""
    from gas_inputs import configs, batches
    from paper_2106_05609_amd import executor
    cfg = configs.config(1, 0.05)
    g = configs.build_graph(cfg)
    sg = batches.batch_subgraph(g, batches.split(g, cfg.blocks_per_batch, cfg.seed)[0], True)
    d = lambda t: t.cuda()
    bg = executor.BatchGraph(sg.nb, d(sg.n_id), d(sg.rowptr), d(sg.col), None, d(sg.colptr), d(sg.row), max_F=max(f_in, f),
                             normalise=False, csc_pos=d(sg.csc_perm).int())
    bf = torch.bfloat16
    x = rng.normal_matrix(3, 880, g.n, stride, dtype=bf).cuda()[:, :f_in]
    ws = [(rng.glorot_uniform(3, 881 + l, (f_in, f)[l], f, dtype=bf).cuda(), rng.normal(3, 884 + l, 0, f, dtype=bf).cuda() * 0.3,
           rng.normal(3, 887 + l, 0, f, dtype=bf).cuda() * 0.3) for l in range(2)]
    hist = rng.normal_matrix(3, 890, g.n, f, dtype=bf).cuda()
    tables = [hist.clone(), hist.clone()]
    y = executor.gat_forward_batch(ws, bg, x, [tables[0]], heads=heads)
    trained, _, _ = executor.gat_train_batch(ws, bg, x, [tables[1]], torch.zeros_like(y), heads=heads)
    assert torch.equal(y, trained) and torch.equal(tables[0], tables[1])
