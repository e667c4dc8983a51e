"""The anisotropic aggregations with what a batch knows of its pattern: the bound on row lengths drops launches and nothing else,
and the copies that ride along (the Push of GAT's rows, the receiving nodes' rows of PNA) are exact, whatever the widths, strides and
alignment of their targets."""
import numpy as np
import pytest
import torch

from gas_inputs import rng
from tests.util import to_np

pytestmark = pytest.mark.gpu


def _pattern(longest, hub=0):
    """Rows of 0 to 40 entries and one of `longest`, in a pattern of 300 columns, with its CSC copy.  Columns have their own limits
    (64, 512 and 2,048 entries): `hub` of the entries lie in one."""
    lens = np.array([(11 * i) % 41 for i in range(70)])
    lens[35] = longest
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    col = ((np.arange(ptr[-1]) * 7919) % 299).astype(np.int32)
    col[:hub] = 299
    rows = np.repeat(np.arange(70), lens).astype(np.int32)
    pos = np.lexsort((rows, col)).astype(np.int32)
    counts = np.bincount(col, minlength=300)
    colptr = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    return [torch.from_numpy(a).cuda() for a in (ptr, col, colptr, rows[pos], pos)], int(counts.max())


def _table(rows, width, dtype, odd):
    t = torch.full((rows, width + 3 if odd else width), 7.0, dtype=dtype, device="cuda")
    return t, t[:, 1:width + 1] if odd else t


@pytest.mark.parametrize("odd", [False, True])
@pytest.mark.parametrize("longest,hub", [(40, 0), (40, 64), (40, 65), (2048, 2048), (2049, 2049)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("F,heads", [(64, 4), (256, 1), (33, 2), (24, 3)])
def test_gat_rows_are_pushed_and_bounds_change_no_bits(F, heads, dtype, longest, hub, odd):
    import paper_2106_05609_amd as gas
    (ptr, col, colptr, row, pos), longest_col = _pattern(longest, hub)
    assert longest_col >= hub
    nb, nv, width = 70, 300, F * heads
    p, gz = (rng.normal_matrix(31, s, n, width, dtype=dtype).cuda() for s, n in ((1, nv), (2, nb)))
    a_dst, a_src = (rng.normal(31, s, 0, width, dtype=dtype).cuda() * 0.2 for s in (3, 4))
    z, z2 = (torch.full((nb, width), float("nan"), dtype=dtype, device="cuda") for _ in range(2))
    gas.gas_gat_aggregate(ptr, col, p, a_dst, a_src, z, relu=True, heads=heads)
    whole, hist = _table(500, width, dtype, odd)
    idx = rng.permutation(31, 5, 500)[:nb].to(torch.int32).cuda()
    want = whole.clone()
    (want[:, 1:width + 1] if odd else want)[idx.long()] = z
    gas.gas_gat_aggregate(ptr, col, p, a_dst, a_src, z2, relu=True, heads=heads, longest=longest, idx=idx, hist=hist)
    assert torch.equal(z, z2) and torch.equal(whole, want)
    for plan_t in (None, gas.gas_plan_create(colptr, col.numel(), F, n_rows=nv, ind=row)):
        _same_backward(gas, (ptr, col, colptr, row, pos, p, a_dst, a_src, gz), heads, plan_t, longest, longest_col)


def _same_backward(gas, args, heads, plan_t, longest, longest_col):
    (nv, width), dtype = args[5].shape, args[5].dtype
    got = []
    for bounds in ({}, dict(longest=longest, longest_col=longest_col)):
        out = [torch.full((nv, width), float("nan"), dtype=dtype, device="cuda")] + [torch.full((width,), float("nan"), device="cuda") for _ in range(2)]
        gas.gas_gat_aggregate_bwd(*args, *out, heads=heads, plan_t=plan_t, **bounds)
        got.append(out)
    assert all(torch.equal(a, b) for a, b in zip(*got)) and not any(bool(torch.isnan(t).any()) for t in got[0])


@pytest.mark.parametrize("odd", [False, True])
@pytest.mark.parametrize("longest,hub", [(40, 0), (40, 512), (40, 513), (2048, 0), (2049, 2049)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("F,F_own,blocks", [(64, 128, 9), (256, 8, 3), (33, 40, 9), (1032, 64, 3), (64, 13, 3), (64, 1000, 9)])
def test_pna_own_rows_are_copied_and_bounds_change_no_bits(F, F_own, blocks, dtype, longest, hub, odd):
    import paper_2106_05609_amd as gas
    (ptr, col, colptr, row, pos), _ = _pattern(longest, hub)
    nb, nv = 70, 300
    x, h = (rng.normal_matrix(32, s, n, w, dtype=dtype).cuda() for s, n, w in ((1, nv, F), (2, nv, F_own)))
    want = _table(nb, F_own + blocks * F, dtype, odd)[1][:, F_own:]      # as the target lies: it decides which kernel runs
    gas.gas_pna_aggregate(ptr, col, x, want, 1.5, blocks=blocks)
    whole, cat = _table(nb + 1, F_own + blocks * F, dtype, odd)
    cat = cat[:nb]
    gas.gas_pna_aggregate(ptr, col, x, cat[:, F_own:], 1.5, blocks=blocks, longest=longest, own=h, own_to=cat[:, :F_own])
    assert torch.equal(cat[:, :F_own], h[:nb]) and torch.equal(cat[:, F_own:], want)
    assert bool((whole[nb] == 7.0).all()) and (not odd or bool((whole[:, 0] == 7.0).all()))
    g = rng.normal_matrix(32, 3, nb, blocks * F, dtype=dtype).cuda()
    got = []
    # a plan whose line lies above the winners' own, one that says there are no long columns, and no bound at all
    for threshold, bound in ((1, {}), (2048, dict(longest=longest)), (512, dict(longest=longest))):
        plan_t = gas.gas_plan_create(colptr, col.numel(), F, n_rows=nv, ind=row, options=dict(heavy_threshold=threshold))
        gx, gadd = (torch.full((n, F), float("nan"), dtype=dtype, device="cuda") for n in (nv, nb))
        gas.gas_pna_aggregate_bwd(ptr, col, colptr, row, pos, x, g, gx, 1.5, gadd=gadd, plan_t=plan_t, blocks=blocks, **bound)
        got.append((gx, gadd))
    # the mean's share is summed in the plan's order: equal to rounding between plans, a missed column is not
    tol = 2e-5 if dtype == torch.float32 else 2e-2
    for gx, gadd in got[1:]:
        assert torch.equal(gadd, got[0][1])
        assert bool(((gx.double() - got[0][0].double()).abs().amax(1) <= tol * got[0][0].double().abs().amax(1)).all())


def test_targets_that_do_not_fit_are_refused():
    import paper_2106_05609_amd as gas
    (ptr, col, *_), _ = _pattern(40)
    x, z, idx = torch.zeros(300, 16, device="cuda"), torch.zeros(70, 16, device="cuda"), torch.arange(70, dtype=torch.int32, device="cuda")
    for idx_, hist in ((idx, None), (None, x), (idx[:5], x), (idx, x[:, :8].contiguous()), (idx, x.bfloat16())):
        with pytest.raises(ValueError):
            gas.gas_gat_aggregate(ptr, col, x, x[0], x[0], z, idx=idx_, hist=hist)
    out = torch.zeros(70, 144, device="cuda")
    for own, to in ((x, None), (None, z), (x, z[:, :8]), (x[:5], z), (x.bfloat16(), z)):
        with pytest.raises(ValueError):
            gas.gas_pna_aggregate(ptr, col, x, out, 1.0, own=own, own_to=to)
    # rows that are stored while others still read them, or over what the same call writes
    for table in (x, z):
        with pytest.raises(gas.GasError):
            gas.gas_gat_aggregate(ptr, col, x, x[0], x[0], z, idx=idx, hist=table)
    add, own = torch.zeros(70, 16, device="cuda"), torch.ones(70, 16, device="cuda")
    for to in (x, add, own, out[:, :16]):
        with pytest.raises(gas.GasError):
            gas.gas_pna_aggregate(ptr, col, x, out, 1.0, add=add, own=own, own_to=to)
    assert to_np(out).max() == 0
