"""Several attention heads in one call: forward and backward against the oracle head by head, for head widths on both sides
of a team of lanes and head counts that are and are not taken together, with rows and columns that a workgroup shares."""
import numpy as np
import pytest
import torch

from gas_inputs import rng
from oracle import ops as oops
from tests.test_gpu_ops import TOL, _gat_bwd_row_scale, _pattern_with_long_rows
from tests.util import node_rel_err, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("planned", [False, True])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("F,heads", [(64, 4), (48, 4), (64, 2), (32, 3), (32, 6), (128, 2), (128, 4), (136, 2), (100, 5), (8, 8)])
def test_heads_in_one_call(dtype, F, heads, planned):
    import paper_2106_05609_amd as gas
    nv = 400
    ptr, col = _pattern_with_long_rows(43, nv, empty_rows=False)
    col[::2] = 3                                               # a column of 17,000 entries
    nb, width = ptr.size - 1, F * heads
    rows = np.repeat(np.arange(nb), np.diff(ptr)).astype(np.int32)
    pos = np.lexsort((rows, col)).astype(np.int32)
    colptr = np.concatenate([[0], np.cumsum(np.bincount(col, minlength=nv))]).astype(np.int32)
    p = rng.normal_matrix(14, 980, nv, width, dtype=dtype) * 0.5
    a_dst, a_src = (rng.normal(14, s, 0, width, dtype=dtype) * 0.2 for s in (981, 982))
    gz = rng.normal_matrix(14, 983, nb, width, dtype=dtype)
    d_ptr, d_col, d_colptr, d_row, d_pos = (torch.from_numpy(a).cuda() for a in (ptr, col, colptr, rows[pos], pos))
    d_p, d_ad, d_as, d_gz = (t.cuda() for t in (p, a_dst, a_src, gz))
    z = torch.full((nb, width), float("nan"), dtype=dtype, device="cuda")
    gas.gas_gat_aggregate(d_ptr, d_col, d_p, d_ad, d_as, z, heads=heads)
    gp = torch.full((nv, width), float("nan"), dtype=dtype, device="cuda")
    gd, gs = (torch.full((width,), float("nan"), device="cuda") for _ in range(2))
    plan_t = gas.gas_plan_create(d_colptr, col.size, F, n_rows=nv, ind=d_row) if planned else None
    gas.gas_gat_aggregate_bwd(d_ptr, d_col, d_colptr, d_row, d_pos, d_p, d_ad, d_as, d_gz, gp, gd, gs, heads=heads, plan_t=plan_t)
    torch.cuda.synchronize()
    for h in range(heads):
        c = slice(h * F, (h + 1) * F)
        one = [np.ascontiguousarray(to_np(t[:, c].contiguous())) for t in (p, gz)]
        ad, asr = to_np(a_dst[c].contiguous()), to_np(a_src[c].contiguous())
        want = oops.gat_aggregate(ptr, col, one[0], ad, asr)
        assert node_rel_err(to_np(z[:, c]), want) <= TOL[dtype], (h, node_rel_err(to_np(z[:, c]), want))
        want_p, want_d, want_s = oops.gat_aggregate_bwd(ptr, col, one[0], ad, asr, one[1], nv, 0.2)
        scale = _gat_bwd_row_scale(ptr, col, one[0], ad, asr, one[1], nb, nv)     # of the sums that cancel
        assert node_rel_err(to_np(gp[:, c]), want_p, scale=scale) <= TOL[dtype], (h, node_rel_err(to_np(gp[:, c]), want_p, scale=scale))
        both = max(np.abs(want_d).max(), np.abs(want_s).max())
        assert np.abs(to_np(gd[c]) - want_d).max() <= TOL[dtype] * both and np.abs(to_np(gs[c]) - want_s).max() <= TOL[dtype] * both


def test_head_counts_that_do_not_divide_are_refused():
    import paper_2106_05609_amd as gas
    t = torch.zeros(3, 10, device="cuda")
    ptr, col = torch.zeros(4, dtype=torch.int32, device="cuda"), torch.zeros(0, dtype=torch.int32, device="cuda")
    for heads in (0, 3):
        with pytest.raises(ValueError):
            gas.gas_gat_aggregate(ptr, col, t, t[0], t[0], torch.empty_like(t), heads=heads)


def test_a_plan_that_is_not_used_may_have_more_entries():
    """Rows that the plain kernels take: the plan is not looked at; rows for the fast path: it is refused."""
    import paper_2106_05609_amd as gas
    nv, F = 6, 16
    ptr, col = torch.arange(nv + 1, dtype=torch.int32, device="cuda"), torch.arange(nv, dtype=torch.int32, device="cuda")
    other_ptr, other = 2 * ptr, torch.cat([col, col])
    plan = gas.gas_plan_create(other_ptr, 2 * nv, F, n_rows=nv, ind=other)
    rows = rng.normal_matrix(14, 995, nv, F + 2).cuda()
    a = rng.normal(14, 996, 0, F).cuda()
    gd, gs, gp = torch.empty(F, device="cuda"), torch.empty(F, device="cuda"), torch.empty(nv, F, device="cuda")
    call = lambda p, g: gas.gas_gat_aggregate_bwd(ptr, col, ptr, col, col, p, a, a, g, gp, gd, gs, plan_t=plan)
    call(rows[:, 1:F + 1], rows[:, 1:F + 1])
    assert torch.equal(gp, rows[:, 1:F + 1])               # one entry a row: its weight is 1, its score has no gradient
    with pytest.raises(gas.GasError):
        call(rows[:, :F].contiguous(), rows[:, :F].contiguous())


def test_more_columns_than_a_launch_has_wavefronts():
    """2^26 + 5 columns, entries in the first and the last of them, against the same entries on a table of those columns."""
    import paper_2106_05609_amd as gas
    if torch.cuda.mem_get_info()[0] < 24 << 30:
        pytest.skip("needs 24 GiB of device memory")
    n_cols, nb, F, heads = (1 << 26) + 5, 10, 8, 2
    width = F * heads
    d = lambda a: torch.from_numpy(a.astype(np.int32)).cuda()
    used = np.concatenate([np.arange(nb), n_cols - nb + np.arange(nb)])           # columns with an entry, in order
    small_col = np.stack([np.arange(nb), nb + np.arange(nb)], 1).reshape(-1)      # row v: columns v and nb + v of those
    pos = np.concatenate([2 * np.arange(nb), 2 * np.arange(nb) + 1])              # CSC order
    ptr, row = d(2 * np.arange(nb + 1)), d(np.concatenate([np.arange(nb), np.arange(nb)]))
    small_p = (rng.normal_matrix(14, 997, 2 * nb, width, dtype=torch.bfloat16) * 0.5).cuda()
    ad, asr = ((rng.normal(14, s, 0, width, dtype=torch.bfloat16) * 0.2).cuda() for s in (998, 999))
    gz = rng.normal_matrix(14, 1000, nb, width, dtype=torch.bfloat16).cuda()
    big_p = torch.zeros(n_cols, width, dtype=torch.bfloat16, device="cuda")
    big_p[torch.from_numpy(used).cuda()] = small_p
    big_ptr = torch.full((n_cols + 1,), nb, dtype=torch.int32, device="cuda")
    big_ptr[:nb + 1] = torch.arange(nb + 1, device="cuda")
    big_ptr[-nb - 1:] += torch.arange(nb + 1, dtype=torch.int32, device="cuda")
    got = []
    for p, col, colptr in ((big_p, used[small_col], big_ptr), (small_p, small_col, d(np.arange(2 * nb + 1)))):
        gp = torch.full_like(p, 7.0)
        gd, gs = (torch.empty(width, device="cuda") for _ in range(2))
        gas.gas_gat_aggregate_bwd(ptr, d(col), colptr, row, d(pos), p, ad, asr, gz, gp, gd, gs, heads=heads)
        got.append((gp, gd, gs))
    at = torch.from_numpy(used).cuda()
    assert torch.equal(got[0][0][at], got[1][0])
    assert bool((got[0][0][nb:n_cols - nb] == 0).all())
    assert torch.allclose(got[0][1], got[1][1], rtol=1e-5, atol=1e-6) and torch.allclose(got[0][2], got[1][2], rtol=1e-5, atol=1e-6)


@pytest.mark.parametrize("F,heads", [(64, 4), (256, 1)])
def test_zero_attention_vectors_cost_no_more_than_others(F, heads):
    """All scores are exactly zero: nothing to form again in 64 bits (which took 1.5 to 1.6 times as long)."""
    import paper_2106_05609_amd as gas
    nb, deg, width = 60000, 12, F * heads
    ptr = (torch.arange(nb + 1) * deg).int().cuda()
    col = ((torch.arange(nb)[:, None] + 37 * torch.arange(deg)[None, :] * (1 + torch.arange(nb)[:, None] % 5)) % nb).reshape(-1)
    rows = torch.arange(nb).repeat_interleave(deg)
    pos = torch.argsort(col, stable=True)
    colptr = torch.cat([torch.zeros(1), torch.cumsum(torch.bincount(col, minlength=nb), 0)]).int().cuda()
    args = (ptr, col.int().cuda(), colptr, rows[pos].int().cuda(), pos.int().cuda())
    p, gz = (rng.normal_matrix(14, s, nb, width).cuda() for s in (1010, 1011))
    gp, gd, gs = torch.empty_like(p), torch.empty(width, device="cuda"), torch.empty(width, device="cuda")
    best = {}
    for scale in (0.1, 0.0, 0.1, 0.0):
        ad, asr = (scale * rng.normal(14, s, 0, width).cuda() for s in (1012, 1013))
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(5):
                gas.gas_gat_aggregate_bwd(*args, p, ad, asr, gz, gp, gd, gs, heads=heads)
            b.record()
            b.synchronize()
            best[scale] = min(best.get(scale, 1e9), a.elapsed_time(b))
    assert best[0.0] <= 1.25 * best[0.1], best
