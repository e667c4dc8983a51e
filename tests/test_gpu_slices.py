"""Light rows by slices at every form that the rule takes (pieces a lane, contiguous and in turn, few and many rows), at widths
around the slices' edges and at widths that are no whole number of 16-byte units; the sums of heavy rows' chunks around the
batches of eight.  Against 64-bit sums, with the bound of an fp32 sum of the row's terms in any order."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gas():
    import paper_2106_05609_amd as g
    g.lib()
    return g


def _pattern(n, mean, seed, longest=None):
    r = np.random.default_rng(seed)
    lengths = r.integers(0, 2 * mean + 1, n)
    lengths[:: max(1, n // 7)] = longest or 2 * mean + 33
    ptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    return torch.from_numpy(ptr).cuda(), r


def _check(z, ptr, terms, extra, own_terms):
    """z against the 64-bit sum of `terms` [nnz, F] (64 bits) over the rows plus `extra`; own_terms: what the extras add to a
    row's magnitude.  A sum of k products in fp32 is within (k + 3) 2^-24 of the terms' magnitudes, and rounding to bf16 2^-9."""
    n = ptr.numel() - 1
    lengths = (ptr[1:] - ptr[:-1]).long()
    row = torch.repeat_interleave(torch.arange(n, device="cuda"), lengths)
    want = torch.zeros(n, terms.shape[1], dtype=torch.float64, device="cuda").index_add_(0, row, terms) + extra
    size = torch.zeros_like(want).index_add_(0, row, terms.abs()) + own_terms
    bound = (lengths[:, None] + 6) * 2.0 ** -24 * size + 1e-30
    if z.dtype == torch.bfloat16:
        bound = bound + 2.0 ** -8 * want.abs()
    worst = ((z.double() - want).abs() / bound).max().item()
    assert worst <= 1.0, worst


WIDTHS = [(torch.float32, f) for f in (4, 29, 61, 64, 65, 124, 128, 130, 190, 193, 250, 256, 257, 1030)] + \
         [(torch.bfloat16, f) for f in (8, 121, 128, 129, 250, 256, 264, 384, 390, 512, 520)]


@pytest.mark.parametrize("dtype,F", WIDTHS)
@pytest.mark.parametrize("n,mean,clustered", [(17, 5, 1), (33, 9, 2), (8193, 4, 1), (9000, 22, 1), (16385, 4, 2), (16400, 30, 2), (65537, 2, 2)])
def test_slices_at_every_form(gas, n, mean, clustered, dtype, F):
    if n * F > 10_000_000:
        F = F % 300 + 4 if dtype == torch.float32 else F
    ptr, r = _pattern(n, mean, n + F)
    nnz, nh = int(ptr[-1]), 40
    gen = torch.Generator(device="cuda").manual_seed(n + F)
    x = torch.randn(n, F, generator=gen, device="cuda").to(dtype)
    hist = torch.randn(nh, F, generator=gen, device="cuda").to(dtype)
    res, y = (torch.randn(n, F, generator=gen, device="cuda").to(dtype) for _ in range(2))
    val = torch.randn(nnz, generator=gen, device="cuda")
    col = torch.from_numpy(r.integers(0, n + nh, nnz).astype(np.int32)).cuda()
    src = torch.where(col < n, col, n - 1 - col)                     # history row h is stored as -1 - h
    plan = gas.gas_plan_create(ptr, nnz, F, ind=src, options=dict(xcd_ranges=clustered))
    assert plan.describe()["n_heavy"] == 0
    rows = torch.cat([x, hist]).double()
    terms = val.double()[:, None] * rows[col.long()]
    for out in (dtype, torch.float32):
        z = torch.full((n, F), float("nan"), dtype=out, device="cuda")
        gas.gas_spmm_hist(plan, ptr, src, val, x, hist, z, diag=1.25, s_agg=0.5, r=res, s_res=2.0)
        extra = 1.25 * x.double() + 2.0 * res.double()
        _check(z, ptr, 0.5 * terms, extra, 1.25 * x.double().abs() + 2.0 * res.double().abs())
    own = torch.minimum(col, torch.full_like(col, n - 1))
    z = torch.full((n, F), float("nan"), dtype=dtype, device="cuda")
    gas.gas_spmm_t_relu(plan, ptr, own, None, x, y, z)
    on = (y > 0).double()
    row = torch.repeat_interleave(torch.arange(n, device="cuda"), (ptr[1:] - ptr[:-1]).long())
    _check(z, ptr, x.double()[own.long()] * on[row], 0.0, 0.0)
    assert (z[y <= 0] == 0).all()
    # the first layer's form: one table, and the diagonal term's rows by ids
    ids = torch.from_numpy(r.permutation(n + nh)[:n].astype(np.int32)).cuda()
    table = torch.cat([x, hist])
    z = torch.full((n, F), float("nan"), dtype=dtype, device="cuda")
    gas.gas_spmm_table(plan, ptr, -1 - col, val, table, z, diag=0.75, own=ids)
    _check(z, ptr, terms, 0.75 * table[ids.long()].double(), 0.75 * table[ids.long()].double().abs())


@pytest.mark.parametrize("F", [40, 64, 100, 150, 250, 256, 300])
@pytest.mark.parametrize("clustered,n", [(1, 8200), (2, 40), (2, 16500)])
def test_slices_with_infinities_and_nan(gas, F, clustered, n):
    """A non-finite value reaches the rows that name it and no other, also as a row's last entry (loads past a row's end are of
    its last entry, and are not folded)."""
    ptr, r = _pattern(n, 5, 3 * n + F)
    nnz = int(ptr[-1])
    x = torch.randn(n, F, device="cuda")
    x[1], x[2, F // 2], x[3] = float("inf"), float("nan"), -float("inf")
    col = torch.from_numpy(r.integers(4, n, nnz).astype(np.int32)).cuda()
    last = (ptr[1:][ptr[1:] > ptr[:-1]] - 1).long()
    col[last[::3]], col[last[1::3]], col[last[2::5]] = 1, 2, 3
    plan = gas.gas_plan_create(ptr, nnz, F, ind=col, options=dict(xcd_ranges=clustered))
    z = torch.empty(n, F, device="cuda")
    gas.gas_spmm(plan, ptr, col, None, x, z)
    row = torch.repeat_interleave(torch.arange(n, device="cuda"), (ptr[1:] - ptr[:-1]).long())
    want = torch.zeros(n, F, device="cuda").index_add_(0, row, x[col.long()])
    assert torch.equal(torch.isnan(z), torch.isnan(want))
    assert torch.equal(torch.where(torch.isinf(z), z, 0.0), torch.where(torch.isinf(want), want, 0.0))


@pytest.mark.parametrize("dtype,F", [(torch.float32, 256), (torch.float32, 37), (torch.bfloat16, 256), (torch.bfloat16, 72)])
def test_chunks_of_heavy_rows_are_added_in_batches(gas, dtype, F):
    """Heavy rows of 1 to 18 chunks, and light ones between them, also where these go by slices."""
    lengths = np.array([k * 16 - (k % 3) + 20 * (k == 1) for k in range(1, 19)] + [3, 0, 8] * 6)
    ptr = torch.from_numpy(np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)).cuda()
    n, nnz = len(lengths), int(lengths.sum())
    gen = torch.Generator(device="cuda").manual_seed(F)
    x = torch.randn(500, F, generator=gen, device="cuda").to(dtype)
    val = torch.randn(nnz, generator=gen, device="cuda")
    col = torch.randint(0, 500, (nnz,), generator=gen, device="cuda", dtype=torch.int32)
    for clustered in (1, 2):
        plan = gas.gas_plan_create(ptr, nnz, F, ind=col, options=dict(heavy_threshold=10, chunk=16, window_rows=-1, xcd_ranges=clustered))
        assert plan.describe()["n_heavy"] == 18
        z = torch.full((n, F), float("nan"), dtype=dtype, device="cuda")
        gas.gas_spmm(plan, ptr, col, val, x, z, diag=0.5)
        _check(z, ptr, val.double()[:, None] * x.double()[col.long()], 0.5 * x[:n].double(), 0.5 * x[:n].double().abs())


def _in_parts(x, ptr, col, parts):
    """The rows' sums in fp32, entry k of a row into sum k % parts, the sums added pair by pair; of eight, the even ones and the odd
    ones each pair by pair first, which two halves of a team hold."""
    ptr, col = ptr.cpu().numpy(), col.cpu().numpy()
    lengths, n = np.diff(ptr), len(ptr) - 1
    acc = np.zeros((parts, n, x.shape[1]), np.float32)
    for k in range(int(lengths.max())):
        rows = np.flatnonzero(lengths > k)
        acc[k % parts, rows] += x[col[ptr[rows] + k]]
    for d in (2, 4, 1) if parts == 8 else [d for d in (1, 2) if d < parts]:
        for t in range(parts):
            if not t & d and not t & (6 if d == 1 and parts == 8 else 0) and t + d < parts:
                acc[t] += acc[t + d]
    return acc[0]


# widths, where their rows start (elements past 16 bytes) and the partial sums of a row: a narrow row has as many as a wavefront's
# teams would make of it, and one of 32 units two unless it is whole and aligned, when a wavefront takes it at once
@pytest.mark.parametrize("dtype,F,offset,parts", [
    (torch.float32, 5, 0, 8), (torch.float32, 31, 1, 8), (torch.float32, 32, 0, 8), (torch.float32, 33, 0, 4), (torch.float32, 64, 0, 4),
    (torch.float32, 65, 0, 2), (torch.float32, 104, 0, 2), (torch.float32, 125, 0, 2), (torch.float32, 126, 3, 2), (torch.float32, 127, 0, 2),
    (torch.float32, 128, 1, 2), (torch.float32, 128, 0, 1), (torch.float32, 129, 0, 1), (torch.float32, 256, 0, 1),
    (torch.bfloat16, 64, 0, 8), (torch.bfloat16, 128, 0, 4), (torch.bfloat16, 200, 0, 2), (torch.bfloat16, 249, 0, 2),
    (torch.bfloat16, 255, 1, 2), (torch.bfloat16, 256, 1, 2), (torch.bfloat16, 256, 0, 1)])
@pytest.mark.parametrize("n", [500, 8200])           # by one piece a lane; above 8,192 rows by two where that form exists
def test_partial_sums_of_a_row(gas, n, dtype, F, offset, parts):
    """Bit for bit the sums in that many parts: rows long enough that one part fewer, or one more, gives other bits."""
    ptr, r = _pattern(n, 12, 5 * n + F, longest=200)
    nnz = int(ptr[-1])
    gen = torch.Generator(device="cuda").manual_seed(F + offset)
    stride = F + offset if offset else (F + 7) // 8 * 8
    x = torch.randn(n, stride, generator=gen, device="cuda").to(dtype)[:, offset:offset + F]
    col = torch.from_numpy(r.integers(0, n, nnz).astype(np.int32)).cuda()
    plan = gas.gas_plan_create(ptr, nnz, F, ind=col, options=dict(xcd_ranges=1))
    assert plan.describe()["n_heavy"] == 0
    z = torch.full((n, F), float("nan"), device="cuda")
    gas.gas_spmm(plan, ptr, col, None, x, z)
    host = x.float().cpu().numpy()
    assert np.array_equal(z.cpu().numpy(), _in_parts(host, ptr, col, parts))
    if parts > 1:
        assert not np.array_equal(z.cpu().numpy(), _in_parts(host, ptr, col, parts // 2))


@pytest.mark.parametrize("F,offset,parts", [(128, 0, 1), (128, 1, 4), (120, 0, 4), (136, 0, 2)])
def test_rows_of_128_bf16_to_bf16_are_summed_in_order(gas, F, offset, parts):
    """Whole ones in one sum, as where a wavefront takes a row at once: a row's first entry is 2^18 times the others and its last takes
    it away again, so that the order shows through the rounding to bf16."""
    n = 3000
    ptr, r = _pattern(n, 12, 77, longest=200)
    gen = torch.Generator(device="cuda").manual_seed(F + offset)
    x = torch.randn(n, F + offset if offset else (F + 7) // 8 * 8, generator=gen, device="cuda")
    x[:100] *= 2.0 ** 18
    x[100:200] = -x[:100]
    x = x.to(torch.bfloat16)[:, offset:offset + F]
    col, ends = r.integers(200, n, int(ptr[-1])).astype(np.int32), ptr.cpu().numpy()
    rows = np.flatnonzero(np.diff(ends) > 1)
    col[ends[rows]], col[ends[rows + 1] - 1] = rows % 100, 100 + rows % 100
    col = torch.from_numpy(col).cuda()
    z = torch.empty(n, F, dtype=torch.bfloat16, device="cuda")
    gas.gas_spmm(gas.gas_plan_create(ptr, int(ptr[-1]), F, ind=col, options=dict(xcd_ranges=1)), ptr, col, None, x, z)
    want = {k: torch.from_numpy(_in_parts(x.float().cpu().numpy(), ptr, col, k)).to(torch.bfloat16) for k in (1, 2, 4)}
    assert torch.equal(z.cpu(), want[parts])
    assert all(not torch.equal(want[parts], w) for k, w in want.items() if k != parts)
