"""bf16 products with a Push: which take it along (one launch) and which leave it to a copy of the rows (two), and that either
stores the product's rows.  The sizes are those on both sides of each line."""
import ctypes as C

import pytest
import torch

from gas_inputs import rng

pytestmark = pytest.mark.gpu


def _launches(call):
    """Kernels of a call, as nodes of a captured graph that is replayed once."""
    from paper_2106_05609_amd import binding as B
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        call()
    count = C.c_size_t()
    assert B.lib().hipGraphGetNodes(C.c_void_p(graph.raw_cuda_graph()), None, C.byref(count)) == 0
    graph.instantiate()
    graph.replay()
    torch.cuda.synchronize()
    return count.value


def _matrices(seed, *shapes):
    return [rng.normal_matrix(13, seed + i, *s).to("cuda").to(torch.bfloat16) for i, s in enumerate(shapes)]


def _target(n, width):
    idx = torch.randperm(2 * n, generator=torch.Generator().manual_seed(n), dtype=torch.int64)[:n].to(torch.int32).cuda()
    return idx, torch.zeros(2 * n, width, dtype=torch.bfloat16, device="cuda")


@pytest.mark.parametrize("n,f_in,f_out,want", [
    (4096, 128, 128, 2), (6144, 128, 128, 2), (6145, 128, 128, 1), (16000, 128, 128, 1), (3072, 128, 256, 2), (16000, 128, 256, 1),
    (1, 64, 64, 1), (24000, 64, 64, 1), (5000, 128, 48, 1), (20480, 128, 48, 1), (20481, 128, 48, 2), (65537, 128, 48, 1),
    (16000, 256, 256, 2), (16448, 256, 256, 1), (1, 136, 8, 2)])
def test_product(n, f_in, f_out, want):
    import paper_2106_05609_amd as gas
    z, w = _matrices(720, (n, f_in), (f_in, f_out))
    y = torch.empty(n, f_out, dtype=torch.bfloat16, device="cuda")
    idx, hist = _target(n, f_out)
    assert _launches(lambda: gas.gas_linear_push(z, w, y, idx, hist, relu=True)) == want
    assert torch.equal(hist[idx.long()], y) and int((hist != 0).any(1).sum()) <= n
    exact = torch.relu(z.double() @ w.double())
    # an fp32 sum of f_in products, rounded to bf16 once
    bound = f_in * 2.0 ** -23 * (z.abs().double() @ w.abs().double()) + 2.0 ** -8 * exact
    assert bool(((y.double() - exact).abs() <= bound).all())


@pytest.mark.parametrize("keep", [False, True])
@pytest.mark.parametrize("n,f_in,hidden,f_out,want,want_keep", [
    (1, 64, 64, 64, 1, 1), (4096, 64, 64, 64, 1, 1), (30000, 64, 64, 64, 1, 1), (30001, 64, 64, 64, 1, 2), (30001, 72, 64, 48, 1, 1),
    (500, 128, 128, 128, 1, 1), (12000, 128, 128, 128, 1, 1), (24000, 256, 64, 64, 1, 1), (300, 256, 256, 256, 1, 1)])
def test_mlp(n, f_in, hidden, f_out, want, want_keep, keep):
    import paper_2106_05609_amd as gas
    z, w1, w2 = _matrices(730, (n, f_in), (f_in, hidden), (hidden, f_out))
    y, h = (torch.empty(n, f, dtype=torch.bfloat16, device="cuda") for f in (f_out, hidden))
    idx, hist = _target(n, f_out)
    if keep:
        assert _launches(lambda: gas.gas_mlp2_keep(z, w1, w2, y, h, idx, hist, relu_out=True)) == want_keep
    else:
        assert _launches(lambda: gas.gas_mlp2_push(z, w1, w2, y, idx, hist, relu_out=True)) == want
        gas.gas_mlp2_keep(z, w1, w2, torch.empty_like(y), h)
    assert torch.equal(hist[idx.long()], y) and int((hist != 0).any(1).sum()) <= n
    exact = torch.relu(h.double() @ w2.double())             # from the hidden rows as they were rounded
    bound = hidden * 2.0 ** -23 * (h.double() @ w2.abs().double()) + 2.0 ** -8 * exact
    if not keep:                                             # another kernel may round a hidden value the other way
        bound = bound + 2.0 ** -7 * (h.double() @ w2.abs().double())
    assert bool(((y.double() - exact).abs() <= bound).all())


@pytest.mark.parametrize("n,f_in,hidden,keep,want", [
    (4096, 256, 64, False, 1), (5000, 128, 128, True, 2), (5001, 128, 128, True, 1), (100000, 256, 64, True, 2), (100001, 256, 64, True, 1),
    (100001, 128, 64, True, 2)])
def test_mlp_without_a_push(n, f_in, hidden, keep, want):
    import paper_2106_05609_amd as gas
    z, w1, w2 = _matrices(740, (n, f_in), (f_in, hidden), (hidden, 64))
    y, h = torch.empty(n, 64, dtype=torch.bfloat16, device="cuda"), torch.empty(n, hidden, dtype=torch.bfloat16, device="cuda")
    if keep:
        assert _launches(lambda: gas.gas_mlp2_keep(z, w1, w2, y, h, relu_out=True)) == want
    else:
        assert _launches(lambda: gas.gas_mlp2(z, w1, w2, y, relu_out=True)) == want
    exact_h = torch.relu(z.double() @ w1.double())
    hidden_bound = f_in * 2.0 ** -23 * (z.abs().double() @ w1.abs().double()) + 2.0 ** -8 * exact_h
    if keep:
        assert bool(((h.double() - exact_h).abs() <= hidden_bound).all())
    exact = torch.relu(exact_h @ w2.double())
    bound = (hidden_bound + hidden * 2.0 ** -23 * exact_h) @ w2.abs().double() + 2.0 ** -8 * exact
    assert bool(((y.double() - exact).abs() <= 1.01 * bound).all())
