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
