"""The aggregation of a first layer, whose rows all lie in the feature table (gas_spmm_table): the bits of gas_pull followed by
gas_spmm (which tests/test_gpu_ops.py holds against the oracle)."""
import pytest
import torch

pytestmark = pytest.mark.gpu


# rows by slices, by groups, by units, element by element, in panels; one row longer than a chunk; a table whose rows are strided
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("f,ld", [(256, 256), (128, 144), (100, 100), (3, 5), (1433, 1433)])
@pytest.mark.parametrize("rows,longest", [(1, 3), (64, 70), (900, 20), (900, 1500)])
@pytest.mark.parametrize("diag", [0.0, 1.25])
def test_spmm_table_has_the_bits_of_pull_and_spmm(rows, longest, f, ld, dtype, diag):
    import paper_2106_05609_amd as gas
    gen = torch.Generator().manual_seed(rows + f)
    n, nv = 4 * rows + 50, 2 * rows + 20
    lengths = torch.randint(0, 12, (rows,), generator=gen)
    lengths[rows // 2] = longest
    ptr = torch.cat([torch.zeros(1, dtype=torch.long), lengths.cumsum(0)]).int().cuda()
    col = torch.cat([torch.randint(0, nv, (int(k),), generator=gen).sort().values for k in lengths]).int().cuda()
    val = torch.rand(col.numel(), generator=gen).cuda()
    ids = torch.randperm(n, generator=gen)[:nv].int().cuda()
    table = torch.randn(n, ld, generator=gen).to(dtype).cuda()[:, :f]
    plan = gas.gas_plan_create(ptr, col.numel(), f, ind=col)
    x, z, want = torch.empty((nv, f), dtype=dtype, device="cuda"), *(torch.full((rows, f), 3.0, dtype=dtype, device="cuda") for _ in range(2))
    gas.gas_pull(table, ids, x)
    gas.gas_spmm(plan, ptr, col, val, x, want, diag=diag, s_agg=0.5)
    src = torch.empty_like(col)
    gas.gas_fuse_sources(col, 0, ids, src)
    gas.gas_spmm_table(plan, ptr, src, val, table, z, diag=diag, s_agg=0.5, own=ids if diag else None)
    assert torch.equal(z, want)
    if diag:
        with pytest.raises(gas.GasError):
            gas.gas_spmm_table(plan, ptr, src, val, table, z, diag=diag)


@pytest.mark.parametrize("op,train", [("gcn", False), ("gcn", True), ("gin", False), ("gin", True), ("gcnii", False), ("gcnii", True)])
def test_first_layer_indices_are_built_for_passes_that_read_them(op, train):
    """By GCN and by GIN's inference, in their first pass and not with the other indices; a captured first pass records the
    building and leaves the batch without them."""
    from gas_inputs import batches, graphs
    from paper_2106_05609_amd import executor
    dev = torch.device("cuda")
    g = graphs.sbm_partners(2_000, 8, 6.0, 0.85, 3, dev)
    sg = batches.batch_subgraph(g, batches.split(g, 2, 0)[0], self_loops=op != "gin")
    gen = torch.Generator(device=dev).manual_seed(1)
    normal = lambda *shape: torch.randn(*shape, generator=gen, device=dev) / shape[0] ** 0.5
    ws = [(normal(200, 200), normal(200, 200)) if op == "gin" else normal(200, 200) for _ in range(2)]
    model = executor.Model(op, ws, normal(200, 200) if op == "gcnii" else None, 0.1 if op == "gcnii" else 0.0)
    x, tables = normal(2_000, 200), [normal(2_000, 200)]
    labels = torch.zeros(sg.nb, dtype=torch.int32, device=dev)

    def batch():
        bg = executor.BatchGraph(sg.nb, sg.n_id, sg.rowptr, sg.col, g.deg, sg.colptr, sg.row, max_F=256, normalise=op != "gin")
        bg.src
        bg.plan_t_all
        return bg

    def run(bg):
        if train:
            return executor.train_step(model, bg, x, tables, labels, 0.0, n_labelled=sg.nb, fused=True)[2]
        return executor.forward_batch_fused(model, bg, x, tables)
    eager, captured = batch(), batch()
    assert eager._src_first is None
    want = run(eager).clone()
    reads = op == "gcn" or (op == "gin" and not train)
    assert (eager._src_first is not None) == reads
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        got = run(captured)
    assert captured._src_first is None and torch.equal(run(captured), want)
    for _ in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(got, want)
