"""Consecutive narrow layers in one call (gas_spmm_linear_layers, gas_spmm_t_relu_linear_layers): the bits of one call per
layer (which tests/test_gpu_ops.py and tests/test_gpu_fused_backward.py hold against the oracle)."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _pattern(rows, cols, degree, gen):
    """int32 CSR of `rows` rows whose lengths run from 0 to 2 * degree, ascending columns below `cols`."""
    n = torch.randint(0, 2 * degree + 1, (rows,), generator=gen)
    n[0] = 0 if rows > 1 else 2
    col = torch.cat([torch.randint(0, cols, (int(k),), generator=gen).sort().values for k in n] + [torch.zeros(0, dtype=torch.long)])
    ptr = torch.cat([torch.zeros(1, dtype=torch.long), n.cumsum(0)])
    return ptr.int().cuda(), col.int().cuda(), torch.rand(col.numel(), generator=gen).cuda()


@pytest.mark.parametrize("rows,f,degree,count", [(1, 64, 3, 1), (33, 32, 5, 4), (500, 48, 40, 5), (2100, 64, 9, 70), (3000, 128, 8, 3)])
@pytest.mark.parametrize("keep", [False, True])
def test_layers_together_have_the_bits_of_single_layers(rows, f, degree, count, keep):
    import paper_2106_05609_amd as gas
    gen = torch.Generator().manual_seed(rows + f)
    nv, n_hist = rows + rows // 2 + 1, 2 * rows + 7
    normal = lambda *shape: torch.randn(*shape, generator=gen).cuda()
    ptr, col, val = _pattern(rows, nv, degree, gen)
    ids = torch.randperm(n_hist, generator=gen)[:nv].int().cuda()
    src = torch.empty_like(col)
    gas.gas_fuse_sources(col, rows, ids, src)
    x0 = normal(nv, f)
    ws = [normal(f, f) / f ** 0.5 for _ in range(count)]
    c_id, c_w = [0.1 * (l % 5) for l in range(count)], [1.0 - 0.1 * (l % 5) for l in range(count)]
    stored = normal(count, n_hist, f)
    results = []
    for together in (False, True):
        hist = stored.clone()
        tables = [hist[l] for l in range(count - 1)]
        zs = [torch.full((rows, f), 7.0, device="cuda") for _ in range(count)] if keep else None
        ys = [torch.empty((rows, f), device="cuda") for _ in range(count if keep else 2)]
        out = [ys[l] if keep else ys[l % 2] for l in range(count)]
        push = ids[:rows].contiguous()
        if together:
            gas.gas_spmm_linear_layers(ptr, col, src, val, x0, ws, out, [None] + tables, s_agg=0.9, r=x0, s_res=0.1,
                                       c_identity=c_id, c_weight=c_w, z_outs=zs, push_idx=push, push_hists=tables + [None])
        else:
            for l in range(count):
                gas.gas_spmm_linear(ptr, col if l == 0 else src, val, x0 if l == 0 else out[l - 1], ws[l], out[l],
                                    hist=None if l == 0 else tables[l - 1], s_agg=0.9, r=x0, s_res=0.1, c_identity=c_id[l],
                                    c_weight=c_w[l], relu=l + 1 < count, z_out=zs[l] if keep else None,
                                    push_idx=push if l + 1 < count else None, push_hist=tables[l] if l + 1 < count else None)
        torch.cuda.synchronize()
        results.append([hist, out[-1]] + (zs + ys if keep else []))
    assert torch.isfinite(results[0][1]).all()
    for a, b in zip(*results):
        assert torch.equal(a, b)


@pytest.mark.parametrize("rows,f,degree,count", [(1, 64, 3, 1), (33, 32, 5, 4), (500, 48, 40, 5), (2100, 64, 9, 70), (3000, 128, 8, 3)])
@pytest.mark.parametrize("with_total", [False, True])
def test_backward_layers_together_have_the_bits_of_single_layers(rows, f, degree, count, with_total):
    import paper_2106_05609_amd as gas
    gen = torch.Generator().manual_seed(rows + f)
    normal = lambda *shape: torch.randn(*shape, generator=gen).cuda()
    ptr, row, val = _pattern(rows, rows, degree, gen)
    g0, start = normal(rows, f), normal(rows, f)
    ws = [normal(f, f) / f ** 0.5 for _ in range(count)]
    ys = [normal(rows, f).clamp_(min=0) for _ in range(count)]
    c_id, c_w = [0.1 * (l % 5) for l in range(count)], [1.0 - 0.1 * (l % 5) for l in range(count)]
    results = []
    for together in (False, True):
        total = start.clone() if with_total else None
        gxs = [torch.empty((rows, f), device="cuda") for _ in range(count)]
        gz = [torch.empty((rows, f), device="cuda") for _ in range(2)]
        gzs = [gz[l % 2] for l in range(count)]
        if together:
            gas.gas_spmm_t_relu_linear_layers(ptr, row, val, g0, ys, gxs, ws, gzs, s_agg=0.9, c_identity=c_id, c_weight=c_w,
                                              total=total, c_total=0.1)
        else:
            for l in range(count):
                gas.gas_spmm_t_relu_linear(ptr, row, val, g0 if l == 0 else gzs[l - 1], ys[l], gxs[l], ws[l], gzs[l], s_agg=0.9,
                                           c_identity=c_id[l], c_weight=c_w[l], total=total, c_total=0.1)
        torch.cuda.synchronize()
        results.append(gxs + [gzs[-1]] + ([total] if with_total else []))
    for a, b in zip(*results):
        assert torch.equal(a, b)


def test_refused_layers():
    """Shapes that do not match, a layer that would write what it reads, a type that the single call refuses."""
    import paper_2106_05609_amd as gas
    gen = torch.Generator().manual_seed(3)
    ptr, col, val = _pattern(700, 700, 6, gen)
    x = torch.randn(700, 64, generator=gen).cuda()
    ws = [torch.randn(64, 64, generator=gen).cuda() / 8 for _ in range(5)]
    ys = [torch.full((700, 64), 2.0, device="cuda") for _ in range(2)]
    with pytest.raises(gas.GasError):
        gas.gas_spmm_linear_layers(ptr, col, col, val, x, ws[:3], [ys[0], ys[1], ys[1]], [None] * 3)
    with pytest.raises(ValueError):
        gas.gas_spmm_linear_layers(ptr, col, col, val, x, ws, ys, [None] * 5)
    b = lambda t: t.bfloat16()
    with pytest.raises(gas.GasError):
        gas.gas_spmm_linear_layers(ptr, col, col, val, b(x), [b(w) for w in ws[:2]], [b(y) for y in ys], [None] * 2)
    torch.cuda.synchronize()
    assert all((y == 2.0).all() for y in ys)                 # nothing was launched


# layers that fill several flushes of waiting weight gradients, and fewer than one; a batch without halo rows
@pytest.mark.parametrize("layers,width,blocks", [(36, 64, 2), (19, 32, 2), (3, 128, 2), (2, 48, 1), (17, 64, 6)])
def test_passes_by_groups_have_the_bits_of_passes_by_single_layers(layers, width, blocks, monkeypatch):
    """Outputs, pushed tables and every gradient of a GCNII, in groups and with the groups switched off, which is what a larger
    batch takes."""
    from gas_inputs import batches, graphs
    from paper_2106_05609_amd import binding as B, executor
    dev = torch.device("cuda")
    g = graphs.sbm_partners(3_000, 6, 7.0, 0.85, 3, dev)
    sg = batches.batch_subgraph(g, batches.split(g, 6 // blocks if blocks < 6 else 6, 0)[0], self_loops=True)
    gen = torch.Generator(device=dev).manual_seed(layers)
    normal = lambda *shape: torch.randn(*shape, generator=gen, device=dev)
    model = executor.Model("gcnii", [normal(width, width) / width ** 0.5 for _ in range(layers)], normal(20, width) / 20 ** 0.5, 0.1)
    x, stored, grad = normal(3_000, 20), normal(layers - 1, 3_000, width).clamp_(min=0), normal(sg.nb, width)
    calls = []
    for name in ("gas_spmm_linear_layers", "gas_spmm_t_relu_linear_layers", "gas_spmm_linear", "gas_spmm_t_relu_linear"):
        monkeypatch.setattr(B, name, lambda *a, _f=getattr(B, name), _n=name, **kw: (calls.append(_n), _f(*a, **kw))[1])
    together, results = executor._layers_together, []
    for on in (True, False):
        monkeypatch.setattr(executor, "_layers_together", together if on else lambda *a: False)
        bg = executor.BatchGraph(sg.nb, sg.n_id, sg.rowptr, sg.col, g.deg, sg.colptr, sg.row, max_F=128)
        tables, tables2 = stored.clone(), stored.clone()
        calls.clear()
        y = executor.forward_batch_fused(model, bg, x, tables)
        assert set(calls) == {"gas_spmm_linear_layers" if on else "gas_spmm_linear"}
        calls.clear()
        y2, grads, kept = executor.train_batch(model, bg, x, tables2, grad, fused=True)
        assert ("gas_spmm_linear_layers" in calls) == on and ("gas_spmm_linear" in calls) != on
        if layers >= 4:                        # fewer do not share their weight gradients' launches
            assert ("gas_spmm_t_relu_linear_layers" in calls) == on and ("gas_spmm_t_relu_linear" in calls) != on
        results.append([y, tables, y2, tables2] + [grads[l] for l in range(layers)] + [grads["w_in"]] +
                       [t for z, _, out in kept["layers"] for t in (z, out)])
    assert torch.isfinite(results[0][0]).all()
    for a, b in zip(*results):
        assert torch.equal(a, b)
