"""Backward calls that take several steps in one pass, against the calls they stand for: the same bits."""
import numpy as np
import pytest
import torch

from gas_inputs import rng

pytestmark = pytest.mark.gpu


def _pattern(n_rows, n_cols, long_row):
    lens = np.array([(5 * i) % 9 for i in range(n_rows)])
    lens[n_rows // 3] = long_row
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    col = np.concatenate([np.sort((np.arange(k) * 31 + 7 * i) % n_cols) for i, k in enumerate(lens)]).astype(np.int32)
    return torch.from_numpy(ptr).cuda(), torch.from_numpy(col).cuda()


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("F", [3, 47, 64, 100, 128, 256, 512, 1433])
@pytest.mark.parametrize("diag", [0.0, 1.1])
def test_adjoint_and_relu_in_one_pass(F, dtype, diag):
    import paper_2106_05609_amd as gas
    n, m = 300, 200
    ptr, col = _pattern(n, m, 1200)
    g = rng.normal_matrix(5, 900, m, F, dtype=dtype).cuda()
    y = rng.normal_matrix(5, 901, n, F, dtype=dtype).clamp(min=0).cuda()
    y[7, 0], y[8, F - 1] = float("nan"), -0.0                     # neither is positive
    val = rng.normal(5, 902, 0, col.numel()).cuda()
    plan = gas.gas_plan_create(ptr, col.numel(), F, ind=col)
    want, got = (torch.full((n, F), float("nan"), dtype=dtype, device="cuda") for _ in range(2))
    gas.gas_spmm_t(plan, ptr, col, val, g, want, diag=diag, s_agg=0.9)
    gas.gas_relu_bwd(want, y, want)
    gas.gas_spmm_t_relu(plan, ptr, col, val, g, y, got, diag=diag, s_agg=0.9)
    assert torch.equal(got, want)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("n,f_out,f_in", [(1, 4, 8), (65, 64, 64), (5000, 64, 72), (30000, 40, 250)])
def test_input_gradient_with_addend_mask_and_total(n, f_out, f_in, dtype):
    import paper_2106_05609_amd as gas
    gp, w, wide, y, t0 = (rng.normal_matrix(5, s, a, b, dtype=dtype).cuda()
                          for s, a, b in ((910, n, f_out), (911, f_in, f_out), (912, n, f_in + 5), (913, n, f_in), (914, n, f_in)))
    add = wide[:, :f_in]                                          # a strided addend
    want = torch.empty(n, f_in, dtype=dtype, device="cuda")
    gas.gas_linear_bwd_input(gp, w, want, c_weight=0.7)
    gas.gas_axpy(add, want, want, 1.0)
    gas.gas_relu_bwd(want, y, want)
    total = t0.clone()
    gas.gas_axpy(total, want, total, 0.1)
    got, total2 = torch.empty_like(want), t0.clone()
    gas.gas_linear_bwd_input_add(gp, w, got, c_weight=0.7, add=add, mask=y, total=total2, c_total=0.1)
    assert torch.equal(got, want) and torch.equal(total2, total)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_many_matrices_updated_in_shared_launches(dtype):
    import paper_2106_05609_amd as gas
    sizes = [(1, 1), (3, 5), (64, 64), (1433, 256), (0, 4)] + [(7, k) for k in range(1, 71)]
    ws = [rng.normal_matrix(5, 930 + k, *s, dtype=dtype).cuda() for k, s in enumerate(sizes)]
    ws += [ws[2], ws[3][100:200]]                                 # a matrix named twice, and a part of another
    dws = [rng.normal_matrix(5, 1030 + k, *w.shape).cuda() for k, w in enumerate(ws)]
    kept = [w.clone() for w in ws[:-2]]
    gas.gas_sgd_steps(list(zip(ws, dws)), 0.1, 0.01)
    got = [w.clone() for w in ws[:-2]]
    for w, k in zip(ws, kept):
        w.copy_(k)
    for w, dw in zip(ws, dws):
        gas.gas_sgd_step(w, dw, 0.1, 0.01)
    assert all(torch.equal(a, b) for a, b in zip(got, ws))


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("n,F", [(70, 64), (5000, 64), (25000, 72), (30000, 256)])
def test_input_gradient_with_identity_and_total(n, F, dtype):
    """GCNII's call: the identity term, no addend, no mask, and the initial residual's running total."""
    import paper_2106_05609_amd as gas
    gp, w, t0 = (rng.normal_matrix(5, s, a, F, dtype=dtype).cuda() for s, a in ((920, n), (921, F), (922, n + 9)))
    want, total = torch.empty_like(gp), t0.clone()
    gas.gas_linear_bwd_input(gp, w, want, c_identity=0.6, c_weight=0.4)
    gas.gas_axpy(total[:n], want, total[:n], 0.1)
    got, total2 = torch.empty_like(want), t0.clone()
    gas.gas_linear_bwd_input_add(gp, w, got, c_identity=0.6, c_weight=0.4, total=total2[:n], c_total=0.1)
    assert torch.equal(got, want) and torch.equal(total2, total)


@pytest.mark.parametrize("n,f_out,f_in", [(65, 64, 64), (5000, 64, 72), (30000, 40, 250)])
def test_input_gradient_in_place_of_the_addend(n, f_out, f_in):
    import paper_2106_05609_amd as gas
    gp, w, add, y = (rng.normal_matrix(5, s, a, b).cuda() for s, a, b in ((923, n, f_out), (924, f_in, f_out), (925, n, f_in), (926, n, f_in)))
    want = torch.empty_like(add)
    gas.gas_linear_bwd_input_add(gp, w, want, c_weight=0.7, add=add, mask=y)
    gas.gas_linear_bwd_input_add(gp, w, add, c_weight=0.7, add=add, mask=y)
    assert torch.equal(add, want)
    t = torch.zeros(4, 8, dtype=torch.bfloat16, device="cuda")
    out = torch.zeros(4, 8, dtype=torch.bfloat16, device="cuda")
    with pytest.raises(gas.GasError):                              # bf16 rounds in between: no addend in place
        gas.gas_linear_bwd_input_add(t, torch.zeros(8, 8, dtype=torch.bfloat16, device="cuda"), out, add=out)
