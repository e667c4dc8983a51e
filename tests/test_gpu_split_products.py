"""fp32 products on the bf16 matrix instructions (gas_linear, gas_linear_bwd_input, gas_linear_bwd_weight): the edges of
the tiles against products in 64 bits, the error against that of fp32 arithmetic, and operands that the split into
bf16 parts cannot represent against fp32 arithmetic on the CPU."""
import numpy as np
import pytest
import torch

from gas_inputs import rng

pytestmark = pytest.mark.gpu


def _call(what, z, w, g):
    import paper_2106_05609_amd as gas
    z, w, g = (t.to("cuda") for t in (z, w, g))
    (m, k), n = z.shape, w.shape[1]
    if what == "linear":
        out = torch.full((m, n), float("nan"), device="cuda")
        gas.gas_linear(z, w, out)
    elif what == "input":
        out = torch.full((m, k), float("nan"), device="cuda")
        gas.gas_linear_bwd_input(g, w, out)
    else:
        out = torch.full((k, n), float("nan"), device="cuda")
        ws = torch.empty(max(1, gas.gas_linear_bwd_weight_workspace(m, k, n)), dtype=torch.uint8, device="cuda")
        gas.gas_linear_bwd_weight(z, g, out, ws)
    torch.cuda.synchronize()
    return out.cpu()


def _product(what, z, w, g):
    return z @ w if what == "linear" else (g @ w.t() if what == "input" else z.t() @ g)


# rows and widths on both sides of the 64-, 128- and 256-wide tiles and of the steps of 16 and 32
SHAPES = [(1, 1, 1), (63, 15, 17), (65, 33, 64), (129, 47, 65), (3000, 257, 129), (24449, 16, 256), (24577, 100, 257),
          (49025, 31, 250), (49153, 256, 130)]


@pytest.mark.parametrize("what", ["linear", "input", "weight"])
@pytest.mark.parametrize("m,k,n", SHAPES)
def test_tile_edges_and_error(what, m, k, n):
    z, w, g = (rng.normal_matrix(11, s, a, b) for s, a, b in ((700, m, k), (701, k, n), (702, m, n)))
    got = _call(what, z, w, g).double()
    want = _product(what, z.double(), w.double(), g.double())
    # an output is a sum of t products of N(0,1) factors; each of the t / 16 steps rounds an accumulator six times by
    # at most 2^-24 of its largest value, about 6 sqrt(t) over all columns
    t = {"linear": k, "input": n, "weight": m}[what]
    bound = 6.0 * np.ceil(t / 16) * 2.0 ** -24 * 6.0 * np.sqrt(t) + 2.0 ** -23 * 6.0 * np.sqrt(t)
    assert float((got - want).abs().max()) <= bound
    # in the 2-norm the errors add as independent roundings: an fp32 sum of t terms in order has sqrt(t / 3) * 2^-24
    # and more, relative; half as much again leaves room for the few outputs of the smallest shapes
    assert float((got - want).norm() / want.norm()) <= 1.5 * (1.0 + np.sqrt(t / 3)) * 2.0 ** -24


@pytest.mark.parametrize("what", ["linear", "input", "weight"])
@pytest.mark.parametrize("bad", [float("inf"), float("-inf"), float("nan"), 3.4e38, 1e-41])
@pytest.mark.parametrize("m,k,n", [(200, 40, 72), (24577, 136, 256)])
def test_operands_that_bf16_parts_cannot_hold(what, bad, m, k, n):
    z, w, g = (rng.normal_matrix(11, s, a, b) for s, a, b in ((710, m, k), (711, k, n), (712, m, n)))
    w[3, :] = w[3, :].abs() + 0.5                     # inf times them is inf, 3.4e38 times them may overflow
    z[m // 2, 3], g[m // 3, 2] = bad, bad
    z[m - 1, k - 1], w[5, 1] = -bad, 0.0
    got, want = _call(what, z, w, g), _product(what, z, w, g)
    assert torch.equal(torch.isnan(got), torch.isnan(want))
    assert torch.equal(torch.isposinf(got), torch.isposinf(want))
    assert torch.equal(torch.isneginf(got), torch.isneginf(want))
    fine = torch.isfinite(want)
    scale = _product(what, z.abs().double(), w.abs().double(), g.abs().double())[fine]
    t = {"linear": k, "input": n, "weight": m}[what]
    assert bool(((got.double()[fine] - want.double()[fine]).abs() <= 2 * t * 2.0 ** -24 * scale).all())
