"""fp32 products of few rows, whose steps eight groups of wavefronts share: edges of its tiles (32 x 64), steps and groups, the last
size that takes it and the first that does not, and operands that the split into bf16 parts cannot represent."""
import numpy as np
import pytest
import torch

from gas_inputs import rng
from tests.test_gpu_split_products import _call, _product

pytestmark = pytest.mark.gpu

# reduced widths on both sides of the first that takes it (97) and of a round of eight steps (256)
SHAPES = [(1, 97, 97), (31, 96, 127), (32, 97, 129), (33, 255, 256), (255, 257, 193), (257, 2240, 224), (2048, 130, 256), (2049, 130, 256)]


@pytest.mark.parametrize("what", ["linear", "input"])
@pytest.mark.parametrize("m,k,n", SHAPES)
def test_tile_edges_and_error(what, m, k, n):
    z, w, g = (rng.normal_matrix(12, s, a, b) for s, a, b in ((700, m, k), (701, k, n), (702, m, n)))
    got, want = _call(what, z, w, g).double(), _product(what, z.double(), w.double(), g.double())
    size = _product(what, z.abs().double(), w.abs().double(), g.abs().double())
    t = k if what == "linear" else n
    # six products a step of 16, each rounding a sum of at most `size`, and eight groups' sums
    assert bool(((got - want).abs() <= (6 * np.ceil(t / 16) + 8) * 2.0 ** -24 * size).all())
    assert float((got - want).norm() / want.norm()) <= 1.5 * (1.0 + np.sqrt(t / 3)) * 2.0 ** -24      # an fp32 sum in order


@pytest.mark.parametrize("what", ["linear", "input"])
@pytest.mark.parametrize("bad", [float("inf"), float("nan"), 3.4e38, 1e-41])
def test_operands_that_bf16_parts_cannot_hold(what, bad):
    m, k, n = 70, 300, 130
    z, w, g = (rng.normal_matrix(12, s, a, b) for s, a, b in ((710, m, k), (711, k, n), (712, m, n)))
    w[3, :] = w[3, :].abs() + 0.5
    z[m // 2, 3], g[m // 3, 2], w[299, 129] = bad, bad, 0.0
    got, want = _call(what, z, w, g), _product(what, z, w, g)
    for same in (torch.isnan, torch.isposinf, torch.isneginf):
        assert torch.equal(same(got), same(want))
    fine = torch.isfinite(want)
    scale = _product(what, z.abs().double(), w.abs().double(), g.abs().double())[fine]
    t = k if what == "linear" else n
    assert bool(((got.double()[fine] - want.double()[fine]).abs() <= 2 * t * 2.0 ** -24 * scale).all())
