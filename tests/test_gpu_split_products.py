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


def _operands(what, m, k, n):
    """(z, w, g) with the two factors of the product first, and how many terms a sum has."""
    z, w, g = (rng.normal_matrix(11, s, a, b) for s, a, b in ((720, m, k), (721, k, n), (722, m, n)))
    return {"linear": (z, w, k), "input": (g, w, n), "weight": (z, g, m)}[what]


def _check_every_element(what, a, b, terms, k, n):
    m = a.shape[0]
    if what == "linear":
        got, (a64, b64) = _call(what, a, b, torch.zeros(m, n)), (a.double(), b.double())
    elif what == "input":
        got, (a64, b64) = _call(what, torch.zeros(m, k), b, a), (a.double(), b.double().t())
    else:
        got, (a64, b64) = _call(what, a, torch.zeros(k, n), b), (a.double().t(), b.double())
    want, size = a64 @ b64, a64.abs() @ b64.abs()
    # each product within 2^-24 of itself, each addition within 2^-24 of a partial sum of at most `size`; below the normal
    # numbers a rounding is at most 2^-150
    bound = (terms + 8) * (2.0 ** -24 * size + 2.0 ** -149)
    assert bool(((got.double() - want).abs() <= bound).all()), float(((got.double() - want).abs() / bound).max())


@pytest.mark.parametrize("what", ["linear", "input", "weight"])
@pytest.mark.parametrize("up_a,up_b", [(-108, 0), (-112, 0), (-116, 0), (-124, 0), (-132, 0), (0, -120), (-116, -10), (-140, 60), (-126, 100), (-64, -64)])
@pytest.mark.parametrize("m,k,n", [(70, 20, 72), (24577, 136, 256)])
def test_operands_near_the_bottom_of_the_range(what, up_a, up_b, m, k, n):
    a, b, terms = _operands(what, m, k, n)
    _check_every_element(what, (a.double() * 2.0 ** up_a).float(), (b.double() * 2.0 ** up_b).float(), terms, k, n)


@pytest.mark.parametrize("what", ["linear", "input", "weight"])
@pytest.mark.parametrize("large", [1.0, 2.0 ** 60, 2.0 ** 100])
def test_small_values_beside_others(what, large):
    """A row and single elements below 2^-110 among ordinary ones, and beside values that leave the range when scaled up."""
    m, k, n = 300, 96, 130
    a, b, terms = _operands(what, m, k, n)
    a[5] *= 2.0 ** -118
    a[::7, 3] = 2.0 ** -130
    b[3] = 0.0
    b[3, ::2] = 2.0 ** 20 / 3.0
    a[11, 2] = large
    _check_every_element(what, a, b, terms, k, n)


@pytest.mark.parametrize("what,t", [("linear", 100), ("linear", 4096), ("weight", 100), ("weight", 4096), ("weight", 100000)])
def test_one_signed_sums(what, t):
    """Sums that only grow, as products of ReLU activations: a rounding that leaned to one side would add up here.  Bound: a
    quarter of what t roundings of one direction would come to at most, and for slabs the fp32 figure (sqrt) as above."""
    m, k, n = (500, t, 64) if what == "linear" else (t, 64, 48)
    z, w, g = (rng.normal_matrix(11, s, a, b).abs() for s, a, b in ((730, m, k), (731, k, n), (732, m, n)))
    got, want = _call(what, z, w, g).double(), _product(what, z.double(), w.double(), g.double())
    err = (got - want) / want
    assert float(err.norm() / np.sqrt(err.numel())) <= (1.0 + np.sqrt(min(t, 4096) / 3)) * 2.0 ** -24
    assert abs(float(err.mean())) <= 0.25 * (1.0 + np.sqrt(min(t, 4096) / 3)) * 2.0 ** -24


@pytest.mark.parametrize("what", ["linear", "input", "weight"])
@pytest.mark.parametrize("rows,cols", [(1, 1), (70, 65), (25000, 130)])
def test_sums_of_one_term_are_rounded_once(what, rows, cols):
    """One input feature, one output feature, one row: the result is the fp32 product."""
    a, b = rng.normal_matrix(11, 740, rows, 1), rng.normal_matrix(11, 741, 1, cols)
    if what == "linear":
        got = _call(what, a, b, torch.zeros(rows, cols))
    elif what == "input":
        got = _call(what, torch.zeros(rows, cols), b.t().contiguous(), a)
    else:
        rows = min(rows, 300)                              # the gradient is [rows, cols]
        a = a[:rows]
        got = _call(what, a.t().contiguous(), torch.zeros(rows, cols), b)
    assert torch.equal(got, a * b)


# the borders of the rules that choose a tile: 16, 17, 64 and 65 input columns, 352 tiles of 128 x 128 (here 345 rows of tiles
# and more), one and several columns of tiles, ragged last tiles
@pytest.mark.parametrize("what", ["linear", "input"])
@pytest.mark.parametrize("m,k,n", [(300, 16, 130), (300, 17, 130), (50000, 5, 7), (44929, 64, 65), (44929, 65, 65), (45057, 65, 65),
                                   (24577, 65, 64), (24449, 65, 47), (262145, 64, 70)])
def test_borders_of_the_tile_rules(what, m, k, n):
    z, w = rng.normal_matrix(11, 750, m, k).cuda(), rng.normal_matrix(11, 751, k, n).cuda()
    import paper_2106_05609_amd as gas
    out = torch.full((m, n), float("nan"), device="cuda")
    if what == "linear":
        gas.gas_linear(z, w, out)
    else:
        gas.gas_linear_bwd_input(z, w.t().contiguous(), out)
    z64, w64 = z.double(), w.double()
    bound = (k + 8) * 2.0 ** -24 * (z64.abs() @ w64.abs())
    assert bool(((out.double() - z64 @ w64).abs() <= bound).all())


def _every_option(m, k, n, z, w):
    """(name, result, oracle, bound) of the transform in each form that keeps its weights in place: bias and ReLU, push, rows with
    a stride, the input gradient, the input gradient with a mask."""
    import paper_2106_05609_amd as gas
    d = "cuda"
    bias, idx, mask = rng.normal_matrix(11, 762, 1, n)[0].to(d), torch.randperm(m, generator=torch.Generator().manual_seed(3)).int().to(d), rng.normal_matrix(11, 763, m, n).to(d)
    want, bound = z.double() @ w.double(), (k + 8) * (2.0 ** -24 * (z.double().abs() @ w.double().abs()) + 2.0 ** -149)
    new = lambda: torch.full((m, n), float("nan"), device=d)
    y = new()
    gas.gas_linear(z, w, y)
    yield "linear", y, want, bound
    y2, hist = new(), torch.full((m, n + 3), float("nan"), device=d)
    gas.gas_linear_push(z, w, y2, idx, hist[:, :n], relu=True)
    yield "push", y2, y.double().clamp(min=0), 0.0
    yield "history", hist[idx.long(), :n], y2.double(), 0.0
    assert bool(torch.isnan(hist[:, n:]).all())
    wide = torch.full((m, n + 5), float("nan"), device=d)
    strided = torch.zeros(m, k + 3, device=d)
    strided[:, 1:1 + k] = z
    gas.gas_linear(strided[:, 1:1 + k], w, wide[:, 2:2 + n], bias=bias, c_weight=0.5)
    yield "strided", wide[:, 2:2 + n], 0.5 * want + bias.double(), 0.5 * bound + 2.0 ** -23 * (0.5 * want.abs() + bias.double().abs())
    assert bool(torch.isnan(wide[:, :2]).all()) and bool(torch.isnan(wide[:, 2 + n:]).all())
    g = new()
    gas.gas_linear_bwd_input(z, w.t().contiguous(), g)
    yield "input", g, want, bound
    g2 = new()
    gas.gas_linear_bwd_input(z, w.t().contiguous(), g2, mask=mask)
    yield "masked", g2, torch.where(mask > 0, g, torch.zeros_like(g)).double(), 0.0


# weights kept in registers: every count of 32-wide steps, widths that are no whole number of fours or of 32 columns, a last row
# tile of one row and of all but one, rows on both sides of the rule (512 tiles of 128 x 128)
@pytest.mark.parametrize("m,k,n", [(32768, 256, 256), (32769, 65, 129), (32800, 97, 131), (33000, 128, 256), (32783, 131, 200),
                                   (32769, 190, 255), (40001, 223, 160), (33001, 254, 256), (33008, 256, 130), (98400, 96, 256),
                                   (60000, 160, 256), (65700, 160, 250), (57473, 128, 252), (49200, 96, 200)])
def test_weights_in_registers(m, k, n):
    z, w = rng.normal_matrix(11, 760, m, k).cuda(), rng.normal_matrix(11, 761, k, n).cuda()
    for name, got, want, bound in _every_option(m, k, n, z, w):
        assert bool(((got.double() - want).abs() <= bound).all()), name


@pytest.mark.parametrize("z_low,w_low,z_bad", [(True, False, None), (False, True, None), (True, True, None), (True, True, 3e38),
                                               (False, False, float("inf")), (True, False, float("nan"))])
def test_weights_in_registers_and_values_that_the_split_cannot_hold(z_low, w_low, z_bad):
    import paper_2106_05609_amd as gas
    m, k, n = 33001, 101, 140
    z, w = rng.normal_matrix(11, 764, m, k), rng.normal_matrix(11, 765, k, n)
    if z_low:
        z[::40] *= 2.0 ** -118                       # some tiles, none and several of their rows
        z[7, 3] = 2.0 ** -130
    if w_low:
        w[:, 5] *= 2.0 ** -116
    if z_bad is not None:
        z[m // 2, 3] = z_bad
        z[m - 1, k - 1] = -z_bad
    z, w = z.cuda(), w.cuda()
    want, size = z.double() @ w.double(), z.double().abs() @ w.double().abs()
    for trans in (False, True):
        y = torch.full((m, n), float("nan"), device="cuda")
        gas.gas_linear_bwd_input(z, w.t().contiguous(), y) if trans else gas.gas_linear(z, w, y)
        fine = size < 3.4e38                         # the rest: what fp32 arithmetic gives, infinite or not a number
        assert bool(((y.double() - want).abs() <= (k + 8) * (2.0 ** -24 * size + 2.0 ** -149))[fine].all())
        assert not bool(torch.isfinite(y)[~torch.isfinite(want)].any())


# few tiles, steps of 32 k dealt to four groups of wavefronts: fewer steps than groups, one group a step ahead, a last step that
# is not whole, and both sides of the rule (32 tiles of 64 x 64 on each of eight XCDs)
@pytest.mark.parametrize("what", ["linear", "input"])
@pytest.mark.parametrize("m,k,n", [(1, 65, 3), (70, 96, 65), (64, 128, 64), (100, 129, 70), (130, 161, 300), (500, 1024, 130), (77, 1433, 63),
                                   (4096, 70, 256), (4097, 70, 256),
                                   # six steps and more; 32 tiles on an XCD and 33 or 36
                                   (1, 161, 3), (70, 161, 65), (64, 192, 64), (100, 193, 70), (4096, 165, 256), (4097, 165, 256),
                                   (5376, 161, 66), (5632, 161, 130)])
def test_steps_in_groups(what, m, k, n):
    a, b, terms = _operands(what, m, k, n) if what == "linear" else _operands(what, m, n, k)
    _check_every_element(what, a, b, terms, *((k, n) if what == "linear" else (n, k)))
