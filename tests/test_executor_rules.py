"""Which form of a call the executor and the binding take."""
import pytest
import torch

from paper_2106_05609_amd import executor


@pytest.mark.parametrize("dtype,rows,f_in,hidden,f_out,in_two", [
    (torch.float32, 2000, 32, 32, 32, False), (torch.float32, 8192, 64, 32, 7, False), (torch.float32, 20, 8, 64, 32, False),
    (torch.float32, 8193, 32, 32, 32, True), (torch.float32, 100, 33, 64, 32, True), (torch.float32, 100, 32, 32, 33, True),
    (torch.float32, 4000, 256, 256, 256, True), (torch.float32, 500, 64, 64, 64, True), (torch.float32, 500, 1433, 32, 7, True),
    # measured: the fused bf16 kernels were the faster ones at a hundred rows of odd widths
    (torch.bfloat16, 100, 250, 250, 250, False), (torch.bfloat16, 5000, 256, 256, 47, False), (torch.bfloat16, 5000, 256, 256, 256, False)])
def test_form_of_the_mlp(dtype, rows, f_in, hidden, f_out, in_two):
    shape = lambda *s: torch.empty(*s, dtype=dtype, device="meta")
    assert executor._mlp_in_two(shape(rows, f_in), shape(f_in, hidden), shape(hidden, f_out)) is in_two


@pytest.mark.parametrize("width,rows,entries,longest,one", [
    (64, 21248, 300_000, 40, True), (32, 512, 7_000, 48, True), (64, 5000, 500_000, 200, True), (64, 8192, 20_000, 512, True),
    (60, 60_000, 140_000, 500, True), (32, 21_248, 2_000_000, 200, True), (128, 5000, 50_000, 20, True), (128, 4096, 90_000, 64, True),
    (80, 21_248, 300_000, 30, True),
    # measured: two launches were the faster form
    (32, 512, 25_000, 100, False), (48, 8000, 60_000, 500, False), (64, 60_000, 450_000, 500, False), (16, 21_248, 157_000, 500, False),
    (128, 10_000, 100_000, 20, False), (96, 5000, 150_000, 60, False), (68, 21_248, 500_000, 40, False), (128, 512, 20_000, 65, False), (64, 500, 10_000, 513, False)])
def test_form_of_the_backward_layer(width, rows, entries, longest, one):
    assert executor._back_in_one_launch(width, rows, entries, longest) is one


@pytest.mark.parametrize("missing", ["_raw_stream", "_device"])
def test_stream_without_torchs_private_functions(missing, monkeypatch):
    from paper_2106_05609_amd import binding

    class Stream:
        cuda_stream = 1234

    monkeypatch.setattr(binding, missing, None)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: Stream)
    assert binding._stream() == 1234


@pytest.mark.parametrize("together", [True, False])
def test_shared_workspace_of_the_weight_gradients_is_bounded(together, monkeypatch):
    """A pass's gradients, and a list given at once, go in parts whose workspace stays below the bound, or one by one; each
    of them once and in order."""
    from paper_2106_05609_amd import binding
    real, calls = binding._calls(), []

    class Recorded:
        gas_linear_bwd_weights_workspace = real.gas_linear_bwd_weights_workspace

        def gas_linear_bwd_weights(self, count, *args):
            calls.append((count, args[-2], list(args[9])))
            return 0
    monkeypatch.setattr(binding, "_calls", lambda: Recorded())
    monkeypatch.setattr(binding, "_stream", lambda: 0)
    shapes = [(16000, 1433, 256), (16000, 256, 256), (16000, 256, 47)] + [(21248, 64, 64)] * 40 + [(16000, 1433, 256)] * 4 + [(16000, 3000, 256)]
    items = [(torch.empty(m, k), torch.empty(m, n), torch.empty(k, n), 1.0) for m, k, n in shapes]
    if together:
        binding.gas_linear_bwd_weights(items)
    else:
        wg = executor._WeightGrads()
        for z, g, dw, c in items:
            assert wg.add(z, g, dw, c) is dw
        wg.done()
    assert all(need <= 128 << 20 or count == 1 for count, need, _ in calls)
    assert [p for _, _, dws in calls for p in dws] == [dw.data_ptr() for _, _, dw, _ in items]
    assert max(count for count, _, _ in calls) >= 6


@pytest.mark.parametrize("rows,longest,f,f1,out,dtype,grouped", [
    (50_000, 26, 256, 64, 256, torch.float32, True), (50_000, 41, 128, 32, 128, torch.float32, True),
    (50_000, 26, 100, 16, 64, torch.float32, False), (16_000, 24, 256, 64, 256, torch.float32, False),
    (50_000, 64, 256, 64, 256, torch.float32, False), (50_000, 26, 256, 64, 256, torch.bfloat16, False)])
def test_which_pna_layers_go_by_degree(rows, longest, f, f1, out, dtype, grouped):
    class Batch:
        nb, max_row, groups = rows, longest, "groups"
    got = executor._by_degree(Batch, torch.empty(0, f, dtype=dtype), torch.empty(f + 9 * f1, out))
    assert (got == "groups") == grouped


@pytest.mark.parametrize("rows,longest,out,second", [
    (30_500, 25, 256, False), (31_500, 25, 256, True), (32_500, 39, 208, True), (33_000, 26, 256, False), (50_000, 26, 256, False),
    (63_000, 28, 128, False), (65_000, 27, 96, True), (66_000, 28, 128, False), (32_000, 26, 192, False)])
def test_pna_forward_products_by_degree_take_no_round_more(rows, longest, out, second):
    """256 compute units hold 512 tiles of 128 x 128 at once: a product of at most that many goes by degree only if its degrees'
    tiles are no more either.  Gradients go by degree all the same."""
    class Batch:
        nb, max_row, groups = rows, longest, "groups"
    w2 = torch.empty(out + 9 * (out // 4), out)
    wide = executor._by_degree(Batch, torch.empty(0, out), w2)
    assert executor._groups_of_layers(Batch, torch.empty(0, out), [(None, w2)]) == [(wide, None if second else wide)]
