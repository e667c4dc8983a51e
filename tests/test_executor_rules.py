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


@pytest.mark.parametrize("missing", ["_raw_stream", "_device"])
def test_stream_without_torchs_private_functions(missing, monkeypatch):
    from paper_2106_05609_amd import binding

    class Stream:
        cuda_stream = 1234

    monkeypatch.setattr(binding, missing, None)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: Stream)
    assert binding._stream() == 1234


def test_shared_workspace_of_the_weight_gradients_is_bounded(monkeypatch):
    """Gradients that wait are flushed before their common workspace would pass the bound, after TOGETHER of them, and
    at the end; one that alone needs more goes alone."""
    from paper_2106_05609_amd import binding
    calls = []
    monkeypatch.setattr(binding, "gas_linear_bwd_weights", lambda items: calls.append(list(items)) if items else None)
    wg = executor._WeightGrads()
    shapes = [(16000, 1433, 256), (16000, 256, 256), (16000, 256, 47)] + [(21248, 64, 64)] * 40 + [(16000, 1433, 256)] * 4 + [(16000, 3000, 256)]
    outs = []
    for m, k, n in shapes:
        outs.append(wg.add(torch.empty(m, k, device="meta"), torch.empty(m, n, device="meta")))
    wg.done()
    need = lambda z, g: binding.gas_linear_bwd_weight_workspace(z.shape[0], z.shape[1], g.shape[1])
    for items in calls:
        assert len(items) <= wg.TOGETHER
        assert len(items) == 1 or sum(need(z, g) for z, g, _, _ in items) <= 128 << 20
    done = [dw for items in calls for _, _, dw, _ in items]
    assert len(done) == len(outs) and all(a is b for a, b in zip(done, outs))           # each once, in order
    assert max(len(items) for items in calls) == wg.TOGETHER
