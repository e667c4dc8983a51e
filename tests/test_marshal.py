"""csrc/marshal.cpp: addresses and sizes of every kind of tensor against the Python functions it stands in for, which tensors it
leaves to them, calls with arguments that don't fit, and a module that was built for something else."""
import ctypes as C
import os

import pytest
import torch

from paper_2106_05609_amd import _build, binding as B

L = B._calls()
from paper_2106_05609_amd import _marshal as M      # noqa: E402   (built for this torch, or the calls above warned)


class Sub(torch.Tensor):
    pass


def _outcome(fn, *args):
    try:
        return fn(*args)
    except Exception as e:
        return type(e)


base = torch.arange(60, dtype=torch.float32).view(6, 10)
OWN = {                                             # read by the module itself
    "matrix": base, "rows": base[1:4], "columns": base[:, 2:7], "steps": base[::2], "one row": base[2:3], "row of a slice": base[2:3, 1:4],
    "one column": base[:, 3:4], "no rows": base[:0], "no columns": base[:, :0], "bf16": base.bfloat16(), "one value": base[:1, :1],
    "parameter": torch.nn.Parameter(base.clone()), "grad": base.clone().requires_grad_(), "int32": base.int(), "vector": base[0].clone()}
LEFT = {                                            # left to Python
    "subclass": base.as_subclass(Sub), "meta": torch.empty(3, 4, device="meta"), "sparse": base.to_sparse(), "number": 3, "list": [1.0], "none": None}


@pytest.fixture
def slow(monkeypatch):
    """The Python functions as the module calls them, counted."""
    calls = []

    def counted(fn):
        return lambda *a: (calls.append(fn), fn(*a))[1]
    M.set_slow(*(counted(f) for f in (B._mat_any, B._size_any, B._ptr_any)))
    yield calls
    M.set_slow(B._mat_any, B._size_any, B._ptr_any)


@pytest.mark.parametrize("name", [*OWN, *LEFT])
def test_addresses_and_sizes(name, slow):
    t = {**OWN, **LEFT}[name]
    for fast, python in ((M.mat, B._mat_any), (M.size, B._size_any), (M.ptr, B._ptr_any)):
        assert _outcome(fast, t) == _outcome(python, t)
    for dtype in (None, torch.float32, torch.int32, torch.bfloat16):
        assert _outcome(M.ptr, t, dtype) == _outcome(B._ptr_any, t, dtype)
    if name in ("matrix", "rows", "bf16", "parameter", "grad", "one value", "no rows"):
        slow.clear()
        M.mat(t), M.size(t), M.ptr(t), M.ptr(t, t.dtype)
        assert not slow
    if name in LEFT and t is not None:
        slow.clear()
        for f in (M.mat, M.size, M.ptr):
            _outcome(f, t)
        assert slow == [B._mat_any, B._size_any, B._ptr_any]


@pytest.mark.parametrize("t", [base.t(), base[:, ::2], base.view(3, 4, 5), base.t()[:1]])
def test_rows_that_are_not_contiguous_are_refused(t):
    for fast, python in ((M.mat, B._mat_any), (M.size, B._size_any), (M.ptr, B._ptr_any)):
        assert _outcome(fast, t) == _outcome(python, t)
    if t.dim() != 2 or t.shape[1] > 1 and t.stride(1) != 1:
        with pytest.raises(ValueError):
            M.mat(t)


def test_under_a_transform():
    seen = []

    def f(x):
        seen.append((_outcome(M.mat, x), _outcome(B._mat_any, x)))
        return x
    torch.func.vmap(f)(base.view(2, 3, 10))
    torch.func.grad(lambda x: f(x).sum())(base)
    assert all(a == b for a, b in seen) and len(seen) == 2


PUSH = (None, 4, None, 0, 0, 4, 0, None, 10, 4, None)        # no rows: nothing is read


def test_arguments():
    assert M.gas_push(*PUSH) == 0
    for n in (0, len(PUSH) - 1, len(PUSH) + 1):
        with pytest.raises(TypeError, match=f"{n} arguments, the call takes {len(PUSH)}"):
            M.gas_push(*(PUSH + (0,))[:n])
    with pytest.raises(OverflowError):
        M.gas_push(*PUSH[:5], 2 ** 31, *PUSH[6:])            # F is 32 bits wide
    with pytest.raises(OverflowError):
        M.gas_push(*PUSH[:4], 2 ** 63, *PUSH[5:])
    with pytest.raises(OverflowError):
        M.gas_push(-1, *PUSH[1:])
    for bad in (0.5, "x", torch.float64):
        with pytest.raises(TypeError):
            M.gas_push(*PUSH[:5], bad, *PUSH[6:])
    with pytest.raises(TypeError):
        M.gas_push(0.5, *PUSH[1:])
    room = (C.c_int64 * 4)()
    for address in (C.addressof(room), room, C.c_void_p(C.addressof(room)), 2 ** 64 - 16):
        assert M.gas_push(address, *PUSH[1:]) == 0
    assert M.gas_pna_groups_workspace(100, 7) == L.gas_pna_groups_workspace(100, 7) > 0


def test_every_call_takes_what_its_signature_says():
    for name, sig in B._SIGNATURES.items():
        if hasattr(M, name):
            with pytest.raises(TypeError, match=f"the call takes {len(sig)}"):
                getattr(M, name)(*[0] * (len(sig) + 1))


def _reset(monkeypatch):
    monkeypatch.setattr(B, "_stream", lambda: 0)
    for name in ("_typed", "_mat", "_size", "_ptr"):
        monkeypatch.setattr(B, name, getattr(B, name))
    B._typed = None


def test_a_module_built_for_another_torch_is_not_used(monkeypatch):
    _reset(monkeypatch)
    monkeypatch.setattr(_build, "built_for", lambda: "torch 0.0")
    with pytest.warns(RuntimeWarning, match="_marshal.so was built for torch .* this is torch 0.0.*|build again"):
        calls = B._calls()
    assert calls.gas_push is not M.gas_push and calls.gas_push(*PUSH) == 0
    assert (B._mat, B._size, B._ptr) == (B._mat_any, B._size_any, B._ptr_any)
    z = torch.empty(0, 4)
    B.gas_pull(torch.empty(3, 4), None, z, n=0)
    wide = torch.empty(3, 4, dtype=torch.float64)
    with pytest.raises(TypeError):
        B.gas_pull(wide, None, wide, n=0)


def test_a_module_that_does_not_load_is_not_needed(monkeypatch):
    import sys
    import paper_2106_05609_amd as package
    _reset(monkeypatch)
    monkeypatch.setitem(sys.modules, "paper_2106_05609_amd._marshal", None)      # its import fails
    monkeypatch.delattr(package, "_marshal", raising=False)
    with pytest.warns(RuntimeWarning, match="_build"):
        calls = B._calls()
    assert calls.gas_push(*PUSH) == 0


def test_what_the_module_was_built_for_makes_it_stale(monkeypatch):
    assert M.built_for == _build.built_for()
    monkeypatch.setattr(os.path, "getmtime", lambda f: 0)                        # whatever the sources' times are
    assert not _build._marshal_stale()
    monkeypatch.setattr(_build, "built_for", lambda: "torch 0.0")
    assert _build._marshal_stale()
