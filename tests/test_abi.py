"""The C-ABI library loads and exports every symbol include/gas.h declares
(no compute calls: this runs without a GPU)."""
import ctypes
import os
import re

import pytest
import torch

from paper_2106_05609_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    text = open(os.path.join(ROOT, "include", "gas.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"GAS_API\s+[\w\s\*]+?\b(gas_\w+)\s*\(", text)))


def test_header_symbols_are_exported():
    names = _declared()
    assert len(names) >= 12 and "gas_pull" in names and "gas_spmm_t" in names
    lib = ctypes.CDLL(binding.LIB_PATH)
    for n in names:
        assert hasattr(lib, n), f"{n} is declared in gas.h but not exported"
    assert sorted(binding.EXPORTS) == names


def test_version_and_error_string_without_a_gpu():
    assert binding.gas_version() >= 100
    assert isinstance(binding.lib().gas_last_error(), bytes)


def test_argument_errors_are_reported_before_any_launch():
    L = binding.lib()
    st = L.gas_pull(None, ctypes.c_int64(10), ctypes.c_int64(4), None, ctypes.c_int64(0), ctypes.c_int64(3),
                    ctypes.c_int32(4), ctypes.c_int(0), None, ctypes.c_int64(4), None)
    assert st == -1 and b"null" in L.gas_last_error()
    st = L.gas_pull(None, ctypes.c_int64(10), ctypes.c_int64(4), None, ctypes.c_int64(0), ctypes.c_int64(3),
                    ctypes.c_int32(4), ctypes.c_int(7), None, ctypes.c_int64(4), None)
    assert st == -2
    # n == 0 is a no-op even with null pointers
    st = L.gas_push(None, ctypes.c_int64(4), None, ctypes.c_int64(0), ctypes.c_int64(0), ctypes.c_int32(4),
                    ctypes.c_int(0), None, ctypes.c_int64(10), ctypes.c_int64(4), None)
    assert st == 0
    one = ctypes.c_void_p(16)
    st = L.gas_linear(one, ctypes.c_int64(8), ctypes.c_int64(5), ctypes.c_int32(8), one, ctypes.c_int32(4), None,
                      ctypes.c_int(0), ctypes.c_float(0.5), ctypes.c_float(0.5), ctypes.c_int(0), ctypes.c_void_p(32),
                      ctypes.c_int64(4), None)
    assert st == -1 and b"identity" in L.gas_last_error()


def _signatures():
    text = open(os.path.join(ROOT, "include", "gas.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    sigs = {}
    for m in re.finditer(r"GAS_API\s+gas_status\s+(gas_\w+)\s*\(([^;]*?)\)\s*;", text, flags=re.S):
        params = [re.sub(r"\s+", " ", p).strip() for p in m.group(2).split(",")]
        sigs[m.group(1)] = params
    return sigs


def _args(params, pointer, dtype, size):
    """ctypes arguments for a parameter list: every pointer = `pointer`, every dtype = `dtype`, the first
    int64 count = `size`, other integers 4, floats 1."""
    out, first = [], True
    for p in params:
        name = p.split()[-1].lstrip("*")
        if "*" in p:
            out.append(None if pointer is None else ctypes.c_void_p(pointer))
        elif p.startswith("gas_dtype"):
            out.append(ctypes.c_int(dtype))
        elif p.startswith("float"):
            out.append(ctypes.c_float(1.0))
        elif p.startswith("int64_t"):
            counts = name in ("n", "n_rows", "nnz")
            out.append(ctypes.c_int64(size if counts and first else 4))
            first = first and not counts
        elif p.startswith("int32_t"):
            out.append(ctypes.c_int32(4))
        elif p.startswith("int "):
            out.append(ctypes.c_int(0))
        else:
            raise AssertionError(f"unhandled parameter {p!r}")
    return out


def test_every_entry_point_rejects_bad_arguments_without_launching():
    """Null pointers, an unknown dtype and a negative count: each call returns an error status and leaves a
    message; nothing is launched (there is no GPU here), nothing crashes."""
    L = binding.lib()
    sigs = _signatures()
    assert len(sigs) >= 25
    for name, params in sigs.items():
        fn = getattr(L, name)
        fn.restype = ctypes.c_int
        st = fn(*_args(params, None, 0, 4))
        if name == "gas_disk_close":      # like free(): closing no table is allowed
            assert st == 0
            continue
        assert st < 0, f"{name} accepted null pointers"
        assert len(L.gas_last_error()) > 0, name
        takes_object = any("gas_plan" in p or "gas_disk_table*" in p.replace(" *", "*") for p in params)
        if takes_object:
            continue                      # a non-null dummy plan or table would be dereferenced
        if any(p.startswith("gas_dtype") for p in params):
            st = fn(*_args(params, 4096, 7, 4))
            assert st < 0, f"{name} accepted dtype 7"
        if any(p.split()[-1] in ("n", "n_rows", "nnz") for p in params if p.startswith("int64_t")):
            st = fn(*_args(params, 4096, 0, -1))
            assert st < 0, f"{name} accepted a negative count"


def test_a_zero_count_is_a_no_op():
    """n = 0 (an empty batch, an empty halo) succeeds without touching any pointer; the weight gradient and the
    squared norm are the exceptions, since an empty sum still has to be written (a zero matrix, a zero), and so are
    the backward aggregations, whose output rows (n_out of them) exist without any row of the pattern."""
    L = binding.lib()
    for name, params in _signatures().items():
        if any("gas_plan" in p or "gas_disk_table" in p for p in params):
            continue
        if not any(p.split()[-1] in ("n", "n_rows", "nnz") for p in params if p.startswith("int64_t")):
            continue
        fn = getattr(L, name)
        fn.restype = ctypes.c_int
        st = fn(*_args(params, None, 0, 0))
        assert st == (-1 if name in ("gas_linear_bwd_weight", "gas_linear_bwd_weight_static", "gas_sq_norm",
                                  "gas_pna_aggregate_bwd", "gas_gat_aggregate_bwd") else 0), name


def test_a_refused_input_gradient_has_launched_nothing():
    """bf16 takes its steps in several launches: a mask whose rows are too narrow is refused before the first (without a GPU a
    launch would be a HIP error)."""
    L = binding.lib()
    L.gas_linear_bwd_input_add.restype = ctypes.c_int
    p, q, i, f = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int32, ctypes.c_float
    a = [p(4096 * k) for k in range(1, 7)]                   # never dereferenced on the host
    st = L.gas_linear_bwd_input_add(a[0], q(8), q(4), i(8), a[1], i(8), ctypes.c_int(1), f(0.0), f(1.0), a[2], q(8), a[3], q(3),
                                    f(0.0), a[4], q(8), a[5], q(8), p(0))
    assert st == -1 and b"row stride" in L.gas_last_error()


def test_workspace_of_weight_gradients_by_degree_is_bounded():
    """Partials of about 128 slabs and one more for a degree, of slabs of up to 4,096 rows: no more than the plain gradient of the
    nine blocks takes where there are many rows."""
    L = binding.lib()
    for f, f1, f_out in ((256, 64, 256), (1433, 64, 256)):
        for n in (1, 50_000, 65_537, 200_000, 1_000_000, 10_000_000):
            got = L.gas_pna_linear_bwd_weight_workspace(ctypes.c_int64(n), 63, f, f1, f_out)
            assert 0 < got <= 4 * (f + 3 * f1) * f_out * (max(128, n // 4096) + 64)
            if n >= 1_000_000:
                assert got <= 1.4 * L.gas_linear_bwd_weight_workspace(ctypes.c_int64(n), f + 9 * f1, f_out)


def test_pna_blocks_are_nine_unless_three_are_asked_for():
    """A matrix of three blocks does not pass for one of nine."""
    ptr, col, x, three = torch.tensor([0, 1], dtype=torch.int32), torch.zeros(1, dtype=torch.int32), torch.zeros(1, 8), torch.zeros(1, 24)
    with pytest.raises(ValueError, match="do not match"):
        binding.gas_pna_aggregate(ptr, col, x, three, 1.0)
    with pytest.raises(ValueError, match="do not match"):
        binding.gas_pna_aggregate_bwd(ptr, col, ptr, col, col, x, three, torch.zeros(1, 8), 1.0)
    with pytest.raises(ValueError, match="do not match"):
        binding.gas_pna_aggregate(ptr, col, x, torch.zeros(1, 72), 1.0, blocks=3)


def test_refused_layers_name_the_call():
    L = binding.lib()
    i64, f32, p = ctypes.c_int64, ctypes.c_float, ctypes.c_void_p
    at = p(1 << 20)                            # never read: the calls are refused
    one, ld, half = (p * 1)(1 << 20), (i64 * 1)(64), (f32 * 1)(0.5)
    for dt, said in ((1, b"fp32 only"), (7, b"unknown dtype")):
        st = L.gas_spmm_linear_layers(1, at, at, at, at, i64(4), at, i64(64), one, i64(4), ld, dt, 64, f32(1), None, i64(0), f32(0), one, half,
                                      half, 1, one, i64(64), None, i64(0), None, None, i64(0), None, None)
        assert st == -2 and L.gas_last_error().startswith(b"gas_spmm_linear_layers: " + said)
    st = L.gas_spmm_linear_layers(1, at, at, at, at, i64(4), at, i64(64), one, i64(4), ld, 0, 66, f32(1), None, i64(0), f32(0), one, half,
                                  half, 1, one, i64(66), None, i64(0), None, None, i64(0), None, None)
    assert st == -1 and L.gas_last_error().startswith(b"gas_spmm_linear_layers: widths")


def test_products_by_degree_of_more_tiles_than_a_launch_holds():
    """Refused before anything is launched."""
    L = binding.lib()
    i64, f32, p = ctypes.c_int64, ctypes.c_float, ctypes.c_void_p
    at, other = p(1 << 20), p(1 << 21)
    n, big = i64((1 << 30) - 1), i64(1 << 50)
    other = p(1 << 21)
    calls = {
        "gas_pna_linear": (at, n, 3, at, i64(1024), 256, 64, at, 1024, f32(1), 0, other, i64(1024), None, None, i64(0), at, big, None),
        "gas_pna_linear_bwd_input": (at, n, 3, at, i64(256), 1024, 256, at, 256, f32(1), other, i64(2048), at, big, None),
        "gas_pna_linear_bwd_weight": (at, n, 3, at, i64(9000), at, i64(4096), 4096, 1024, 4096, f32(1), other, at, big, None)}
    for name, args in calls.items():
        assert getattr(L, name)(*args) == -1
        assert L.gas_last_error() == name.encode() + b": too many rows for one launch", name
