"""Thin binding of libgas.so: same names as the C ABI (include/gas.h),
argument marshalling only.  Tensors are torch tensors on the GPU; every step
runs in the library's kernels on torch's current stream.  The calls of a pass go
through csrc/marshal.cpp, the others through ctypes."""
import ctypes as C
import os
import warnings

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libgas.so")

F32, BF16 = 0, 1
OK = 0

EXPORTS = [
    "gas_last_error", "gas_version", "gas_validate_indices",
    "gas_pull", "gas_push", "gas_host_table_pointer", "gas_pull_host", "gas_push_host",
    "gas_gcn_norm", "gas_plan_create", "gas_plan_create_opt", "gas_plan_destroy", "gas_plan_describe", "gas_plan_copy_lists", "gas_spmm", "gas_spmm_hist", "gas_spmm_table", "gas_fuse_sources", "gas_spmm_t", "gas_spmm_t_relu",
    "gas_linear", "gas_mlp2", "gas_linear_push", "gas_mlp2_push", "gas_mlp2_keep", "gas_spmm_linear", "gas_spmm_t_relu_linear",
    "gas_spmm_linear_layers", "gas_spmm_t_relu_linear_layers",
    "gas_relu_bwd", "gas_linear_bwd_input", "gas_linear_bwd_input_add", "gas_linear_bwd_weight", "gas_linear_bwd_weight_workspace",
    "gas_linear_bwd_weight_static", "gas_linear_bwd_weights", "gas_linear_bwd_weights_workspace",
    "gas_softmax_xent", "gas_sgd_step", "gas_sgd_steps", "gas_sq_norm", "gas_sgd_step_clipped", "gas_axpy", "gas_row_distance", "gas_row_distance_bwd", "gas_row_dot",
    "gas_pna_aggregate", "gas_pna_aggregate_blocks", "gas_pna_aggregate_bwd_blocks", "gas_pna_groups", "gas_pna_groups_workspace",
    "gas_pna_linear", "gas_pna_linear_workspace", "gas_pna_linear_bwd_input", "gas_pna_linear_bwd_weight",
    "gas_pna_linear_bwd_weight_workspace", "gas_gat_aggregate", "gas_gat_aggregate_heads", "gas_pna_aggregate_bwd", "gas_gat_aggregate_bwd",
    "gas_gat_aggregate_bwd_heads", "gas_pna_aggregate_bwd_workspace", "gas_gat_aggregate_bwd_workspace",
    "gas_gat_aggregate_bwd_heads_workspace", "gas_linear_in_order", "gas_gat_aggregate_push", "gas_pna_aggregate_own", "gas_pna_aggregate_bwd_bounded",
    "gas_gat_aggregate_bwd_bounded",
    "gas_disk_open", "gas_disk_close", "gas_disk_pull", "gas_disk_push", "gas_disk_wait", "gas_disk_read_rows",
    "gas_disk_write_rows", "gas_disk_sync",
]

_lib = None


class GasError(RuntimeError):
    def __init__(self, status, message):
        super().__init__(f"gas status {status}: {message}")
        self.status = status


def lib():
    """Load libgas.so.  There is no fallback: without the HIP library nothing runs."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise ImportError(f"{LIB_PATH} is missing: build it with `python -m paper_2106_05609_amd._build` "
                              "(or __graft_entry__.build())")
        L = C.CDLL(LIB_PATH)
        L.gas_last_error.restype = C.c_char_p
        L.gas_version.restype = C.c_int
        L.gas_plan_destroy.restype = None
        L.gas_linear_bwd_weight_workspace.restype = C.c_int64
        L.gas_linear_bwd_weights_workspace.restype = C.c_int64
        for name in ("gas_pna_groups_workspace", "gas_pna_linear_workspace", "gas_pna_linear_bwd_weight_workspace"):
            getattr(L, name).restype = C.c_int64
        L.gas_pna_aggregate_bwd_workspace.restype = C.c_int64
        L.gas_gat_aggregate_bwd_workspace.restype = C.c_int64
        L.gas_gat_aggregate_bwd_heads_workspace.restype = C.c_int64
        for name in EXPORTS:
            if name not in ("gas_last_error", "gas_version", "gas_plan_destroy") and not name.endswith("_workspace"):
                getattr(L, name).restype = C.c_int
        _lib = L
    return _lib


# Argument types of the calls: p pointer, q int64, i int32 / enum, f float, in the order of include/gas.h.
_SIGNATURES = dict(
    gas_validate_indices="pqqp", gas_pull="pqqpqqiipqp", gas_push="pqpqqiipqqp", gas_host_table_pointer="pp",
    gas_pull_host="pqqpqqiipqp", gas_push_host="pqpqqiipqqp", gas_gcn_norm="ppqpppp", gas_plan_create_opt="ppqqippp",
    gas_plan_describe="pp", gas_plan_copy_lists="ppppp", gas_spmm="ppppfpqiifpqfpqip",
    gas_spmm_hist="ppppfpqpqqiifpqfpqip", gas_spmm_table="ppppfppqqiifpqip", gas_fuse_sources="pqqppp", gas_spmm_t="ppppffqpqiipqip",
    gas_spmm_t_relu="ppppffqpqiipqpqp", gas_linear_bwd_input_add="pqqipiiffpqpqfpqpqp", gas_sgd_steps="ippipffp",
    gas_linear="pqqipipiffipqp", gas_linear_in_order="pqqipiipqp", gas_mlp2="pqqipippipiipqp", gas_linear_push="pqqipipiffipqppqqp",
    gas_mlp2_push="pqqipippipiipqppqqp", gas_mlp2_keep="pqqipippipiipqpqppqqp",
    gas_spmm_linear="pppqpqpqqiiffpqfpipffipqpqppqqp", gas_relu_bwd="pqpqqiipqp", gas_linear_bwd_input="pqqipiiffpqpqp",
    gas_spmm_t_relu_linear="pppqpqiifpqpqpifffpqpqp",
    gas_spmm_linear_layers="ippppqpqpqpiifpqfpppipqpqppqpp", gas_spmm_t_relu_linear_layers="ipppqpqiifpqpqpppfpqpqp",
    gas_linear_bwd_weights_workspace="ipppi", gas_linear_bwd_weights="ipppppppipppqp",
    gas_linear_bwd_weight_workspace="qii", gas_linear_bwd_weight="pqpqqiiifppqp",
    gas_linear_bwd_weight_static="pqpqqiiifpp", gas_softmax_xent="pqqiipfpppqp", gas_sgd_step="pqipffp",
    gas_sq_norm="pqpp", gas_sgd_step_clipped="pqipffpifp", gas_pna_aggregate="ppqpqiipqfpqp", gas_pna_aggregate_blocks="ppqpqiipqfipqp",
    gas_pna_aggregate_bwd_blocks="pppqqpppqpqiifipqpqpqpqp", gas_pna_aggregate_bwd_bounded="pppqiqpppqpqiifipqpqpqpqp",
    gas_pna_aggregate_own="ppqipqiipqfipqpqipqp", gas_gat_aggregate_push="ppqipqiiippfipqppqqp",
    gas_gat_aggregate_bwd_bounded="pppqiipppqqqpqiiippfpqpqpppqp", gas_pna_groups="pqipp", gas_pna_groups_workspace="qi",
    gas_pna_linear="pqipqiipifipqppqpqp", gas_pna_linear_workspace="iiii", gas_pna_linear_bwd_input="pqipqiipifpqpqp",
    gas_pna_linear_bwd_weight="pqipqpqiiifppqp", gas_pna_linear_bwd_weight_workspace="qiiii",
    gas_gat_aggregate_heads="ppqpqiiippfipqp", gas_pna_aggregate_bwd_workspace="qqi",
    gas_pna_aggregate_bwd="pppqqpppqpqiifpqpqpqpqp", gas_gat_aggregate_bwd_heads_workspace="qqqii",
    gas_gat_aggregate_bwd_heads="pppqpppqqqpqiiippfpqpqpppqp", gas_axpy="pqpqqiifpqp", gas_row_distance="pqpqqiippp",
    gas_row_dot="pqpqqiippp", gas_row_distance_bwd="pqpqqiifpqp", gas_disk_open="pqiiiiqp", gas_disk_close="p",
    gas_disk_pull="ppqqpqpp", gas_disk_push="ppqqpqpp", gas_disk_wait="pq", gas_disk_read_rows="ppqqpq",
    gas_disk_write_rows="ppqqpq", gas_disk_sync="p",
)


def _marshalling():
    """The marshalling module; None, with a warning, if it can't be loaded or was built for another torch or interpreter."""
    from . import _build
    try:
        from . import _marshal
        if getattr(_marshal, "built_for", None) != _build.built_for():
            raise ImportError(f"_marshal.so was built for {getattr(_marshal, 'built_for', None)}, this is {_build.built_for()}")
        return _marshal
    except ImportError as e:
        warnings.warn("every call goes through ctypes, which takes 3 to 11 us longer: build again with "
                      f"`python -m paper_2106_05609_amd._build` ({e})", RuntimeWarning, stacklevel=2)
        return None


def _by_ctypes(fn):
    def call(*args):
        try:
            return fn(*args)
        except C.ArgumentError as e:                     # a type that no call takes
            raise TypeError(str(e)) from None
    return call


class _Calls:
    """The library's functions with their argument types declared: plain Python numbers are converted by ctypes itself, and those
    of a pass by the marshalling module (30 arguments: 0.4 us, ctypes 3).  A handle of its own: what lib() returns takes
    any ctypes objects, as before."""

    def __init__(self):
        global _mat, _size, _ptr
        lib()
        native = _marshalling()
        if native is None:
            _mat, _size, _ptr = _mat_any, _size_any, _ptr_any
        else:
            native.set_slow(_mat_any, _size_any, _ptr_any)
            _mat, _size, _ptr = native.mat, native.size, native.ptr
        raw = C.CDLL(LIB_PATH)
        types = dict(p=C.c_void_p, q=C.c_int64, i=C.c_int32, f=C.c_float)
        for name, sig in _SIGNATURES.items():
            fn = getattr(raw, name)
            fn.argtypes = [types[c] for c in sig]
            fn.restype = C.c_int64 if name.endswith("_workspace") else C.c_int
            setattr(self, name, _by_ctypes(fn) if native is None else getattr(native, name, fn))


_typed = None


def _calls():
    global _typed
    if _typed is None:
        _typed = _Calls()
    return _typed


def _check(st):
    if st != OK:
        raise GasError(st, lib().gas_last_error().decode())


def _dt(t: torch.Tensor) -> int:
    if t.dtype == torch.float32:
        return F32
    if t.dtype == torch.bfloat16:
        return BF16
    raise TypeError(f"feature tensors are float32 or bfloat16, got {t.dtype}")


def _mat_any(t):
    """(pointer, leading dimension in elements) of a 2-D row-major tensor or view."""
    if t.dim() != 2 or (t.shape[1] > 1 and t.stride(1) != 1):
        raise ValueError("need a 2-D tensor with contiguous rows")
    return t.data_ptr(), t.stride(0) if t.shape[0] > 1 else max(t.stride(0), t.shape[1])


_CODES = {torch.float32: F32, torch.bfloat16: BF16}


def _size_any(t):
    """_mat(t), rows, columns and the dtype's code (of any other type the dtype itself: equal only to itself, and no call takes
    it)."""
    return _mat_any(t) + (t.shape[0], t.shape[1], _CODES.get(t.dtype, t.dtype))


def _ptr_any(t, dtype=None):
    if t is None:
        return 0
    if dtype is not None and t.dtype != dtype:
        raise TypeError(f"expected {dtype}, got {t.dtype}")
    if not t.is_contiguous():
        raise ValueError("need a contiguous tensor")
    return t.data_ptr()


_mat, _size, _ptr = _mat_any, _size_any, _ptr_any        # until the library is loaded (_Calls)
_NONE = (0, 0, 0, 0, None)                               # _size of an argument that is not given


def _weights(w):
    """(pointer, rows, columns, dtype code) of a contiguous matrix."""
    p, ld, rows, cols, dt = _size(w)
    return _ptr(w) if ld != cols else p, rows, cols, dt


# the current stream's handle without a Stream object around it, where torch has these (they are not public)
_raw_stream = getattr(torch._C, "_cuda_getCurrentRawStream", None)
_device = getattr(torch._C, "_cuda_getDevice", None)


def _stream():
    if _raw_stream is None or _device is None:
        return torch.cuda.current_stream().cuda_stream
    return _raw_stream(_device())


def gas_version() -> int:
    return int(lib().gas_version())


def gas_pull(hist, idx, dst, base=0, n=None):
    """dst[i] = hist[idx[i]] (idx int32 tensor) or hist[base+i] (idx None)."""
    hp, ldh, rows, F, dt = _size(hist)
    dp, ldd, room, Fd, dtd = _size(dst)
    if n is None:
        n = idx.numel() if idx is not None else room
    if dtd != dt or Fd != F or room < n:
        raise ValueError("gas_pull: dst does not match")
    fn = _calls().gas_pull_host if isinstance(hist, HostTable) else _calls().gas_pull
    _check(fn(hp, rows, ldh, _ptr(idx, torch.int32), base, n, F, dt, dp, ldd, _stream()))


def gas_push(src, idx, hist, base=0, n=None):
    """hist[idx[i]] = src[i] (idx int32 tensor, distinct) or hist[base+i] = src[i] (idx None)."""
    hp, ldh, rows, F, dt = _size(hist)
    sp, lds, there, Fs, dts = _size(src)
    if n is None:
        n = idx.numel() if idx is not None else there
    if dts != dt or Fs != F or there < n:
        raise ValueError("gas_push: src does not match")
    fn = _calls().gas_push_host if isinstance(hist, HostTable) else _calls().gas_push
    _check(fn(sp, lds, _ptr(idx, torch.int32), base, n, F, dt, hp, rows, ldh, _stream()))


def gas_gcn_norm(ptr, ind, n_id, deg, val):
    _check(_calls().gas_gcn_norm(_ptr(ptr, torch.int32), _ptr(ind, torch.int32), ptr.numel() - 1,
                              _ptr(n_id, torch.int32), _ptr(deg, torch.int32), _ptr(val, torch.float32), _stream()))


class PlanOptions(C.Structure):
    """gas_plan_options of the C ABI; a zero field means the default."""
    _fields_ = [("heavy_threshold", C.c_int32), ("chunk", C.c_int32), ("min_chunk", C.c_int32),
                ("window_rows", C.c_int32), ("xcd_ranges", C.c_int32), ("host_builder", C.c_int32)]


class Plan:
    """Owner of a gas_plan handle."""

    def __init__(self, ptr: torch.Tensor, nnz: int, max_F: int, n_rows=None, ind=None, options=None):
        """options: dict with any of heavy_threshold, chunk, min_chunk, window_rows, xcd_ranges (gas_plan_options)."""
        self.n_rows = ptr.numel() - 1 if n_rows is None else n_rows
        self.handle = C.c_void_p(0)
        if ind is not None and ind.numel() < nnz:
            raise ValueError("gas_plan_create: ind is shorter than nnz")
        opt = None
        if options:
            opt = PlanOptions(**options)
        _check(_calls().gas_plan_create_opt(_ptr(ptr, torch.int32), _ptr(ind, torch.int32), self.n_rows,
                                         nnz, max_F, None if opt is None else C.byref(opt),
                                         _stream(), C.byref(self.handle)))

    def describe(self) -> dict:
        info = (C.c_int64 * 16)()
        _check(_calls().gas_plan_describe(self.handle, info))
        keys = ["n_rows", "nnz", "n_groups", "n_heavy", "n_chunks", "xcd_ranges", "max_F"]
        d = {k: int(info[i]) for i, k in enumerate(keys)}
        d["xcd_start"] = [int(info[7 + x]) for x in range(9)]
        return d

    def lists(self):
        """(group, heavy, chunk) as numpy int32 arrays on the host."""
        import numpy as np
        d = self.describe()
        group = np.zeros(2 * d["n_groups"], dtype=np.int32)
        heavy = np.zeros(2 * d["n_heavy"] + 1 if d["n_heavy"] else 0, dtype=np.int32)
        chunk = np.zeros(3 * d["n_chunks"], dtype=np.int32)
        as_p = lambda a: a.ctypes.data_as(C.c_void_p) if a.size else None
        _check(_calls().gas_plan_copy_lists(self.handle, as_p(group), as_p(heavy), as_p(chunk), _stream()))
        return group, heavy, chunk

    def close(self):
        if self.handle:
            lib().gas_plan_destroy(self.handle)
            self.handle = C.c_void_p(0)

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass


def gas_plan_create(ptr, nnz, max_F, n_rows=None, ind=None, options=None) -> Plan:
    return Plan(ptr, nnz, max_F, n_rows, ind, options)


def gas_plan_destroy(plan: Plan):
    plan.close()


def gas_spmm(plan, rowptr, col, val, x, z, diag=0.0, s_agg=1.0, r=None, s_res=0.0):
    xp, ldx, _, F, dt = _size(x)
    zp, ldz, rows, Fz, dtz = _size(z)
    rp, ldr, _, _, dtr = _NONE if r is None else _size(r)
    if r is not None and dtr != dt:
        raise TypeError("gas_spmm: R must have X's dtype")
    if Fz != F or rows < plan.n_rows:
        raise ValueError("gas_spmm: Z does not match")
    _check(_calls().gas_spmm(plan.handle, _ptr(rowptr, torch.int32), _ptr(col, torch.int32), _ptr(val, torch.float32),
                             diag, xp, ldx, dt, F, s_agg, rp, ldr, s_res, zp, ldz, dtz, _stream()))


def gas_fuse_sources(col, nb, n_id, src):
    _check(_calls().gas_fuse_sources(_ptr(col, torch.int32), col.numel(), nb, _ptr(n_id, torch.int32),
                                  _ptr(src, torch.int32), _stream()))


def gas_spmm_hist(plan, rowptr, src, val, x, hist, z, diag=0.0, s_agg=1.0, r=None, s_res=0.0):
    """x: the in-batch rows [n_rows, F]; hist: the history table the halo rows are read from."""
    xp, ldx, there, F, dt = _size(x)
    hp, ldh, n_hist, Fh, dth = _size(hist)
    zp, ldz, rows, Fz, dtz = _size(z)
    rp, ldr, _, _, dtr = _NONE if r is None else _size(r)
    if dth != dt or Fh != F or (r is not None and dtr != dt):
        raise TypeError("gas_spmm_hist: hist and R must match X")
    if Fz != F or rows < plan.n_rows or there < plan.n_rows:
        raise ValueError("gas_spmm_hist: shapes do not match")
    _check(_calls().gas_spmm_hist(plan.handle, _ptr(rowptr, torch.int32), _ptr(src, torch.int32), _ptr(val, torch.float32),
                                  diag, xp, ldx, hp, n_hist, ldh, dt, F, s_agg, rp, ldr, s_res, zp, ldz, dtz, _stream()))


def gas_spmm_table(plan, rowptr, src, val, table, z, diag=0.0, s_agg=1.0, own=None):
    """Every row is one of the table's: an entry's -1 - src, the diagonal term's own[v]."""
    tp, ldt, n_table, F, dt = _size(table)
    zp, ldz, rows, Fz, dtz = _size(z)
    if Fz != F or rows < plan.n_rows or (own is not None and own.numel() < plan.n_rows):
        raise ValueError("gas_spmm_table: shapes do not match")
    _check(_calls().gas_spmm_table(plan.handle, _ptr(rowptr, torch.int32), _ptr(src, torch.int32), _ptr(val, torch.float32), diag,
                                   _ptr(own, torch.int32), tp, n_table, ldt, dt, F, s_agg, zp, ldz, dtz, _stream()))


def gas_spmm_t(plan, colptr, row, val, g, gx, diag=0.0, s_agg=1.0):
    gp, ldg, there, F, dt = _size(g)
    op, ldo, rows, Fo, dto = _size(gx)
    if Fo != F or rows < plan.n_rows:
        raise ValueError("gas_spmm_t: GX does not match")
    _check(_calls().gas_spmm_t(plan.handle, _ptr(colptr, torch.int32), _ptr(row, torch.int32), _ptr(val, torch.float32),
                               diag, s_agg, there, gp, ldg, dt, F, op, ldo, dto, _stream()))


def gas_spmm_t_relu(plan, colptr, row, val, g, y, gx, diag=0.0, s_agg=1.0):
    """gas_spmm_t, then zero where the activations y [n_rows, F] are not positive."""
    gp, ldg, there, F, dt = _size(g)
    yp, ldy, ny, Fy, dty = _size(y)
    op, ldo, rows, Fo, dto = _size(gx)
    if Fo != F or rows < plan.n_rows or Fy != F or ny < plan.n_rows or not (dt == dty == dto):
        raise ValueError("gas_spmm_t_relu: shapes or dtypes do not match")
    _check(_calls().gas_spmm_t_relu(plan.handle, _ptr(colptr, torch.int32), _ptr(row, torch.int32), _ptr(val, torch.float32),
                                    diag, s_agg, there, gp, ldg, dt, F, yp, ldy, op, ldo, _stream()))


def gas_linear(z, w, y, bias=None, c_identity=0.0, c_weight=1.0, relu=False):
    zp, ldz, n, f_in, dt = _size(z)
    yp, ldy, ny, f_out, dty = _size(y)
    wp, w_in, w_out, dtw = _weights(w)
    if dtw != dt or dty != dt or w_in != f_in or ny != n or f_out != w_out:
        raise ValueError("gas_linear: shapes or dtypes do not match")
    _check(_calls().gas_linear(zp, ldz, n, f_in, wp, f_out, _ptr(bias), dt, c_identity, c_weight, int(relu), yp, ldy, _stream()))


def gas_linear_in_order(z, w, y):
    """y = z @ w, every sum in the order of k where the rows and widths take no 16-byte pieces (bf16)."""
    zp, ldz, n, f_in, dt = _size(z)
    yp, ldy, ny, f_out, dty = _size(y)
    if ny != n or dty != dt or w.dtype != z.dtype or w.shape != (f_in, f_out):
        raise ValueError("gas_linear_in_order: shapes or dtypes do not match")
    _check(_calls().gas_linear_in_order(zp, ldz, n, f_in, _ptr(w), f_out, dt, yp, ldy, _stream()))


def gas_mlp2(z, w1, w2, y, b1=None, b2=None, relu_out=False):
    zp, ldz, n, f_in, dt = _size(z)
    yp, ldy, ny, f_out, dty = _size(y)
    p1, w1_in, hidden, dt1 = _weights(w1)
    p2, w2_in, w2_out, dt2 = _weights(w2)
    if not (dt1 == dt2 == dt == dty) or w1_in != f_in or w2_in != hidden or ny != n or f_out != w2_out:
        raise ValueError("gas_mlp2: shapes or dtypes do not match")
    _check(_calls().gas_mlp2(zp, ldz, n, f_in, p1, hidden, _ptr(b1), p2, f_out, _ptr(b2), dt, int(relu_out), yp, ldy, _stream()))


def gas_validate_indices(idx, limit) -> bool:
    st = _calls().gas_validate_indices(_ptr(idx, torch.int32), idx.numel(), limit, _stream())
    if st == -4:
        return False
    _check(st)
    return True


def gas_relu_bwd(gy, y, gp):
    """gp = gy where y > 0 else 0 (gp may be gy itself)."""
    a, lda = _mat(gy)
    b, ldb = _mat(y)
    c, ldc = _mat(gp)
    if not (gy.shape == y.shape == gp.shape and gy.dtype == y.dtype == gp.dtype):
        raise ValueError("gas_relu_bwd: shapes or dtypes do not match")
    _check(_calls().gas_relu_bwd(a, lda, b, ldb, gy.shape[0], gy.shape[1], _dt(gy), c, ldc,
                              _stream()))


def gas_linear_bwd_input(gp, w, gz, c_identity=0.0, c_weight=1.0, mask=None):
    """gz [n, F_in] = c_identity * gp + c_weight * gp @ w.T, zeroed where mask <= 0; w is [F_in, F_out]."""
    a, lda, n, f_out, dt = _size(gp)
    c, ldc, nz, f_in, dtz = _size(gz)
    wp, w_in, w_out, dtw = _weights(w)
    mp, ldm, nm, fm, dtm = (0, 0, nz, f_in, dt) if mask is None else _size(mask)
    if dtw != dt or dtz != dt or w_out != f_out or nz != n or f_in != w_in or nm != nz or fm != f_in or dtm != dt:
        raise ValueError("gas_linear_bwd_input: shapes or dtypes do not match")
    _check(_calls().gas_linear_bwd_input(a, lda, n, f_out, wp, f_in, dt, c_identity, c_weight, mp, ldm, c, ldc, _stream()))


def gas_linear_bwd_input_add(gp, w, gz, c_identity=0.0, c_weight=1.0, add=None, mask=None, total=None, c_total=0.0):
    """gas_linear_bwd_input with `add` added before the mask; total += c_total * gz where given."""
    a, lda, n, f_out, dt = _size(gp)
    c, ldc, nz, f_in, dtz = _size(gz)
    wp, w_in, w_out, dtw = _weights(w)
    same = (nz, f_in, dt)
    ap, ldadd, *like_a = (0, 0, *same) if add is None else _size(add)
    mp, ldm, *like_m = (0, 0, *same) if mask is None else _size(mask)
    tp, ldt, *like_t = (0, 0, *same) if total is None else _size(total)
    if dtw != dt or dtz != dt or w_out != f_out or nz != n or f_in != w_in or not (tuple(like_a) == tuple(like_m) == tuple(like_t) == same):
        raise ValueError("gas_linear_bwd_input_add: shapes or dtypes do not match")
    _check(_calls().gas_linear_bwd_input_add(a, lda, n, f_out, wp, f_in, dt, c_identity, c_weight, ap, ldadd, mp, ldm, c_total, tp,
                                             ldt, c, ldc, _stream()))


def gas_linear_bwd_weight_workspace(n_rows, f_in, f_out) -> int:
    return int(_calls().gas_linear_bwd_weight_workspace(n_rows, f_in, f_out))


def gas_linear_bwd_weight(z, gp, dw, workspace, c_weight=1.0):
    """dw [F_in, F_out] float32 = c_weight * z.T @ gp; workspace: a uint8 tensor of at least
    gas_linear_bwd_weight_workspace(...) bytes."""
    a, lda = _mat(z)
    b, ldb = _mat(gp)
    if z.dtype != gp.dtype or z.shape[0] != gp.shape[0] or dw.dtype != torch.float32 or \
            dw.shape != (z.shape[1], gp.shape[1]) or not dw.is_contiguous():
        raise ValueError("gas_linear_bwd_weight: shapes or dtypes do not match")
    nbytes = 0 if workspace is None else workspace.numel() * workspace.element_size()
    _check(_calls().gas_linear_bwd_weight(a, lda, b, ldb, z.shape[0], z.shape[1],
                                       gp.shape[1], _dt(z), c_weight, _ptr(dw),
                                       _ptr(workspace), nbytes, _stream()))


SHARED_WORKSPACE = 128 << 20


def gas_linear_bwd_weights(items):
    """gas_linear_bwd_weight of every (z, gp, dw, c_weight) of a list, of one dtype; in float32 they share launches.  The
    workspace is allocated here, once for all; a list that would share more than SHARED_WORKSPACE bytes goes in halves (16 of
    21,248 rows of 64 x 64 take 44 MB together, 16,000 rows of 1,433 x 256 62 MB each)."""
    n = len(items)
    if n == 0:
        return
    dev = items[0][0].device
    zs, gs = [_size(z) for z, _, _, _ in items], [_size(g) for _, g, _, _ in items]
    dt, dws = zs[0][4], []
    for (_, _, rows, f_in, dtz), (_, _, rows_g, f_out, dtg), (_, _, dw, _) in zip(zs, gs, items):
        if dtz != dt or dtg != dt or dw.dtype != torch.float32 or not dw.is_contiguous() or rows != rows_g or dw.shape != (f_in, f_out):
            raise ValueError("gas_linear_bwd_weights: shapes or dtypes do not match")
        dws.append(dw.data_ptr())
    pointers, longs, ints = C.c_void_p * n, C.c_int64 * n, C.c_int32 * n
    rows, f_in, f_out = longs(*[t[2] for t in zs]), ints(*[t[3] for t in zs]), ints(*[t[3] for t in gs])
    need = _calls().gas_linear_bwd_weights_workspace(n, rows, f_in, f_out, dt)
    if need > SHARED_WORKSPACE and n > 1:
        gas_linear_bwd_weights(items[:n // 2])
        gas_linear_bwd_weights(items[n // 2:])
        return
    ws = torch.empty(max(1, need), dtype=torch.uint8, device=dev)
    _check(_calls().gas_linear_bwd_weights(
        n, pointers(*[t[0] for t in zs]), longs(*[t[1] for t in zs]), pointers(*[t[0] for t in gs]), longs(*[t[1] for t in gs]),
        rows, f_in, f_out, dt, (C.c_float * n)(*[c for _, _, _, c in items]), pointers(*dws), ws.data_ptr(), need, _stream()))


def gas_linear_bwd_weight_static(z, gp, dw, c_weight=1.0):
    """gas_linear_bwd_weight with the slab partials in the library's static scratch array (no workspace)."""
    a, lda = _mat(z)
    b, ldb = _mat(gp)
    if z.dtype != gp.dtype or z.shape[0] != gp.shape[0] or dw.dtype != torch.float32 or \
            dw.shape != (z.shape[1], gp.shape[1]) or not dw.is_contiguous():
        raise ValueError("gas_linear_bwd_weight_static: shapes or dtypes do not match")
    _check(_calls().gas_linear_bwd_weight_static(a, lda, b, ldb, z.shape[0], z.shape[1],
                                              gp.shape[1], _dt(z), c_weight,
                                              _ptr(dw), _stream()))


def gas_linear_push(z, w, y, idx, hist, bias=None, c_identity=0.0, c_weight=1.0, relu=False):
    """gas_linear, and y[i] is also stored to hist[idx[i]] (Push fused into the epilogue)."""
    zp, ldz, n, f_in, dt = _size(z)
    yp, ldy, ny, f_out, dty = _size(y)
    hp, ldh, n_hist, fh, dth = _size(hist)
    wp, w_in, w_out, dtw = _weights(w)
    if dtw != dt or dty != dt or dth != dt or w_in != f_in or ny != n or f_out != w_out or fh != w_out or idx.numel() != n:
        raise ValueError("gas_linear_push: shapes or dtypes do not match")
    _check(_calls().gas_linear_push(zp, ldz, n, f_in, wp, f_out, _ptr(bias), dt, c_identity, c_weight, int(relu), yp, ldy,
                                    _ptr(idx, torch.int32), hp, n_hist, ldh, _stream()))


def gas_mlp2_keep(z, w1, w2, y, h_out, idx=None, hist=None, b1=None, b2=None, relu_out=False):
    """gas_mlp2 that also stores the hidden activation relu(z w1 + b1) to h_out, and (idx, hist given) pushes y."""
    zp, ldz, n, f_in, dt = _size(z)
    yp, ldy, ny, f_out, dty = _size(y)
    hp, ldh, nh, fh, dth = _size(h_out)
    p1, w1_in, hidden, dt1 = _weights(w1)
    p2, w2_in, w2_out, dt2 = _weights(w2)
    tp, ldt, n_hist, ft, dtt = (0, 0, 0, w2_out, dt) if hist is None else _size(hist)
    if not (dt1 == dt2 == dt == dty == dth == dtt) or w1_in != f_in or w2_in != hidden or ny != n or f_out != w2_out or nh != n or \
            fh != hidden or (hist is None) != (idx is None) or ft != w2_out or (hist is not None and idx.numel() != n):
        raise ValueError("gas_mlp2_keep: shapes or dtypes do not match")
    _check(_calls().gas_mlp2_keep(zp, ldz, n, f_in, p1, hidden, _ptr(b1), p2, f_out, _ptr(b2), dt, int(relu_out), yp, ldy, hp, ldh,
                                  _ptr(idx, torch.int32), tp, n_hist, ldt, _stream()))


def spmm_linear_supported(x, f_out) -> bool:
    """Whether gas_spmm_linear takes this layer (fp32, widths multiples of 4 up to 128)."""
    f_in = x.shape[1]
    return f_out <= 128 and f_in <= 128 and f_in % 4 == 0 and f_out % 4 == 0 and x.dtype == torch.float32


def gas_spmm_linear(rowptr, src, val, x, w, y, hist=None, diag=0.0, s_agg=1.0, r=None, s_res=0.0, bias=None,
                    c_identity=0.0, c_weight=1.0, relu=False, push_idx=None, push_hist=None, z_out=None):
    """One layer in one launch: aggregation of the rows of y (sources: rows of x, or rows of hist for negative
    indices), transform by w, optional store of every output row to push_hist[push_idx[i]]."""
    xp, ldx, _, f_in, dt = _size(x)
    yp, ldy, n_rows, f_out, dty = _size(y)
    wp, w_in, w_out, dtw = _weights(w)
    hp, ldh, n_hist, fh, dth = (0, 0, 0, f_in, dt) if hist is None else _size(hist)
    rp, ldr, nr, fr, dtr = (0, 0, n_rows, f_in, dt) if r is None else _size(r)
    pp, ldp, n_push, fp, dtp = (0, 0, 0, w_out, dt) if push_hist is None else _size(push_hist)
    zp, ldzo, nz, fz, dtz = (0, 0, n_rows, f_in, dt) if z_out is None else _size(z_out)
    if dtz != dt or fz != f_in or nz < n_rows:
        raise ValueError("gas_spmm_linear: z_out does not match")
    if dtw != dt or dty != dt or w_in != f_in or f_out != w_out or rowptr.numel() != n_rows + 1 or dth != dt or fh != f_in or \
            dtr != dt or fr != f_in or nr < n_rows or dtp != dt or fp != w_out or \
            (push_hist is not None and (push_idx is None or push_idx.numel() != n_rows)):
        raise ValueError("gas_spmm_linear: shapes or dtypes do not match")
    _check(_calls().gas_spmm_linear(
        _ptr(rowptr, torch.int32), _ptr(src, torch.int32), _ptr(val, torch.float32), n_rows, xp, ldx, hp, n_hist, ldh, dt, f_in, diag,
        s_agg, rp, ldr, s_res, wp, f_out, _ptr(bias), c_identity, c_weight, int(relu), yp, ldy, zp, ldzo,
        _ptr(push_idx, torch.int32), pp, n_push, ldp, _stream()))


def gas_spmm_t_relu_linear(colptr, row, val, g, y, gx, w, gz, s_agg=1.0, c_identity=0.0, c_weight=1.0, total=None, c_total=0.0):
    """gx = (y > 0) * s_agg * (adjoint of the aggregation applied to g), gz = c_identity * gx + c_weight * gx @ w.T (w: the
    weights of the layer below) and total += c_total * gz in one launch."""
    a, lda, _, fg, dt = _size(g)
    yp, ldy, ny, fy, dty = _size(y)
    xp, ldx, n, f, dtx = _size(gx)
    zp, ldz, nz, f_below, dtz = _size(gz)
    wp, w_in, w_out, dtw = _weights(w)
    tp, ldt, nt, ft, dtt = (0, 0, n, w_in, dt) if total is None else _size(total)
    if fg != f or fy != f or ny < n or w_out != f or nz != n or f_below != w_in or colptr.numel() < n + 1 or \
            not (dt == dtx == dty == dtw == dtz == dtt) or ft != f_below or nt < n:
        raise ValueError("gas_spmm_t_relu_linear: shapes or dtypes do not match")
    _check(_calls().gas_spmm_t_relu_linear(
        _ptr(colptr, torch.int32), _ptr(row, torch.int32), _ptr(val, torch.float32), n, a, lda, dt, f, s_agg, yp, ldy, xp,
        ldx, wp, f_below, c_identity, c_weight, c_total, tp, ldt, zp, ldz, _stream()))


def _pointers(mats, n, shape, like, what, null=False):
    """(pointers, row strides) of `n` matrices of one shape and type (None: a null pointer, where allowed)."""
    if len(mats) != n:
        raise ValueError(f"{what}: {len(mats)} matrices for {n} layers")
    ptrs, lds = [], []
    for t in mats:
        if t is None and null:
            ptrs.append(None)
            lds.append(0)
            continue
        size, step = t.shape, t.stride()                     # as _mat, with few calls: there are hundreds of matrices
        if len(size) != 2 or size[1] != shape[1] or size[0] < shape[0] or t.dtype != like or (step[1] != 1 and size[1] > 1):
            raise ValueError(f"{what}: shapes, dtypes or strides do not match")
        ptrs.append(t.data_ptr())
        lds.append(step[0] if size[0] > 1 else max(step[0], size[1]))
    return (C.c_void_p * n)(*ptrs), lds


def _one_stride(lds, what):
    if any(ld != lds[0] for ld in lds):
        raise ValueError(f"{what}: row strides do not match")
    return lds[0]


def gas_spmm_linear_layers(rowptr, src_first, src, val, x, ws, ys, hists, s_agg=1.0, r=None, s_res=0.0,
                           c_identity=None, c_weight=None, relu_last=False, z_outs=None, push_idx=None, push_hists=None):
    """gas_spmm_linear of len(ws) layers of one width, each reading the one before: lists of weights, outputs (of one row stride;
    an output may come again from the layer after next on), history tables and, optionally, kept aggregated rows and tables to
    push to (None: none)."""
    n, (n_rows, f) = len(ws), ys[0].shape
    xp, ldx = _mat(x)
    rp, ldr = (0, 0) if r is None else _mat(r)
    wp, _ = _pointers(ws, n, (f, f), x.dtype, "gas_spmm_linear_layers: weights")
    yp, ldy = _pointers(ys, n, (n_rows, f), x.dtype, "gas_spmm_linear_layers: outputs")
    hp, lds_h = _pointers(hists, n, (0, f), x.dtype, "gas_spmm_linear_layers: histories", null=True)
    zp, ldz = (None, [0]) if z_outs is None else _pointers(z_outs, n, (n_rows, f), x.dtype, "gas_spmm_linear_layers: kept rows")
    pp, lds_p = (None, []) if push_hists is None else _pointers(push_hists, n, (0, f), x.dtype, "gas_spmm_linear_layers: tables", null=True)
    if x.shape[1] != f or rowptr.numel() != n_rows + 1 or not all(w.is_contiguous() for w in ws) or \
            (r is not None and (r.dtype != x.dtype or r.shape[1] != f or r.shape[0] < n_rows)) or \
            (push_idx is None) != (push_hists is None) or (push_idx is not None and push_idx.numel() != n_rows):
        raise ValueError("gas_spmm_linear_layers: shapes or dtypes do not match")
    floats, longs = C.c_float * n, C.c_int64 * n
    n_hist_rows = min((t.shape[0] for t in hists if t is not None), default=0)
    n_push_rows = min((t.shape[0] for t in push_hists or () if t is not None), default=0)
    ldy, ldz = _one_stride(ldy, "gas_spmm_linear_layers: outputs"), _one_stride(ldz, "gas_spmm_linear_layers: kept rows")
    _check(_calls().gas_spmm_linear_layers(
        n, _ptr(rowptr, torch.int32), _ptr(src_first, torch.int32), _ptr(src, torch.int32), _ptr(val, torch.float32), n_rows, xp, ldx,
        hp, n_hist_rows, longs(*lds_h), _dt(x), f, s_agg, rp, ldr, s_res, wp, floats(*(c_identity or [0.0] * n)),
        floats(*(c_weight or [1.0] * n)), int(relu_last), yp, ldy, zp, ldz, _ptr(push_idx, torch.int32), pp, n_push_rows,
        longs(*lds_p), _stream()))


def gas_spmm_t_relu_linear_layers(colptr, row, val, g, ys, gxs, ws, gzs, s_agg=1.0, c_identity=None, c_weight=None, total=None,
                                  c_total=0.0):
    """gas_spmm_t_relu_linear of len(ws) layers of one width, from the top one down, each reading the gz of the one before."""
    n, (n_rows, f) = len(ws), gxs[0].shape
    a, lda = _mat(g)
    tp, ldt = (0, 0) if total is None else _mat(total)
    what = "gas_spmm_t_relu_linear_layers"
    yp, ldy = _pointers(ys, n, (n_rows, f), g.dtype, what)
    xp, ldx = _pointers(gxs, n, (n_rows, f), g.dtype, what)
    wp, _ = _pointers(ws, n, (f, f), g.dtype, what)
    zp, ldz = _pointers(gzs, n, (n_rows, f), g.dtype, what)
    if g.shape[1] != f or colptr.numel() < n_rows + 1 or not all(w.is_contiguous() for w in ws) or \
            (total is not None and (total.dtype != g.dtype or total.shape[1] != f or total.shape[0] < n_rows)):
        raise ValueError("gas_spmm_t_relu_linear_layers: shapes or dtypes do not match")
    floats = C.c_float * n
    ldy, ldx, ldz = (_one_stride(ld, what) for ld in (ldy, ldx, ldz))
    _check(_calls().gas_spmm_t_relu_linear_layers(
        n, _ptr(colptr, torch.int32), _ptr(row, torch.int32), _ptr(val, torch.float32), n_rows, a, lda, _dt(g), f, s_agg, yp, ldy, xp,
        ldx, wp, floats(*(c_identity or [0.0] * n)), floats(*(c_weight or [1.0] * n)), c_total, tp, ldt, zp, ldz, _stream()))


def gas_mlp2_push(z, w1, w2, y, idx, hist, b1=None, b2=None, relu_out=False):
    """gas_mlp2, and y[i] is also stored to hist[idx[i]]."""
    zp, ldz, n, f_in, dt = _size(z)
    yp, ldy, ny, f_out, dty = _size(y)
    hp, ldh, n_hist, fh, dth = _size(hist)
    p1, w1_in, hidden, dt1 = _weights(w1)
    p2, w2_in, w2_out, dt2 = _weights(w2)
    if not (dt1 == dt2 == dt == dty == dth) or w1_in != f_in or w2_in != hidden or ny != n or f_out != w2_out or fh != w2_out or \
            idx.numel() != n:
        raise ValueError("gas_mlp2_push: shapes or dtypes do not match")
    _check(_calls().gas_mlp2_push(zp, ldz, n, f_in, p1, hidden, _ptr(b1), p2, f_out, _ptr(b2), dt, int(relu_out), yp, ldy,
                                  _ptr(idx, torch.int32), hp, n_hist, ldh, _stream()))


def gas_softmax_xent(a, labels, grad, loss_rows, loss_sum=None, scale=1.0):
    """Softmax cross-entropy per row and its gradient (scaled); rows with a label outside [0, C) are skipped."""
    ap, lda, n, classes, dt = _size(a)
    gp, ldg, ng, fg, dtg = _size(grad)
    if dtg != dt or ng != n or fg != classes or labels.numel() != n or \
            loss_rows.dtype != torch.float32 or loss_rows.numel() != n or not loss_rows.is_contiguous():
        raise ValueError("gas_softmax_xent: shapes or dtypes do not match")
    _check(_calls().gas_softmax_xent(ap, lda, n, classes, dt, _ptr(labels, torch.int32), scale, _ptr(loss_rows, torch.float32),
                                     _ptr(loss_sum, torch.float32), gp, ldg, _stream()))


def gas_sgd_step(w, dw, lr, weight_decay=0.0):
    """In place: w <- w - lr * (dw + weight_decay * w); dw float32 of the same shape."""
    if not w.is_contiguous() or not dw.is_contiguous() or dw.dtype != torch.float32 or dw.numel() != w.numel():
        raise ValueError("gas_sgd_step: w and dw must be contiguous and of equal size, dw float32")
    _check(_calls().gas_sgd_step(_ptr(w), w.numel(), _dt(w), _ptr(dw, torch.float32),
                              lr, weight_decay, _stream()))


def gas_sgd_steps(pairs, lr, weight_decay=0.0):
    """gas_sgd_step on every (w, dw) of a list of matrices of one dtype, in order; they share launches."""
    n = len(pairs)
    if n == 0:
        return
    dt, ws, dws, sizes = pairs[0][0].dtype, [], [], []
    for w, dw in pairs:
        size = w.numel()
        if not w.is_contiguous() or not dw.is_contiguous() or dw.dtype != torch.float32 or dw.numel() != size or w.dtype != dt:
            raise ValueError("gas_sgd_steps: w and dw must be contiguous and of equal size, dw float32, w of one dtype")
        ws.append(w.data_ptr())
        dws.append(dw.data_ptr())
        sizes.append(size)
    pointers = C.c_void_p * n
    _check(_calls().gas_sgd_steps(n, pointers(*ws), (C.c_int64 * n)(*sizes), _dt(pairs[0][0]), pointers(*dws), lr, weight_decay,
                                  _stream()))


def gas_sq_norm(x, out):
    """out[0] = sum of the squares of x (float32, contiguous); out: a 1-element float32 view."""
    if not x.is_contiguous() or x.dtype != torch.float32 or out.dtype != torch.float32 or out.numel() < 1:
        raise ValueError("gas_sq_norm: x float32 contiguous, out float32")
    _check(_calls().gas_sq_norm(_ptr(x, torch.float32), x.numel(), _ptr(out, torch.float32), _stream()))


def gas_sgd_step_clipped(w, dw, lr, sq_norms, max_norm, weight_decay=0.0):
    """gas_sgd_step with dw scaled by min(1, max_norm / (sqrt(sum(sq_norms)) + 1e-6)), formed on the device."""
    if not w.is_contiguous() or not dw.is_contiguous() or dw.dtype != torch.float32 or dw.numel() != w.numel():
        raise ValueError("gas_sgd_step_clipped: w and dw must be contiguous and of equal size, dw float32")
    if sq_norms.dtype != torch.float32 or not sq_norms.is_contiguous():
        raise ValueError("gas_sgd_step_clipped: sq_norms float32 contiguous")
    _check(_calls().gas_sgd_step_clipped(_ptr(w), w.numel(), _dt(w), _ptr(dw, torch.float32),
                                      lr, weight_decay, _ptr(sq_norms, torch.float32),
                                      sq_norms.numel(), max_norm, _stream()))


ANY_LENGTH = 0x7FFFFFFF          # of rows and columns: nothing is known


def gas_pna_aggregate(rowptr, col, x, out, delta, add=None, blocks=9, longest=ANY_LENGTH, own=None, own_to=None):
    """out [n_rows, 9F] = scalers [1, s, 1/s] (x) aggregators [mean, min, max] over the neighbours (+ add); blocks = 3: out
    [n_rows, 3F], the aggregators alone.  longest: no row has more entries; own_to[v] = own[v] if given."""
    n_rows = rowptr.numel() - 1
    xp, ldx, _, F, dt = _size(x)
    op, ldo, no, Fo, dto = _size(out)
    ap, lda, na, Fa, dta = (0, 0, n_rows, F, dt) if add is None else _size(add)
    if dto != dt or no < n_rows or Fo != blocks * F or dta != dt or Fa != F or na < n_rows:
        raise ValueError("gas_pna_aggregate: shapes or dtypes do not match")
    wp, ldw, nw, Fw, dtw = (0, 0, n_rows, 0, dt) if own is None else _size(own)
    tp, ldt, nt, Ft, dtt = (0, 0, n_rows, 0, dt) if own_to is None else _size(own_to)
    if Fw != Ft or nw < n_rows or nt < n_rows or dtw != dt or dtt != dt:
        raise ValueError("gas_pna_aggregate: the own rows and their target do not match")
    _check(_calls().gas_pna_aggregate_own(_ptr(rowptr, torch.int32), _ptr(col, torch.int32), n_rows, longest, xp, ldx, dt, F, ap, lda,
                                          delta, blocks, op, ldo, wp, ldw, Fw, tp, ldt, _stream()))


PNA_MAX_DEGREE = 63


def gas_pna_groups(rowptr, max_degree):
    """The rows of a pattern by their number of entries (at most max_degree, itself at most PNA_MAX_DEGREE), for gas_pna_linear
    and its backward calls."""
    n_rows = rowptr.numel() - 1
    groups = torch.empty(max(1, _calls().gas_pna_groups_workspace(n_rows, max_degree)), dtype=torch.uint8, device=rowptr.device)
    _check(_calls().gas_pna_groups(_ptr(rowptr, torch.int32), n_rows, max_degree, groups.data_ptr(), _stream()))
    return groups


def _pna_widths(x, w, f1, groups, max_degree):
    """F of w [F + 9 F1, F_out], checked against a matrix of the rows' [h | A ..] and the groups."""
    f = w.shape[0] - 9 * f1
    if f <= 0 or x.shape[1] < f + 3 * f1 or groups.numel() != _calls().gas_pna_groups_workspace(x.shape[0], max_degree) or \
            x.dtype != torch.float32:
        raise ValueError("gas_pna_linear: shapes or dtypes do not match")
    return f


def gas_pna_linear(groups, max_degree, x, w, f1, delta, y, relu=False, idx=None, hist=None):
    """y = act(h Wh + A (Wa + s Wb + Wc / s)) for x = [h | A ..], w = [Wh; Wa; Wb; Wc] with blocks of 3 f1 rows, and (idx, hist)
    push y."""
    f, (xp, ldx), (yp, ldy) = _pna_widths(x, w, f1, groups, max_degree), _mat(x), _mat(y)
    hp, ldh = (0, 0) if hist is None else _mat(hist)
    if w.dtype != x.dtype or y.dtype != x.dtype or y.shape != (x.shape[0], w.shape[1]) or (idx is None) != (hist is None) or \
            (hist is not None and (hist.dtype != x.dtype or hist.shape[1] != w.shape[1] or idx.numel() != x.shape[0])):
        raise ValueError("gas_pna_linear: shapes or dtypes do not match")
    ws = torch.empty(_calls().gas_pna_linear_workspace(max_degree, f, f1, w.shape[1]), dtype=torch.uint8, device=x.device)
    _check(_calls().gas_pna_linear(groups.data_ptr(), x.shape[0], max_degree, xp, ldx, f, f1, _ptr(w), w.shape[1], delta, int(relu), yp,
                                ldy, _ptr(idx, torch.int32), hp, ldh, ws.data_ptr(), ws.numel(), _stream()))


def gas_pna_linear_bwd_input(groups, max_degree, g, w, f1, delta, gx):
    """gx = [g Wh^T | g (Wa + s Wb + Wc / s)^T]."""
    f, (gp, ldg), (op, ldo) = _pna_widths(gx, w, f1, groups, max_degree), _mat(g), _mat(gx)
    if g.shape != (gx.shape[0], w.shape[1]) or g.dtype != gx.dtype or w.dtype != gx.dtype:
        raise ValueError("gas_pna_linear_bwd_input: shapes or dtypes do not match")
    ws = torch.empty(_calls().gas_pna_linear_workspace(max_degree, f, f1, w.shape[1]), dtype=torch.uint8, device=g.device)
    _check(_calls().gas_pna_linear_bwd_input(groups.data_ptr(), g.shape[0], max_degree, gp, ldg, f, f1, _ptr(w), w.shape[1], delta, op,
                                          ldo, ws.data_ptr(), ws.numel(), _stream()))


def gas_pna_linear_bwd_weight(groups, max_degree, x, g, f1, delta, dw):
    """dw [F + 9 f1, F_out] for x = [h | A ..] and the gradient g at the output."""
    f, (xp, ldx), (gp, ldg) = _pna_widths(x, dw, f1, groups, max_degree), _mat(x), _mat(g)
    if g.shape != (x.shape[0], dw.shape[1]) or g.dtype != x.dtype or dw.dtype != torch.float32 or not dw.is_contiguous():
        raise ValueError("gas_pna_linear_bwd_weight: shapes or dtypes do not match")
    ws = torch.empty(_calls().gas_pna_linear_bwd_weight_workspace(x.shape[0], max_degree, f, f1, g.shape[1]), dtype=torch.uint8, device=x.device)
    _check(_calls().gas_pna_linear_bwd_weight(groups.data_ptr(), x.shape[0], max_degree, xp, ldx, gp, ldg, f, f1, g.shape[1], delta,
                                           dw.data_ptr(), ws.data_ptr(), ws.numel(), _stream()))


def gas_gat_aggregate(rowptr, col, p, a_dst, a_src, z, negative_slope=0.2, relu=False, heads=1, longest=ANY_LENGTH, idx=None,
                      hist=None):
    """z[v] = sum_k softmax_k(LeakyReLU(a_dst.p[v] + a_src.p[col k])) p[col k] over the entries of row v.  heads > 1: the
    columns of p and z and the elements of a_dst and a_src are that many equal blocks, a head each.  longest: no row has more
    entries; z[v] also goes to hist[idx[v]] if given (distinct)."""
    pp, ldp, _, width, dt = _size(p)
    zp, ldz, nz, fz, dtz = _size(z)
    n_rows = rowptr.numel() - 1
    if dtz != dt or a_dst.dtype != p.dtype or a_src.dtype != p.dtype or fz != width or \
            nz < n_rows or a_dst.numel() != width or a_src.numel() != width or heads < 1 or width % heads:
        raise ValueError("gas_gat_aggregate: shapes or dtypes do not match")
    hp, ldh, n_hist, fh, dth = (0, 0, 0, width, dt) if hist is None else _size(hist)
    if (idx is None) != (hist is None) or fh != width or dth != dt or (idx is not None and idx.numel() != n_rows):
        raise ValueError("gas_gat_aggregate: the history table or its indices do not match")
    _check(_calls().gas_gat_aggregate_push(_ptr(rowptr, torch.int32), _ptr(col, torch.int32), n_rows, longest, pp, ldp, dt,
                                           width // heads, heads, _ptr(a_dst), _ptr(a_src), negative_slope, int(relu), zp,
                                           ldz, _ptr(idx, torch.int32), hp, n_hist, ldh, _stream()))


def gas_axpy(x, e, y, alpha=1.0):
    """y = x + alpha * e over [n, F] (y may be x)."""
    xp, ldx = _mat(x)
    ep, lde = _mat(e)
    yp, ldy = _mat(y)
    if x.shape != e.shape or x.shape != y.shape or x.dtype != e.dtype or x.dtype != y.dtype:
        raise ValueError("gas_axpy: shapes or dtypes do not match")
    _check(_calls().gas_axpy(xp, ldx, ep, lde, x.shape[0], x.shape[1], _dt(x),
                          alpha, yp, ldy, _stream()))


def gas_row_dot(a, b, dot, dot_sum=None):
    """dot[i] = <a[i], b[i]> (float32 [n]); dot_sum (float32 [1]) receives their sum in a fixed order."""
    ap, lda, n, F, dt = _size(a)
    bp, ldb, nb, Fb, dtb = _size(b)
    if nb != n or Fb != F or dtb != dt or dot.dtype != torch.float32 or dot.numel() < n:
        raise ValueError("gas_row_dot: shapes or dtypes do not match")
    _check(_calls().gas_row_dot(ap, lda, bp, ldb, n, F, dt, _ptr(dot), _ptr(dot_sum), _stream()))


def gas_row_distance(a, b, dist, dist_sum=None):
    """dist[i] = ||a[i] - b[i]||_2 (float32 [n]); dist_sum (float32 [1]) receives their sum."""
    ap, lda = _mat(a)
    bp, ldb = _mat(b)
    if a.shape != b.shape or a.dtype != b.dtype or dist.dtype != torch.float32 or dist.numel() != a.shape[0] or \
            not dist.is_contiguous():
        raise ValueError("gas_row_distance: shapes or dtypes do not match")
    _check(_calls().gas_row_distance(ap, lda, bp, ldb, a.shape[0], a.shape[1], _dt(a),
                                  _ptr(dist, torch.float32), _ptr(dist_sum, torch.float32), _stream()))


def gas_row_distance_bwd(a, b, g, scale=1.0):
    """g[i] = scale * (a[i] - b[i]) / ||a[i] - b[i]||_2 (zero where the rows are equal)."""
    ap, lda = _mat(a)
    bp, ldb = _mat(b)
    gp, ldg = _mat(g)
    if a.shape != b.shape or g.shape != a.shape or not (a.dtype == b.dtype == g.dtype):
        raise ValueError("gas_row_distance_bwd: shapes or dtypes do not match")
    _check(_calls().gas_row_distance_bwd(ap, lda, bp, ldb, a.shape[0], a.shape[1], _dt(a),
                                      scale, gp, ldg, _stream()))


class HostTable:
    """A history table in pinned host memory, usable as the `hist` argument of gas_pull / gas_push: it carries
    the device-side address of the allocation and looks like a 2-D tensor to the marshalling code."""

    def __init__(self, t: torch.Tensor):
        if t.is_cuda or not t.is_pinned() or t.dim() != 2 or not t.is_contiguous():
            raise ValueError("HostTable: need a contiguous 2-D tensor in pinned host memory")
        dev = C.c_void_p(0)
        _check(_calls().gas_host_table_pointer(t.data_ptr(), C.byref(dev)))
        self.tensor, self._dev = t, dev.value
        self.shape, self.dtype = t.shape, t.dtype

    def data_ptr(self):
        return self._dev

    def dim(self):
        return 2

    def stride(self, *i):
        return self.tensor.stride(*i)


class DiskTable:
    """A history table in a file (gas_disk_* of the C ABI).  Index lists are int32 tensors or arrays in HOST memory;
    pull and push return a ticket and run beside the caller, wait(ticket) blocks until that transfer is complete.
    The tensors of a transfer are kept alive here until it has been waited for."""

    def __init__(self, path, n_rows, width, dtype, create=True, io_threads=0, staging_bytes=0, calls=False):
        self.shape, self.dtype, self.path = (int(n_rows), int(width)), dtype, path
        self._code = _dt(torch.empty(0, dtype=dtype))
        self._h = C.c_void_p(0)
        self._held = {}
        _check(_calls().gas_disk_open(os.fsencode(path), n_rows, width, self._code,
                                   (1 if create else 0) | (2 if calls else 0), io_threads,
                                   staging_bytes,
                                   C.byref(self._h)))

    def _idx(self, idx):
        if idx is None:
            return None, 0
        t = torch.as_tensor(idx)
        if t.is_cuda or t.dtype != torch.int32 or t.dim() != 1 or not t.is_contiguous():
            raise ValueError("DiskTable: idx must be a contiguous 1-D int32 tensor in host memory")
        return t, t.data_ptr()

    def _rows(self, t, n, device):
        if t.dtype != self.dtype or t.dim() != 2 or t.shape[1] != self.shape[1] or t.shape[0] < n \
                or t.is_cuda != device:
            raise ValueError("DiskTable: rows do not match the table")
        return _mat(t)

    def _transfer(self, fn, idx, base, n, rows):
        it, ip = self._idx(idx)
        n = (it.numel() if it is not None else rows.shape[0]) if n is None else n
        rp, ld = self._rows(rows, n, True)
        ticket = C.c_int64(0)
        _check(fn(self._h, ip, base, n, rp, ld, _stream(), C.byref(ticket)))
        self._held[ticket.value] = rows
        return ticket.value

    def pull(self, idx, dst, base=0, n=None) -> int:
        """dst[i] = table[idx[i]] (or table[base + i]); starts after the current stream's work so far."""
        return self._transfer(_calls().gas_disk_pull, idx, base, n, dst)

    def push(self, src, idx, base=0, n=None) -> int:
        """table[idx[i]] = src[i] (or table[base + i]); reads src after the current stream's work so far."""
        return self._transfer(_calls().gas_disk_push, idx, base, n, src)

    def wait(self, ticket=0):
        try:
            _check(_calls().gas_disk_wait(self._h, ticket))
        finally:
            for k in [k for k in self._held if ticket <= 0 or k <= ticket]:
                del self._held[k]

    def read_rows(self, dst, idx=None, base=0, n=None):
        it, ip = self._idx(idx)
        n = (it.numel() if it is not None else dst.shape[0]) if n is None else n
        rp, ld = self._rows(dst, n, False)
        _check(_calls().gas_disk_read_rows(self._h, ip, base, n, rp, ld))
        self._held.clear()

    def write_rows(self, src, idx=None, base=0, n=None):
        it, ip = self._idx(idx)
        n = (it.numel() if it is not None else src.shape[0]) if n is None else n
        rp, ld = self._rows(src, n, False)
        _check(_calls().gas_disk_write_rows(self._h, ip, base, n, rp, ld))
        self._held.clear()

    def sync(self):
        _check(_calls().gas_disk_sync(self._h))
        self._held.clear()

    def close(self):
        if self._h:
            h, self._h = self._h, C.c_void_p(0)
            self._held.clear()
            _check(_calls().gas_disk_close(h))

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass


def gas_pna_aggregate_bwd(rowptr, col, colptr, row, csc_pos, x, g, gx, delta, gadd=None, plan_t=None, blocks=9,
                          longest=ANY_LENGTH):
    """Backward of gas_pna_aggregate: gx [n_out, F] (n_out = gx.shape[0] columns of the pattern), gadd [n_rows, F]; g of nine
    blocks, or of blocks = 3, folded with their scalers.
    plan_t: a Plan of the CSC copy for those n_out columns (fast path), or None (plain kernels).  longest: no row has more entries."""
    xp, ldx = _mat(x)
    gp, ldg = _mat(g)
    op, ldo = _mat(gx)
    ap, lda = (0, 0) if gadd is None else _mat(gadd)
    n_rows, F = rowptr.numel() - 1, x.shape[1]
    if g.shape != (n_rows, blocks * F) or gx.shape[1] != F or g.dtype != x.dtype or gx.dtype != x.dtype:
        raise ValueError("gas_pna_aggregate_bwd: shapes or dtypes do not match")
    nnz = col.numel()
    nbytes = int(_calls().gas_pna_aggregate_bwd_workspace(n_rows, nnz, F))
    ws = torch.empty(max(nbytes, 1), dtype=torch.uint8, device=x.device)
    _check(_calls().gas_pna_aggregate_bwd_bounded(plan_t.handle if plan_t is not None else 0,
                                              _ptr(rowptr, torch.int32), _ptr(col, torch.int32), n_rows, longest,
                                              nnz, _ptr(colptr, torch.int32), _ptr(row, torch.int32), _ptr(csc_pos, torch.int32),
                                              gx.shape[0], xp, ldx, _dt(x), F, delta, blocks,
                                              gp, ldg, op, ldo, ap, lda, _ptr(ws), nbytes, _stream()))


def gas_gat_aggregate_bwd(rowptr, col, colptr, row, csc_pos, p, a_dst, a_src, gz, gp_out, ga_dst, ga_src,
                          negative_slope=0.2, plan_t=None, heads=1, longest=ANY_LENGTH, longest_col=ANY_LENGTH):
    """Backward of gas_gat_aggregate (gz: gradient before any activation): gp_out [n_out, F] rows of P's gradient,
    ga_dst / ga_src float32 [F].  plan_t: a Plan of the CSC copy for those n_out columns, or None; used where the heads are taken
    one by one (see gas.h).  heads > 1: as in gas_gat_aggregate.  No row has more than longest entries, no column longest_col."""
    pp, ldp = _mat(p)
    zp, ldz = _mat(gz)
    op, ldo = _mat(gp_out)
    n_rows, n_cols, F, nnz = rowptr.numel() - 1, p.shape[0], p.shape[1], col.numel()
    if gz.shape != (n_rows, F) or gp_out.shape[1] != F or colptr.numel() != n_cols + 1 or gz.dtype != p.dtype or \
            gp_out.dtype != p.dtype or ga_dst.dtype != torch.float32 or ga_src.dtype != torch.float32 or heads < 1 or F % heads:
        raise ValueError("gas_gat_aggregate_bwd: shapes or dtypes do not match")
    nbytes = int(_calls().gas_gat_aggregate_bwd_heads_workspace(n_rows, n_cols, nnz, F // heads, heads))
    ws = torch.empty(max(nbytes, 1), dtype=torch.uint8, device=p.device)
    _check(_calls().gas_gat_aggregate_bwd_bounded(plan_t.handle if plan_t is not None else 0,
                                                _ptr(rowptr, torch.int32), _ptr(col, torch.int32), n_rows, longest, longest_col,
                                                _ptr(colptr, torch.int32), _ptr(row, torch.int32), _ptr(csc_pos, torch.int32),
                                                n_cols, gp_out.shape[0], nnz, pp, ldp, _dt(p), F // heads, heads, _ptr(a_dst),
                                                _ptr(a_src), negative_slope, zp, ldz, op, ldo, _ptr(ga_dst), _ptr(ga_src),
                                                _ptr(ws), nbytes, _stream()))
