// Argument marshalling for binding.py: addresses, strides and sizes of tensors, and the C ABI's calls with plain Python
// numbers as arguments.  A small pass is bounded by what the host does between two launches: through ctypes and tensor
// attributes a call of 30 arguments over six matrices took 14 us, so 3.
//
// Only torch.Tensor itself (and Parameter) is read here; anything else (a table in host memory, a subclass, a tensor without
// memory of its own under a transform) goes to the Python functions that binding.py registers, which decide and raise as before.
#include <Python.h>

#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

#include <tuple>
#include <utility>

#include "gas.h"

namespace {

PyObject* slow_mat = nullptr;      // binding._mat_any
PyObject* slow_size = nullptr;     // binding._size_any
PyObject* slow_ptr = nullptr;      // binding._ptr_any

const at::Tensor* plain(PyObject* o) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || t.layout() != at::kStrided || !t.unsafeGetTensorImpl()->has_storage() ||
        t.unsafeGetTensorImpl()->key_set().has(c10::DispatchKey::Python) || t.unsafeGetTensorImpl()->is_python_dispatch())
        return nullptr;
    const at::DeviceType d = t.device().type();
    return d == at::kCUDA || d == at::kCPU ? &t : nullptr;
}

// Whether t is a matrix with contiguous rows; its row stride as the C ABI takes it.
bool matrix(const at::Tensor& t, int64_t* ld) {
    if (t.dim() != 2 || (t.size(1) > 1 && t.stride(1) != 1)) return false;
    *ld = t.size(0) > 1 ? t.stride(0) : std::max(t.stride(0), t.size(1));
    return true;
}

PyObject* mat(PyObject*, PyObject* o) {
    try {
        int64_t ld;
        const at::Tensor* t = plain(o);
        if (t && matrix(*t, &ld)) {
            PyObject* out = PyTuple_New(2);
            if (!out) return nullptr;
            PyTuple_SET_ITEM(out, 0, PyLong_FromVoidPtr(t->data_ptr()));
            PyTuple_SET_ITEM(out, 1, PyLong_FromLongLong(ld));
            return out;
        }
    } catch (...) {
    }
    return PyObject_CallOneArg(slow_mat, o);
}

// (pointer, row stride, rows, columns, dtype code) of a matrix of the feature types
PyObject* size(PyObject*, PyObject* o) {
    try {
        int64_t ld;
        const at::Tensor* t = plain(o);
        const at::ScalarType s = t ? t->scalar_type() : at::kDouble;
        if (t && (s == at::kFloat || s == at::kBFloat16) && matrix(*t, &ld)) {
            PyObject* out = PyTuple_New(5);
            if (!out) return nullptr;
            PyTuple_SET_ITEM(out, 0, PyLong_FromVoidPtr(t->data_ptr()));
            PyTuple_SET_ITEM(out, 1, PyLong_FromLongLong(ld));
            PyTuple_SET_ITEM(out, 2, PyLong_FromLongLong(t->size(0)));
            PyTuple_SET_ITEM(out, 3, PyLong_FromLongLong(t->size(1)));
            PyTuple_SET_ITEM(out, 4, PyLong_FromLong(s == at::kFloat ? GAS_F32 : GAS_BF16));
            return out;
        }
    } catch (...) {
    }
    return PyObject_CallOneArg(slow_size, o);
}

// ptr(t, dtype=None): the address of a contiguous tensor (of that type), 0 for None
PyObject* ptr(PyObject*, PyObject* const* args, Py_ssize_t n) {
    if (n >= 1 && n <= 2) {
        if (args[0] == Py_None) return PyLong_FromLong(0);
        try {
            const at::Tensor* t = plain(args[0]);
            const bool any = n == 1 || args[1] == Py_None;
            if (t && (any || (THPDtype_Check(args[1]) && reinterpret_cast<THPDtype*>(args[1])->scalar_type == t->scalar_type())) &&
                t->is_contiguous())
                return PyLong_FromVoidPtr(t->data_ptr());
        } catch (...) {
        }
    }
    return PyObject_Vectorcall(slow_ptr, args, n, nullptr);
}

// ---- calls
// A pointer argument: an address, None, a ctypes array (its memory) or a ctypes pointer (its value).
bool get(PyObject* o, uintptr_t* out) {
    if (PyLong_Check(o)) {
        *out = (uintptr_t)PyLong_AsUnsignedLongLong(o);
        return !(*out == (uintptr_t)-1 && PyErr_Occurred());
    }
    if (o == Py_None) {
        *out = 0;
        return true;
    }
    Py_buffer view;
    if (PyObject_GetBuffer(o, &view, PyBUF_FORMAT | PyBUF_ND) != 0) return false;
    const bool ok = view.ndim > 0 || view.itemsize == (Py_ssize_t)sizeof(void*);
    if (ok) *out = view.ndim > 0 ? (uintptr_t)view.buf : *(uintptr_t*)view.buf;
    PyBuffer_Release(&view);             // the argument's reference is the caller's and outlives the call
    if (!ok) PyErr_SetString(PyExc_TypeError, "expected an address");
    return ok;
}

template <class T>
bool convert(PyObject* o, T* out) {
    if constexpr (std::is_pointer_v<T>) {
        uintptr_t p;
        if (!get(o, &p)) return false;
        *out = reinterpret_cast<T>(p);
    } else if constexpr (std::is_floating_point_v<T>) {
        const double v = PyFloat_AsDouble(o);
        if (v == -1.0 && PyErr_Occurred()) return false;
        *out = (T)v;
    } else {
        const long long v = PyLong_AsLongLong(o);
        if (v == -1 && PyErr_Occurred()) return false;
        *out = (T)v;
        if ((long long)*out != v) {
            PyErr_SetString(PyExc_OverflowError, "an argument does not fit its type");
            return false;
        }
    }
    return true;
}

template <auto Fn, class R, class... A, size_t... I>
PyObject* invoke(R (*)(A...), PyObject* const* args, std::index_sequence<I...>) {
    std::tuple<A...> v;
    if (!(convert(args[I], &std::get<I>(v)) && ...)) return nullptr;
    PyThreadState* state = PyEval_SaveThread();          // a launch may wait for room in its queue
    const R r = std::apply(Fn, v);
    PyEval_RestoreThread(state);
    return PyLong_FromLongLong((long long)r);
}

template <class R, class... A>
constexpr size_t arity(R (*)(A...)) { return sizeof...(A); }

template <auto Fn>
PyObject* call(PyObject*, PyObject* const* args, Py_ssize_t n) {
    constexpr size_t want = arity(Fn);
    if (n != (Py_ssize_t)want) {
        PyErr_Format(PyExc_TypeError, "%zd arguments, the call takes %zu", n, want);
        return nullptr;
    }
    return invoke<Fn>(Fn, args, std::make_index_sequence<want>{});
}

PyObject* set_slow(PyObject*, PyObject* args) {
    PyObject *m, *s, *p;
    if (!PyArg_ParseTuple(args, "OOO", &m, &s, &p)) return nullptr;
    Py_INCREF(m); Py_INCREF(s); Py_INCREF(p);
    Py_XDECREF(slow_mat); Py_XDECREF(slow_size); Py_XDECREF(slow_ptr);
    slow_mat = m; slow_size = s; slow_ptr = p;
    Py_RETURN_NONE;
}

#define GAS_CALL(name) {#name, (PyCFunction)(void (*)())call<&name>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"mat", mat, METH_O, nullptr},
    {"size", size, METH_O, nullptr},
    {"ptr", (PyCFunction)(void (*)())ptr, METH_FASTCALL, nullptr},
    {"set_slow", set_slow, METH_VARARGS, nullptr},
    GAS_CALL(gas_pull), GAS_CALL(gas_push), GAS_CALL(gas_pull_host), GAS_CALL(gas_push_host), GAS_CALL(gas_gcn_norm),
    GAS_CALL(gas_spmm), GAS_CALL(gas_spmm_hist), GAS_CALL(gas_spmm_table), GAS_CALL(gas_fuse_sources), GAS_CALL(gas_spmm_t),
    GAS_CALL(gas_spmm_t_relu), GAS_CALL(gas_linear), GAS_CALL(gas_linear_in_order), GAS_CALL(gas_linear_push), GAS_CALL(gas_mlp2), GAS_CALL(gas_mlp2_push),
    GAS_CALL(gas_mlp2_keep), GAS_CALL(gas_spmm_linear), GAS_CALL(gas_spmm_t_relu_linear), GAS_CALL(gas_spmm_linear_layers),
    GAS_CALL(gas_spmm_t_relu_linear_layers), GAS_CALL(gas_relu_bwd), GAS_CALL(gas_linear_bwd_input),
    GAS_CALL(gas_linear_bwd_input_add), GAS_CALL(gas_linear_bwd_weight), GAS_CALL(gas_linear_bwd_weight_workspace),
    GAS_CALL(gas_linear_bwd_weights), GAS_CALL(gas_linear_bwd_weights_workspace), GAS_CALL(gas_softmax_xent),
    GAS_CALL(gas_sgd_step), GAS_CALL(gas_sgd_steps), GAS_CALL(gas_axpy), GAS_CALL(gas_row_dot),
    GAS_CALL(gas_pna_aggregate_own), GAS_CALL(gas_pna_aggregate_bwd_bounded), GAS_CALL(gas_pna_aggregate_bwd_workspace),
    GAS_CALL(gas_pna_groups), GAS_CALL(gas_pna_groups_workspace), GAS_CALL(gas_pna_linear), GAS_CALL(gas_pna_linear_workspace),
    GAS_CALL(gas_pna_linear_bwd_input), GAS_CALL(gas_pna_linear_bwd_weight), GAS_CALL(gas_pna_linear_bwd_weight_workspace),
    GAS_CALL(gas_gat_aggregate_push), GAS_CALL(gas_gat_aggregate_bwd_bounded), GAS_CALL(gas_gat_aggregate_bwd_heads_workspace),
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// built_for: the torch and the interpreter whose layouts were compiled in (_build.built_for); binding.py compares it with those it runs in.
PyMODINIT_FUNC PyInit__marshal() {
    PyObject* m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "built_for", GAS_BUILT_FOR) != 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
