// The binding's calls that a training step or a decoding loop makes once per layer, without Python between the caller and
// the library: argument checks, the output's allocation and the library call in one C function.
//
// Why: a linear call spent 5.7 us in Python (1.8 of them in torch.empty) beside 2.6 us per kernel launch, more than many of
// these calls take on the GPU; here it spends about 2.  Only the plain case is handled -- exact torch.Tensor arguments that
// pass every check, and no torch mode that wants to see the allocations.  For anything else (a subclass, a wrong type, shape or
// device, an exception from torch) the functions return None with nothing launched, and lowra.py goes through its own checks,
// which raise what they always raised.  So every object that a call returns exists before the library is called.  The interpreter's
// lock is given up for the allocations too, as torch.empty does (one may wait for the GPU).  Nothing is kept between calls but
// the library's entry points.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

namespace {

typedef int (*linear_fn)(const void*, const void*, const void*, const void*, const void*, int, const void*, const void*, int, float, void*,
                         void*, size_t, void*);
typedef const void* (*side_fn)(const void*, int, int, int, const void*);
typedef int (*grads_fn)(const void*, const void*, const void*, int, const void*, const void*, int, float, void*, void*, void*, size_t, void*);
typedef int (*grads_side_fn)(const void*, const void*, const void*, int, int, const void*, const void*, void*, void*, void*, size_t, void*);
typedef int (*dequant_fn)(const void*, const void*, const void*, const void*, int, void*, void*);
linear_fn lib_linear[2];
side_fn lib_side;
grads_fn lib_grads;
grads_side_fn lib_grads_side;
dequant_fn lib_dequant;

// what a call needs of a layout, in the order of Layout.native (lowra.py)
struct Lay { const void* handle; int64_t N, K, C, packed_bytes; bool bf16_scales; };

bool layout_of(PyObject* o, Lay& l) {
    if (!PyTuple_CheckExact(o) || PyTuple_GET_SIZE(o) != 6) return false;
    l.handle = PyLong_AsVoidPtr(PyTuple_GET_ITEM(o, 0));
    l.N = PyLong_AsLongLong(PyTuple_GET_ITEM(o, 1));
    l.K = PyLong_AsLongLong(PyTuple_GET_ITEM(o, 2));
    l.C = PyLong_AsLongLong(PyTuple_GET_ITEM(o, 3));
    l.packed_bytes = PyLong_AsLongLong(PyTuple_GET_ITEM(o, 4));
    l.bf16_scales = PyTuple_GET_ITEM(o, 5) == Py_True;
    return l.handle != nullptr && !PyErr_Occurred();
}

// a plain, contiguous device tensor of this type, or null
const at::Tensor* plain(PyObject* o, at::ScalarType type) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    return t.scalar_type() == type && t.is_cuda() && t.is_contiguous() ? &t : nullptr;
}
bool shape2(const at::Tensor& t, int64_t a, int64_t b) { return t.dim() == 2 && t.size(0) == a && t.size(1) == b; }

bool state_ok(const Lay& l, const at::Tensor* packed, const at::Tensor* absmax, const at::Tensor* mappings) {
    return packed && absmax && mappings && packed->numel() == l.packed_bytes && absmax->numel() == l.N * (l.K / 64) && shape2(*mappings, l.C, 16);
}
bool modes() { return c10::impl::TorchDispatchModeTLS::any_modes_set() || at::impl::torch_function_mode_enabled(); }
void* current_stream() { return (void*)c10::hip::getCurrentHIPStream().stream(); }

PyObject* none() {
    PyErr_Clear();
    Py_RETURN_NONE;
}
// the interpreter's lock, given up for a scope
struct Unlocked {
    PyThreadState* const state = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(state); }
};
at::Tensor empty(at::IntArrayRef sizes, const at::TensorOptions& options) {
    Unlocked u;
    return at::empty(sizes, options);
}
// what the caller returns: the result, or the library's status when that is not zero
PyObject* done(int status, PyObject* result) {
    if (status == 0) return result;
    Py_DECREF(result);
    return PyLong_FromLong(status);
}

// linear(which, layout, packed, absmax, mappings, act, A, B, s, workspace): which = 0 forward, 1 input gradient
PyObject* linear(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 10) return none();
    try {
        if (modes()) return none();
        const long which = PyLong_AsLong(a[0]);
        Lay l;
        if ((which != 0 && which != 1) || !layout_of(a[1], l)) return none();
        const at::Tensor* packed = plain(a[2], at::kByte);
        const at::Tensor* absmax = plain(a[3], l.bf16_scales ? at::kBFloat16 : at::kFloat);
        const at::Tensor* mappings = plain(a[4], at::kFloat);
        const at::Tensor* act = plain(a[5], at::kBFloat16);
        const int64_t in = which ? l.N : l.K, cols = which ? l.K : l.N;
        if (!state_ok(l, packed, absmax, mappings) || !act || act->dim() != 2 || act->size(1) != in || !PyFloat_Check(a[8])) return none();
        const int64_t M = act->size(0);
        if (M > INT32_MAX) return none();
        const at::Tensor *A = nullptr, *B = nullptr;
        int64_t r = 0;
        if (a[6] != Py_None && a[7] != Py_None) {
            A = plain(a[6], at::kBFloat16); B = plain(a[7], at::kBFloat16);
            if (!A || !B || A->dim() != 2 || A->size(0) < 1) return none();
            r = A->size(0);
            if (r > INT32_MAX || A->size(1) != l.K || !shape2(*B, l.N, r)) return none();
        }
        if (!THPVariable_CheckExact(a[9])) return none();             // the caller's own workspace; the library checks its size
        const at::Tensor& ws = THPVariable_Unpack(a[9]);
        void* const wp = ws.data_ptr();
        const size_t ws_bytes = (size_t)ws.numel() * ws.element_size();
        const float s = (float)PyFloat_AS_DOUBLE(a[8]);
        at::Tensor out = empty({M, cols}, act->options());
        void *po = out.data_ptr(), *st = current_stream();
        const void *pp = packed->data_ptr(), *pa = absmax->data_ptr(), *pm = mappings->data_ptr(), *px = act->data_ptr();
        const void *pA = A ? A->data_ptr() : nullptr, *pB = B ? B->data_ptr() : nullptr;
        PyObject* res = THPVariable_Wrap(std::move(out));
        if (!res) return none();
        int status;
        {
            Unlocked u;
            status = lib_linear[which](l.handle, pp, pa, pm, px, (int)M, pA, pB, (int)r, s, po, wp, ws_bytes, st);
        }
        return done(status, res);
    } catch (...) {
        return none();
    }
}

// side_product(layout, op, M, r, workspace) -> (view,) or (None,)
PyObject* side_product(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 5) return none();
    try {
        if (modes()) return none();
        Lay l;
        if (!layout_of(a[0], l) || !PyLong_CheckExact(a[1]) || !PyLong_CheckExact(a[2]) || !PyLong_CheckExact(a[3])) return none();
        const long op = PyLong_AsLong(a[1]), M = PyLong_AsLong(a[2]), r = PyLong_AsLong(a[3]);
        const at::Tensor* ws = plain(a[4], at::kByte);
        if (PyErr_Occurred() || !ws || op != (int)op || M != (int)M || r != (int)r || ws->dim() != 1) return none();
        const uint8_t* base = static_cast<const uint8_t*>(ws->data_ptr());
        const uint8_t* p = static_cast<const uint8_t*>(lib_side(l.handle, (int)op, (int)M, (int)r, base));
        if (!p) return PyTuple_Pack(1, Py_None);
        const int64_t off = p - base, bytes = (int64_t)M * 128;
        if (off < 0 || off + bytes > ws->numel()) return none();
        PyObject* v = THPVariable_Wrap(ws->narrow(0, off, bytes).view(at::kBFloat16).view({M, 64}));
        if (!v) return none();
        PyObject* t = PyTuple_Pack(1, v);
        Py_DECREF(v);
        return t;
    } catch (...) {
        return none();
    }
}

PyObject* pair(at::Tensor dA, at::Tensor dB) {
    PyObject* x = THPVariable_Wrap(std::move(dA));
    PyObject* y = x ? THPVariable_Wrap(std::move(dB)) : nullptr;
    PyObject* t = y ? PyTuple_Pack(2, x, y) : nullptr;
    Py_XDECREF(x);
    Py_XDECREF(y);
    return t;
}

// grads(layout, x, dY, A, B, s, workspace)
PyObject* grads(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 7) return none();
    try {
        if (modes()) return none();
        Lay l;
        if (!layout_of(a[0], l) || !PyFloat_Check(a[5])) return none();
        const at::Tensor *x = plain(a[1], at::kBFloat16), *dY = plain(a[2], at::kBFloat16), *A = plain(a[3], at::kBFloat16), *B = plain(a[4], at::kBFloat16);
        const at::Tensor* ws = plain(a[6], at::kByte);
        if (!x || !dY || !A || !B || !ws || x->dim() != 2 || A->dim() != 2) return none();
        const int64_t M = x->size(0), r = A->size(0);
        if (M > INT32_MAX || r > INT32_MAX || !shape2(*x, M, l.K) || !shape2(*dY, M, l.N) || !shape2(*A, r, l.K) || !shape2(*B, l.N, r)) return none();
        const auto opt = x->options().dtype(at::kFloat);
        at::Tensor dA = empty({r, l.K}, opt), dB = empty({l.N, r}, opt);
        const void *px = x->data_ptr(), *py = dY->data_ptr(), *pA = A->data_ptr(), *pB = B->data_ptr();
        void *qa = dA.data_ptr(), *qb = dB.data_ptr(), *wp = ws->data_ptr(), *st = current_stream();
        const size_t ws_bytes = (size_t)ws->numel();
        const float s = (float)PyFloat_AS_DOUBLE(a[5]);
        PyObject* res = pair(std::move(dA), std::move(dB));
        if (!res) return none();
        int status;
        {
            Unlocked u;
            status = lib_grads(l.handle, px, py, (int)M, pA, pB, (int)r, s, qa, qb, wp, ws_bytes, st);
        }
        return done(status, res);
    } catch (...) {
        return none();
    }
}

// grads_from_side(layout, x, dY, r, st, su, workspace)
PyObject* grads_from_side(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 7) return none();
    try {
        if (modes()) return none();
        Lay l;
        if (!layout_of(a[0], l) || !PyLong_CheckExact(a[3])) return none();
        const int64_t r = PyLong_AsLongLong(a[3]);
        const at::Tensor *x = plain(a[1], at::kBFloat16), *dY = plain(a[2], at::kBFloat16), *ts = plain(a[4], at::kBFloat16), *us = plain(a[5], at::kBFloat16);
        const at::Tensor* ws = plain(a[6], at::kByte);
        if (PyErr_Occurred() || !x || !dY || !ts || !us || !ws || x->dim() != 2 || r < 0 || r > INT32_MAX) return none();
        const int64_t M = x->size(0);
        if (M > INT32_MAX || !shape2(*x, M, l.K) || !shape2(*dY, M, l.N) || !shape2(*ts, M, 64) || !shape2(*us, M, 64)) return none();
        const auto opt = x->options().dtype(at::kFloat);
        at::Tensor dA = empty({r, l.K}, opt), dB = empty({l.N, r}, opt);
        const void *px = x->data_ptr(), *py = dY->data_ptr(), *pt = ts->data_ptr(), *pu = us->data_ptr();
        void *qa = dA.data_ptr(), *qb = dB.data_ptr(), *wp = ws->data_ptr(), *st = current_stream();
        const size_t ws_bytes = (size_t)ws->numel();
        PyObject* res = pair(std::move(dA), std::move(dB));
        if (!res) return none();
        int status;
        {
            Unlocked u;
            status = lib_grads_side(l.handle, px, py, (int)M, (int)r, pt, pu, qa, qb, wp, ws_bytes, st);
        }
        return done(status, res);
    } catch (...) {
        return none();
    }
}

// dequantize(layout, packed, absmax, mappings): bf16
PyObject* dequantize(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 4) return none();
    try {
        if (modes()) return none();
        Lay l;
        if (!layout_of(a[0], l)) return none();
        const at::Tensor* packed = plain(a[1], at::kByte);
        const at::Tensor* absmax = plain(a[2], l.bf16_scales ? at::kBFloat16 : at::kFloat);
        const at::Tensor* mappings = plain(a[3], at::kFloat);
        if (!state_ok(l, packed, absmax, mappings)) return none();
        at::Tensor out = empty({l.N, l.K}, packed->options().dtype(at::kBFloat16));
        const void *pp = packed->data_ptr(), *pa = absmax->data_ptr(), *pm = mappings->data_ptr();
        void *po = out.data_ptr(), *st = current_stream();
        PyObject* res = THPVariable_Wrap(std::move(out));
        if (!res) return none();
        int status;
        {
            Unlocked u;
            status = lib_dequant(l.handle, pp, pa, pm, 0, po, st);
        }
        return done(status, res);
    } catch (...) {
        return none();
    }
}

// init(addresses): the library's entry points, in the order of lowra.py
PyObject* init(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 6) { PyErr_SetString(PyExc_TypeError, "init: six addresses"); return nullptr; }
    void* f[6];
    for (int i = 0; i < 6; ++i) f[i] = PyLong_AsVoidPtr(a[i]);
    if (PyErr_Occurred()) return nullptr;
    lib_linear[0] = (linear_fn)f[0]; lib_linear[1] = (linear_fn)f[1]; lib_side = (side_fn)f[2];
    lib_grads = (grads_fn)f[3]; lib_grads_side = (grads_side_fn)f[4]; lib_dequant = (dequant_fn)f[5];
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"init", (PyCFunction)(void (*)())init, METH_FASTCALL, nullptr},
                         {"linear", (PyCFunction)(void (*)())linear, METH_FASTCALL, nullptr},
                         {"side_product", (PyCFunction)(void (*)())side_product, METH_FASTCALL, nullptr},
                         {"grads", (PyCFunction)(void (*)())grads, METH_FASTCALL, nullptr},
                         {"grads_from_side", (PyCFunction)(void (*)())grads_from_side, METH_FASTCALL, nullptr},
                         {"dequantize", (PyCFunction)(void (*)())dequantize, METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_lowra_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__lowra_call() { return PyModule_Create(&module); }
