// The binding's small calls in native code.  One token's projection takes 4.1 us on the GPU and took 5.3 on the host (4096 x 4096 int4), of
// which 3 went into reading the tensors' attributes one by one from Python and converting thirteen arguments; here they are read from the
// tensors themselves.  Only what needs no decision is done here: tensors of the plain types, all buffers given.  Anything else -- missing
// buffers, wrong types, subclasses, a tensor without storage -- returns None, and the Python code beside the call takes it from the start
// and raises what there is to raise.
#include <Python.h>
#include <ATen/core/Tensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/rtn.h"

namespace {

decltype(&rtn_linear) linear_fn = nullptr;
decltype(&rtn_linear_asym) asym_fn = nullptr;

bool plain(PyObject* o) {
    return Py_TYPE(o) == reinterpret_cast<PyTypeObject*>(THPVariableClass) || Py_TYPE(o) == reinterpret_cast<PyTypeObject*>(ParameterClass);
}

// (A, qweight, scales[, zeros], bits, group_size, out, workspace) -> status, or None
PyObject* call(PyObject* const* args, bool zp) {
    const int extra = zp ? 1 : 0;
    PyObject *const pa = args[0], *const pq = args[1], *const ps = args[2], *const pz = args[2 + extra], *const pbits = args[3 + extra],
             *const pg = args[4 + extra], *const pc = args[5 + extra], *const pw = args[6 + extra];
    for (PyObject* t : {pa, pq, ps, pz, pc, pw})
        if (!plain(t)) Py_RETURN_NONE;
    if (!PyLong_CheckExact(pbits) || !PyLong_CheckExact(pg)) Py_RETURN_NONE;
    const long bits = PyLong_AsLong(pbits), g = PyLong_AsLong(pg);
    if (PyErr_Occurred()) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    if (bits != (int)bits || g != (int)g) Py_RETURN_NONE;
    const void *da, *dq, *ds, *dz = nullptr;
    void *dc, *dw, *stream;
    int64_t M, N, K;
    size_t bytes;
    try {
        const at::Tensor &a = THPVariable_Unpack(pa), &q = THPVariable_Unpack(pq), &s = THPVariable_Unpack(ps), &c = THPVariable_Unpack(pc),
                         &w = THPVariable_Unpack(pw);
        if (!a.is_cuda() || a.scalar_type() != at::kHalf || a.dim() != 2 || !a.is_contiguous() || s.dim() < 1) Py_RETURN_NONE;
        da = a.data_ptr(); dq = q.data_ptr(); ds = s.data_ptr(); dc = c.data_ptr(); dw = w.data_ptr();
        if (zp) dz = THPVariable_Unpack(pz).data_ptr();
        M = a.size(0); K = a.size(1); N = s.size(0);
        bytes = zp ? (size_t)w.numel() : w.nbytes();
        stream = c10::hip::getCurrentHIPStream().stream();
    } catch (...) {                                       // no storage to point to
        Py_RETURN_NONE;
    }
    rtn_status st;
    Py_BEGIN_ALLOW_THREADS
    st = zp ? asym_fn(da, M, dq, ds, dz, N, K, (int)bits, (int)g, dc, dw, bytes, stream)
            : linear_fn(da, M, dq, ds, N, K, (int)bits, (int)g, dc, dw, bytes, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong((long)st);
}

PyObject* linear(PyObject*, PyObject* const* args, Py_ssize_t n) {
    if (n != 7 || !linear_fn) Py_RETURN_NONE;
    return call(args, false);
}

PyObject* linear_asym(PyObject*, PyObject* const* args, Py_ssize_t n) {
    if (n != 8 || !asym_fn) Py_RETURN_NONE;
    return call(args, true);
}

// bind(rtn_linear, rtn_linear_asym): their addresses in the loaded library
PyObject* bind(PyObject*, PyObject* const* args, Py_ssize_t n) {
    if (n != 2) {
        PyErr_SetString(PyExc_TypeError, "bind takes two addresses");
        return nullptr;
    }
    void* const f = PyLong_AsVoidPtr(args[0]);
    void* const h = PyErr_Occurred() ? nullptr : PyLong_AsVoidPtr(args[1]);
    if (PyErr_Occurred()) return nullptr;
    linear_fn = reinterpret_cast<decltype(linear_fn)>(f);
    asym_fn = reinterpret_cast<decltype(asym_fn)>(h);
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"linear", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(linear)), METH_FASTCALL, nullptr},
    {"linear_asym", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(linear_asym)), METH_FASTCALL, nullptr},
    {"bind", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(bind)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// built_for: the PyTorch and Python of this build
PyMODINIT_FUNC PyInit__native() {
    PyObject* const m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "built_for", RTN_BUILT_FOR) != 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
