// Python side of a call: tensors to device addresses, and the whole of the two smallest products.
//
// A product of a few thousand entries takes 3.3 us on the device and in the runtime, 3.9 as a whole; looking at six tensors from Python
// (device, type, stride, address) and passing fifteen arguments through ctypes took 2.5 us more (6.4).  Here a plain tensor is looked at
// through its C++ object.  Whatever is not plain (a subclass, another device or type, no storage, a stride) goes to the
// Python function given to use(), which raises or converts as it always did.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

#include <stdint.h>

namespace {

PyObject *slow = nullptr, *current = nullptr;

// Address of a plain CUDA tensor of the given type (Undefined: any); false: not plain.
bool address(PyObject *o, at::ScalarType type, void **out)
{
    if (o == Py_None) { *out = nullptr; return true; }
    if (!THPVariable_CheckExact(o)) return false;
    try {
        const at::Tensor &t = THPVariable_Unpack(o);
        if (!t.is_cuda() || (type != at::ScalarType::Undefined && t.scalar_type() != type) || t.dim() == 0 || t.stride(-1) != 1) return false;
        *out = t.data_ptr();
        return true;
    } catch (...) {
        return false;
    }
}

// What int() and ctypes make of it: the low bits.
bool integer(PyObject *o, int64_t *out)
{
    if (PyLong_CheckExact(o)) {
        *out = (int64_t)PyLong_AsUnsignedLongLongMask(o);
        return !PyErr_Occurred();
    }
    PyObject *l = PyNumber_Long(o);
    if (!l) return false;
    *out = (int64_t)PyLong_AsUnsignedLongLongMask(l);
    Py_DECREF(l);
    return !PyErr_Occurred();
}

// ptr(tensor or None, dtype=None) -> int or None
PyObject *py_ptr(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n < 1 || n > 2) { PyErr_SetString(PyExc_TypeError, "ptr(tensor, dtype=None)"); return nullptr; }
    if (args[0] == Py_None) Py_RETURN_NONE;
    const bool any = n < 2 || args[1] == Py_None;
    if (any || THPDtype_Check(args[1])) {
        void *p;
        if (address(args[0], any ? at::ScalarType::Undefined : reinterpret_cast<THPDtype *>(args[1])->scalar_type, &p))
            return PyLong_FromUnsignedLongLong(reinterpret_cast<uintptr_t>(p));
    }
    return PyObject_CallFunctionObjArgs(slow, args[0], n < 2 ? Py_None : args[1], nullptr);
}

// spmv(f64, function, rows, cols, nnz, pos, crd, vals, x, y, tile, col_passes, phases, ws, stream or None) -> status, or None: not plain
typedef int (*spmv_t)(int64_t, int64_t, int64_t, const int32_t *, const int32_t *, const void *, const void *, void *, int32_t, int32_t, int,
                      void *, size_t, void *);
PyObject *py_spmv(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 15) { PyErr_SetString(PyExc_TypeError, "spmv takes 15 arguments"); return nullptr; }
    int64_t f64, fn, rows, cols, nnz, tile, passes, phases, stream;
    if (!integer(a[0], &f64) || !integer(a[1], &fn) || !integer(a[2], &rows) || !integer(a[3], &cols) || !integer(a[4], &nnz) ||
        !integer(a[10], &tile) || !integer(a[11], &passes) || !integer(a[12], &phases))
        return nullptr;
    const at::ScalarType vt = f64 ? at::ScalarType::Double : at::ScalarType::Float;
    void *pos, *crd, *vals, *x, *y, *ws;
    if (a[13] == Py_None || !address(a[5], at::ScalarType::Int, &pos) || !address(a[6], at::ScalarType::Int, &crd) || !address(a[7], vt, &vals) ||
        !address(a[8], vt, &x) || !address(a[9], vt, &y) || !address(a[13], at::ScalarType::Undefined, &ws))
        Py_RETURN_NONE;
    PyObject *const which = a[14] == Py_None ? PyObject_CallNoArgs(current) : Py_NewRef(a[14]);
    if (!which) return nullptr;
    const bool known = integer(which, &stream);
    Py_DECREF(which);
    if (!known) return nullptr;
    const size_t bytes = (size_t)THPVariable_Unpack(a[13]).numel();
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = reinterpret_cast<spmv_t>((uintptr_t)fn)(rows, cols, nnz, static_cast<int32_t *>(pos), static_cast<int32_t *>(crd), vals, x, y,
                                                 (int32_t)tile, (int32_t)passes, (int)phases, ws, bytes,
                                                 reinterpret_cast<void *>((uintptr_t)stream));
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
}

PyObject *py_use(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != 2) { PyErr_SetString(PyExc_TypeError, "use(slow, current)"); return nullptr; }
    Py_INCREF(args[0]);
    Py_XSETREF(slow, args[0]);
    Py_INCREF(args[1]);
    Py_XSETREF(current, args[1]);
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"ptr", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(py_ptr)), METH_FASTCALL, "device address of a tensor"},
    {"spmv", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(py_spmv)), METH_FASTCALL, "psk_spmv_csr or psk_spmv_csr_f64 on tensors"},
    {"use", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(py_use)), METH_FASTCALL, "the function for what is not a plain tensor, the current stream"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void)
{
    PyObject *m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "built_for", PSK_BUILT_FOR) < 0) Py_CLEAR(m);      // the torch and Python whose headers these are
    return m;
}
