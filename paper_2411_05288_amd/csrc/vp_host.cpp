// Host side of the Python binding: the checks of the tensors of a call (on the GPU, contiguous, of the expected type and
// shape) and their addresses, and the current stream, without a Python call per property.  A pass over the input layer of 8
// shards of N=512 h=1024 hands over 28 tensors; their checks in Python took longer than its kernels: 30.3 us a pass with them,
// 15.5 us so.  N=98 h=128 V=2929 p=8 fp32 step: 85 -> 53 us.
//
// Every function returns None where a check fails or anything is unusual (a subclass of Tensor, a tensor without memory of its
// own): the caller then goes through the same checks in Python, which say what is wrong.  Nothing is kept between calls.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/version.h>

#include <cstdint>
#include <cstring>

namespace {

bool type_ok(const at::Tensor& t, PyObject* dtypes) {
    if (dtypes == Py_None) return true;
    if (!PyTuple_Check(dtypes)) return false;
    for (Py_ssize_t i = 0; i < PyTuple_GET_SIZE(dtypes); ++i) {
        PyObject* d = PyTuple_GET_ITEM(dtypes, i);
        if (THPDtype_Check(d) && reinterpret_cast<THPDtype*>(d)->scalar_type == t.scalar_type()) return true;
    }
    return false;
}

bool shape_ok(const at::Tensor& t, PyObject* shape) {
    if (shape == Py_None) return true;
    if (!PyTuple_Check(shape) || PyTuple_GET_SIZE(shape) != t.dim()) return false;
    for (int64_t i = 0; i < t.dim(); ++i) {
        const long long n = PyLong_AsLongLong(PyTuple_GET_ITEM(shape, i));
        if (n != t.size(i)) {
            PyErr_Clear();
            return false;
        }
    }
    return true;
}

// The address of the tensor's first element in `out`, if it passes all checks.
bool address(PyObject* o, PyObject* dtypes, PyObject* shape, uint64_t& out) {
    if (!THPVariable_CheckExact(o)) return false;
    try {
        const at::Tensor& t = THPVariable_Unpack(o);
        if (!t.defined() || !t.is_cuda() || !t.is_contiguous() || !type_ok(t, dtypes) || !shape_ok(t, shape)) return false;
        out = reinterpret_cast<uint64_t>(t.data_ptr());
        return true;
    } catch (...) {
        return false;
    }
}

// ptr(tensor, dtypes or None, shape or None) -> int
PyObject* ptr(PyObject*, PyObject* const* a, Py_ssize_t n) {
    uint64_t p;
    if (n != 3 || !address(a[0], a[1], a[2], p)) Py_RETURN_NONE;
    return PyLong_FromUnsignedLongLong(p);
}

// ptrs(list of tensors, dtypes or None, shape of each or list of their shapes) -> bytes: an array of pointers
PyObject* ptrs(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 3 || !PyList_Check(a[0])) Py_RETURN_NONE;
    const Py_ssize_t k = PyList_GET_SIZE(a[0]);
    const bool each = PyList_Check(a[2]);
    if (each && PyList_GET_SIZE(a[2]) != k) Py_RETURN_NONE;
    PyObject* out = PyBytes_FromStringAndSize(nullptr, k * (Py_ssize_t)sizeof(uint64_t));
    if (!out) return nullptr;
    for (Py_ssize_t i = 0; i < k; ++i) {
        uint64_t p;
        if (!address(PyList_GET_ITEM(a[0], i), a[1], each ? PyList_GET_ITEM(a[2], i) : a[2], p)) {
            Py_DECREF(out);
            Py_RETURN_NONE;
        }
        std::memcpy(PyBytes_AS_STRING(out) + i * sizeof(uint64_t), &p, sizeof p);
    }
    return out;
}

// same_shapes(list of tensors) -> bool
PyObject* same_shapes(PyObject*, PyObject* list) {
    if (!PyList_Check(list)) Py_RETURN_NONE;
    try {
        for (Py_ssize_t i = 0; i < PyList_GET_SIZE(list); ++i) {
            if (!THPVariable_CheckExact(PyList_GET_ITEM(list, i))) Py_RETURN_NONE;
            if (THPVariable_Unpack(PyList_GET_ITEM(list, i)).sizes() != THPVariable_Unpack(PyList_GET_ITEM(list, 0)).sizes())
                Py_RETURN_FALSE;
        }
    } catch (...) {
        Py_RETURN_NONE;
    }
    Py_RETURN_TRUE;
}

// stream() -> int: the current stream of the current device
PyObject* stream(PyObject*, PyObject*) {
    try {
        return PyLong_FromVoidPtr(reinterpret_cast<void*>(c10::hip::getCurrentHIPStream().stream()));
    } catch (...) {
        Py_RETURN_NONE;
    }
}

PyMethodDef methods[] = {
    {"ptr", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(ptr)), METH_FASTCALL, nullptr},
    {"ptrs", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(ptrs)), METH_FASTCALL, nullptr},
    {"same_shapes", same_shapes, METH_O, nullptr},
    {"stream", stream, METH_NOARGS, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_vphost", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__vphost(void) {
    PyObject* m = PyModule_Create(&module);
    // the PyTorch whose objects this code reads: another one's may be laid out otherwise
    if (m && PyModule_AddStringConstant(m, "torch_version", TORCH_VERSION) < 0) Py_CLEAR(m);
    return m;
}
