// Argument marshalling of binding.py: tensors to addresses.
//
// A call of the package hands over 5 to 60 tensors; in Python an address costs about 0.7 us (two checks, the address, a store
// into a ctypes field), which set the pace of calls whose kernels are short: the eight argument blocks of four packed
// minibatches took 190 us of host time for 47 us of kernels.  Here it costs about 30 ns.  Tensors only in the exact sense; any
// other object (a subclass, a look-alike) goes through the Python function that was given to init(), as does a
// tensor whose address cannot be taken, so that the error is Python's own.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstring>

namespace {

PyObject* g_any = nullptr;   // Python: address of anything else

// The address as an integer in *out; 0 with a Python error set.
bool address_of(PyObject* o, unsigned long long* out) {
    if (o == Py_None) {
        *out = 0;
        return true;
    }
    if (THPVariable_CheckExact(o)) {
        try {
            const at::Tensor& t = THPVariable_Unpack(o);
            if (t.is_cuda() && t.is_contiguous()) {
                *out = reinterpret_cast<unsigned long long>(t.data_ptr());
                return true;
            }
        } catch (...) {   // (the Python function raises what there is to raise)
        }
    }
    PyObject* r = PyObject_CallFunctionObjArgs(g_any, o, nullptr);
    if (!r) return false;
    *out = r == Py_None ? 0 : PyLong_AsUnsignedLongLong(r);
    Py_DECREF(r);
    return !PyErr_Occurred();
}

PyObject* init(PyObject*, PyObject* any) {
    Py_INCREF(any);
    Py_XDECREF(g_any);
    g_any = any;
    Py_RETURN_NONE;
}

// ptr(tensor or None) -> address or None
PyObject* ptr(PyObject*, PyObject* o) {
    if (o == Py_None) Py_RETURN_NONE;
    unsigned long long p;
    if (!address_of(o, &p)) return nullptr;
    return PyLong_FromUnsignedLongLong(p);
}

// fill(buffer, tensors): the addresses of a list or tuple of tensors, 8 bytes each, into a writable buffer
PyObject* fill(PyObject*, PyObject* const* args, Py_ssize_t n) {
    if (n != 2) return PyErr_Format(PyExc_TypeError, "fill(buffer, tensors)");
    PyObject* seq = PySequence_Tuple(args[1]);   // (a copy: an object's own address function could change the list)
    if (!seq) return nullptr;
    Py_buffer b;
    if (PyObject_GetBuffer(args[0], &b, PyBUF_WRITABLE) != 0) {
        Py_DECREF(seq);
        return nullptr;
    }
    bool ok = PyTuple_GET_SIZE(seq) * 8 <= b.len;
    if (!ok) PyErr_SetString(PyExc_ValueError, "buffer too short");
    for (Py_ssize_t i = 0; ok && i < PyTuple_GET_SIZE(seq); ++i) {
        unsigned long long p;
        ok = address_of(PyTuple_GET_ITEM(seq, i), &p);
        if (ok) std::memcpy(static_cast<char*>(b.buf) + i * 8, &p, 8);
    }
    PyBuffer_Release(&b);
    Py_DECREF(seq);
    if (!ok) return nullptr;
    Py_RETURN_NONE;
}

// pointers(struct, offsets, values): for every name in the dict `values` that `offsets` knows (a pointer field's offset in the
// struct) and whose value is exactly a tensor, the address goes into the struct; the names that are left come back as a list.
PyObject* pointers(PyObject*, PyObject* const* args, Py_ssize_t n) {
    if (n != 3 || !PyDict_Check(args[1]) || !PyDict_Check(args[2])) return PyErr_Format(PyExc_TypeError, "pointers(struct, offsets, values)");
    Py_buffer b;
    if (PyObject_GetBuffer(args[0], &b, PyBUF_WRITABLE) != 0) return nullptr;
    PyObject* left = PyList_New(0);
    PyObject *name, *value;
    Py_ssize_t at = 0;
    bool ok = left != nullptr;
    while (ok && PyDict_Next(args[2], &at, &name, &value)) {
        PyObject* offset = THPVariable_CheckExact(value) ? PyDict_GetItemWithError(args[1], name) : nullptr;
        if (!offset) {
            ok = !PyErr_Occurred() && PyList_Append(left, name) == 0;
            continue;
        }
        unsigned long long p;
        const Py_ssize_t o = PyLong_AsSsize_t(offset);
        ok = address_of(value, &p);
        if (ok && (o < 0 || o + 8 > b.len)) {
            PyErr_SetString(PyExc_ValueError, "offset beyond the struct");
            ok = false;
        }
        if (ok) std::memcpy(static_cast<char*>(b.buf) + o, &p, 8);
    }
    PyBuffer_Release(&b);
    if (!ok) {
        Py_XDECREF(left);
        return nullptr;
    }
    return left;
}

PyMethodDef methods[] = {
    {"init", init, METH_O, nullptr},
    {"ptr", ptr, METH_O, nullptr},
    {"fill", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(fill)), METH_FASTCALL, nullptr},
    {"pointers", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(pointers)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&module); }
