// Argument tables of the ctypes binding (lowdiff.py): addresses, sizes and devices of a list of torch
// tensors in one call. A window of 50 diffs or the layers of a model are hundreds of tensors; asked
// one by one from Python for their type, layout, device, address and size they cost a microsecond each,
// more than the GPU work of the call (161 layers of ResNet-50: 163 us against 24 us of kernels).
// Nothing is checked here that is not checked by the caller: the first tensor that does not fit is
// reported by its index, and the binding raises.
#include <Python.h>

#include <string.h>

#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

namespace {

// gather(tensors, dtype, pinned) -> (addresses: bytes of uint64, sizes: bytes of int64, device, bad)
//   device  index of the device all tensors lie on, -1 for host memory, -2 when they differ or there are none
//   bad     index of the first tensor that is not contiguous, of `dtype` and on a GPU (with `pinned`: or in
//           page-locked host memory); -1 when there is none. Its address is left 0.
PyObject* gather(PyObject*, PyObject* args) {
    PyObject *list, *dtype;
    int pinned;
    if (!PyArg_ParseTuple(args, "OOp", &list, &dtype, &pinned)) return nullptr;
    if (!THPDtype_Check(dtype)) {
        PyErr_SetString(PyExc_TypeError, "gather: a torch.dtype expected");
        return nullptr;
    }
    const at::ScalarType want = reinterpret_cast<THPDtype*>(dtype)->scalar_type;
    PyObject* seq = PySequence_Fast(list, "a sequence of tensors expected");
    if (!seq) return nullptr;
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(seq);
    PyObject* addresses = PyBytes_FromStringAndSize(nullptr, n * 8);
    PyObject* sizes = PyBytes_FromStringAndSize(nullptr, n * 8);
    Py_ssize_t bad = -1;
    long device = -2;
    bool ok = addresses && sizes;
    if (ok) {
        char* at_address = PyBytes_AS_STRING(addresses);
        char* at_size = PyBytes_AS_STRING(sizes);
        try {
            for (Py_ssize_t i = 0; i < n && ok; ++i) {
                PyObject* item = PySequence_Fast_GET_ITEM(seq, i);
                if (!THPVariable_Check(item)) {
                    PyErr_SetString(PyExc_TypeError, "a torch tensor expected");
                    ok = false;
                    break;
                }
                const at::Tensor& t = THPVariable_Unpack(item);
                const bool gpu = t.is_cuda();
                const long dev = gpu ? static_cast<long>(t.get_device()) : -1;
                device = i == 0 ? dev : (device == dev ? device : -2);
                uint64_t address = 0;
                const bool fits = t.scalar_type() == want && t.is_contiguous() && (gpu || (pinned && t.is_pinned()));
                if (fits) address = reinterpret_cast<uint64_t>(t.data_ptr());
                else if (bad < 0) bad = i;
                const int64_t count = t.numel();
                memcpy(at_address + i * 8, &address, 8);
                memcpy(at_size + i * 8, &count, 8);
            }
        } catch (const std::exception& e) {
            PyErr_SetString(PyExc_RuntimeError, e.what());
            ok = false;
        }
    }
    Py_DECREF(seq);
    PyObject* result = ok ? Py_BuildValue("(OOln)", addresses, sizes, device, bad) : nullptr;
    Py_XDECREF(addresses);
    Py_XDECREF(sizes);
    return result;
}

PyMethodDef methods[] = {{"gather", gather, METH_VARARGS, "Addresses, sizes and device of a list of tensors."},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// Torch's classes are used here as its headers lay them out: a module built for another torch or another
// Python must not run. It fails to import, and the binding builds it anew or does without.
PyMODINIT_FUNC PyInit__marshal(void) {
    PyObject* torch = PyImport_ImportModule("torch");
    PyObject* version = torch ? PyObject_GetAttrString(torch, "__version__") : nullptr;
    PyObject* have = version ? PyObject_Str(version) : nullptr;
    const char* text = have ? PyUnicode_AsUTF8(have) : nullptr;
    const bool same = text && strcmp(text, LD_BUILT_FOR_TORCH) == 0 &&
                      strncmp(Py_GetVersion(), PY_VERSION, strlen(PY_VERSION)) == 0;
    PyErr_Clear();
    Py_XDECREF(torch);
    Py_XDECREF(version);
    Py_XDECREF(have);
    if (!same) {
        PyErr_SetString(PyExc_ImportError, "_marshal was built for torch " LD_BUILT_FOR_TORCH " and Python " PY_VERSION);
        return nullptr;
    }
    return PyModule_Create(&module);
}
