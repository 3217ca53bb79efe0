// Extension module _cgx_args: the checks the binding makes on every tensor argument, and its address.
//
// Written against the Python objects a check costs half a microsecond per tensor, and a reduction of 8 chunks has 17 of
// them: with the rest of the marshalling 20 us per call where the launch itself takes 3.  A tensor that fails a check
// (or is anything but a plain tensor with storage) is reported as such and looked at again in Python, which words
// the error.  The module also tells whether the arrays of a plan still hold what a size was worked out from.
#define PY_SSIZE_T_CLEAN
#include <torch/csrc/autograd/python_variable.h>

#include <cstring>

namespace {

// Element types by the numbers the binding passes: any, float32, float16, float64.
bool type_matches(c10::ScalarType type, long code)
{
    switch (code) {
    case 0: return true;
    case 1: return type == c10::ScalarType::Float;
    case 2: return type == c10::ScalarType::Half;
    case 3: return type == c10::ScalarType::Double;
    default: return false;
    }
}

// Address of a contiguous device tensor of the type with at least nbytes bytes; false: not that, or not to be decided here.
bool address_of(PyObject *obj, long long nbytes, long code, void **out)
{
    if (!THPVariable_CheckExact(obj)) return false;
    try {
        const at::Tensor &t = THPVariable_Unpack(obj);
        if (!t.defined() || t.layout() != c10::kStrided || !t.has_storage() || !t.is_cuda() || !t.is_contiguous() ||
            !type_matches(t.scalar_type(), code) || static_cast<long long>(t.nbytes()) < nbytes)
            return false;
        *out = t.mutable_data_ptr();
        return true;
    } catch (...) {
        return false;
    }
}

// address(tensor, nbytes, type) -> int, or None
PyObject *address(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != 3) {
        PyErr_SetString(PyExc_TypeError, "address(tensor, nbytes, type)");
        return nullptr;
    }
    const long long nbytes = PyLong_AsLongLong(args[1]);
    const long code = PyLong_AsLong(args[2]);
    if (PyErr_Occurred()) return nullptr;
    void *p = nullptr;
    if (!address_of(args[0], nbytes, code, &p)) Py_RETURN_NONE;
    return PyLong_FromVoidPtr(p);
}

// tables(packed, meta, packed_bytes, meta_bytes) -> (addresses of the packed tensors, of the float32 meta tensors), each
// as the bytes of a C array of pointers, or None
PyObject *tables(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != 4) {
        PyErr_SetString(PyExc_TypeError, "tables(packed, meta, packed_bytes, meta_bytes)");
        return nullptr;
    }
    const long long packed_bytes = PyLong_AsLongLong(args[2]), meta_bytes = PyLong_AsLongLong(args[3]);
    if (PyErr_Occurred()) return nullptr;
    // (other sequences go through Python)
    if (!(PyList_Check(args[0]) || PyTuple_Check(args[0])) || !(PyList_Check(args[1]) || PyTuple_Check(args[1]))) Py_RETURN_NONE;
    const Py_ssize_t count = PySequence_Fast_GET_SIZE(args[0]);
    constexpr Py_ssize_t kMost = 64;
    if (count < 1 || count > kMost || PySequence_Fast_GET_SIZE(args[1]) != count) Py_RETURN_NONE;
    void *packed[kMost], *meta[kMost];
    for (Py_ssize_t i = 0; i < count; i++)
        if (!address_of(PySequence_Fast_GET_ITEM(args[1], i), meta_bytes, 1, &meta[i]) ||
            !address_of(PySequence_Fast_GET_ITEM(args[0], i), packed_bytes, 0, &packed[i]))
            Py_RETURN_NONE;
    const Py_ssize_t bytes = count * Py_ssize_t(sizeof(void *));
    return Py_BuildValue("(y#y#)", reinterpret_cast<const char *>(packed), bytes, reinterpret_cast<const char *>(meta), bytes);
}

// unchanged((address, bytes, address, bytes, ...)) -> whether the memory at every address still holds the bytes beside it
PyObject *unchanged(PyObject *, PyObject *pairs)
{
    if (!PyTuple_Check(pairs) || PyTuple_GET_SIZE(pairs) % 2) {
        PyErr_SetString(PyExc_TypeError, "unchanged((address, bytes, ...))");
        return nullptr;
    }
    for (Py_ssize_t i = 0; i < PyTuple_GET_SIZE(pairs); i += 2) {
        const void *at = PyLong_AsVoidPtr(PyTuple_GET_ITEM(pairs, i));
        if (PyErr_Occurred()) return nullptr;
        PyObject *held = PyTuple_GET_ITEM(pairs, i + 1);
        if (!PyBytes_Check(held)) {
            PyErr_SetString(PyExc_TypeError, "unchanged((address, bytes, ...))");
            return nullptr;
        }
        const size_t bytes = size_t(PyBytes_GET_SIZE(held));
        if (bytes && std::memcmp(at, PyBytes_AS_STRING(held), bytes) != 0) Py_RETURN_FALSE;
    }
    Py_RETURN_TRUE;
}

PyMethodDef methods[] = {
    {"address", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(address)), METH_FASTCALL, nullptr},
    {"tables", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(tables)), METH_FASTCALL, nullptr},
    {"unchanged", unchanged, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_cgx_args", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__cgx_args(void) { return PyModule_Create(&module); }
