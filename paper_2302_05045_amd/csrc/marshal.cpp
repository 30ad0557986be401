// Argument marshalling of the Python binding in native code: a tensor argument's checks and its device
// pointer in one call.  In Python the same checks are eight attribute reads, about 1 us per tensor, and an
// entry point takes up to seven tensors: more host time than the kernel of a small layer runs.
// Nothing but reads of tensor metadata happens here.  Whatever is not a plain torch.Tensor or Parameter (subclasses
// may override attributes, other objects have to be refused) goes to the Python function that makes the
// same checks, given once by use().
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

namespace {

PyObject *must_be(PyObject *name, const char *what)
{
    return PyErr_Format(PyExc_TypeError, "%U must be %s", name, what);
}

PyObject *pointer_or_none(const at::Tensor &t)
{
    if (t.numel() == 0) Py_RETURN_NONE;
    return PyLong_FromVoidPtr(t.data_ptr());
}

PyObject *python_vector = nullptr, *python_matrix = nullptr;

// vector(tensor, dtype, name[, length]): device pointer of a contiguous 1-D GPU tensor of that dtype with at least
// `length` elements (None: any number); None for None and for an empty tensor.
PyObject *vector(PyObject *, PyObject *const *args, Py_ssize_t count)
{
    HANDLE_TH_ERRORS
    if (count < 3 || count > 4) {
        PyErr_SetString(PyExc_TypeError, "vector(tensor, dtype, name[, length])");
        return nullptr;
    }
    if (args[0] == Py_None) Py_RETURN_NONE;
    if (!THPVariable_CheckExact(args[0]) || !THPDtype_Check(args[1]) || !PyUnicode_Check(args[2]))
        return PyObject_Vectorcall(python_vector, args, (size_t)count, nullptr);
    const at::Tensor &t = THPVariable_Unpack(args[0]);
    if (!t.is_cuda()) return must_be(args[2], "a tensor on the GPU");
    if (t.scalar_type() != reinterpret_cast<THPDtype *>(args[1])->scalar_type || t.dim() != 1 || !t.is_contiguous())
        return PyErr_Format(PyExc_TypeError, "%U must be a contiguous 1-D %S tensor", args[2], args[1]);
    if (count == 4 && args[3] != Py_None) {
        const long long length = PyLong_AsLongLong(args[3]);
        if (length == -1 && PyErr_Occurred()) return nullptr;
        if (t.numel() < length)
            return PyErr_Format(PyExc_ValueError, "%U holds %lld elements, needs %lld", args[2], (long long)t.numel(), length);
    }
    return pointer_or_none(t);
    END_HANDLE_TH_ERRORS
}

// matrix(tensor, name): (device pointer, rows, columns) of a contiguous 2-D float16 GPU tensor.
PyObject *matrix(PyObject *, PyObject *const *args, Py_ssize_t count)
{
    HANDLE_TH_ERRORS
    if (count != 2) {
        PyErr_SetString(PyExc_TypeError, "matrix(tensor, name)");
        return nullptr;
    }
    if (!THPVariable_CheckExact(args[0]) || !PyUnicode_Check(args[1]))
        return PyObject_Vectorcall(python_matrix, args, (size_t)count, nullptr);
    const at::Tensor &t = THPVariable_Unpack(args[0]);
    if (!t.is_cuda()) return must_be(args[1], "a tensor on the GPU");
    if (t.scalar_type() != at::kHalf || t.dim() != 2 || !t.is_contiguous())
        return must_be(args[1], "a contiguous 2-D float16 tensor");
    PyObject *pointer = pointer_or_none(t);
    if (!pointer) return nullptr;
    return Py_BuildValue("NLL", pointer, (long long)t.size(0), (long long)t.size(1));
    END_HANDLE_TH_ERRORS
}

// use(vector, matrix): the Python functions for everything that is no plain tensor.
PyObject *use(PyObject *, PyObject *const *args, Py_ssize_t count)
{
    if (count != 2 || !PyCallable_Check(args[0]) || !PyCallable_Check(args[1])) {
        PyErr_SetString(PyExc_TypeError, "use(vector, matrix)");
        return nullptr;
    }
    Py_INCREF(args[0]);
    Py_INCREF(args[1]);
    Py_XDECREF(python_vector);
    Py_XDECREF(python_matrix);
    python_vector = args[0];
    python_matrix = args[1];
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"vector", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(vector)), METH_FASTCALL, nullptr},
    {"matrix", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(matrix)), METH_FASTCALL, nullptr},
    {"use", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(use)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) { return PyModule_Create(&module); }
