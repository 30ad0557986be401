// Argument marshalling of the Python binding in native code: a tensor argument's checks and its device
// pointer in one call.  In Python the same checks are eight attribute reads, about 1 us per tensor, and an
// entry point takes up to seven tensors: more host time than the kernel of a small layer runs.
// Nothing but reads of tensor metadata happens in vector() and matrix().  Whatever is not a plain torch.Tensor or Parameter
// (subclasses may override attributes, other objects have to be refused) goes to the Python function that makes the
// same checks, given once by use().
//
// build_indices() is the index build of a list of masks with its loops over them in native code, for the same reason:
// while the device waits for the host between the count and the fill, a mask costs 0.8 us here and 3 in Python.
#include <ATen/ops/empty.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/object_ptr.h>

#include <chrono>
#include <vector>

#include "samo.h"

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

// The GIL given up for as long as this lives.
struct WithoutGil {
    PyThreadState *state = PyEval_SaveThread();
    ~WithoutGil() { PyEval_RestoreThread(state); }
};

// Elements of masks from which on build_indices launches the fill of those that have their index allocated while it goes on
// with the others; twice as many for every further launch.  28 matrices of 550 M elements: four launches.  A launch costs the host
// 5 us and fills 32 M elements in 3, so the first one starts the device early and the last ones keep it busy.
constexpr int64_t kFirstFill = 32 << 20;

// Waits until a count has appeared in page-locked memory; false if that takes longer than kPatience: other work ahead on the
// stream.  The caller then reads the counts back, which waits for the stream.
constexpr int64_t kNoCount = -1;
constexpr std::chrono::microseconds kPatience(2000);
bool seen(const int64_t *count)
{
    if (__atomic_load_n(count, __ATOMIC_ACQUIRE) != kNoCount) return true;
    const auto until = std::chrono::steady_clock::now() + kPatience;
    for (int spins = 1; __atomic_load_n(count, __ATOMIC_ACQUIRE) == kNoCount; ++spins) {
        __builtin_ia32_pause();
        if (spins % 64 == 0 && std::chrono::steady_clock::now() > until) return false;
    }
    return true;
}

// Page-locked memory goes back to torch's cache when the build leaves it, also by an exception (no memory for an index): not before
// the last count was stored in it.
struct CountsAwaited {
    const at::Tensor &nnz;
    const int64_t *counts = nullptr;
    size_t k = 0;
    ~CountsAwaited()
    {
        for (size_t i = 0; i < k; ++i) {
            if (seen(counts + i)) continue;
            try {
                nnz.cpu();
            } catch (...) {
            }
            return;
        }
    }
};

// Elements of masks from which on they are counted in two launches: the counts of the first half are there, and the
// fill of its masks is launched, while the second half is counted.
constexpr int64_t kCountInParts = 64 << 20;

// build_indices(masks, stream, scratch, count, fill[, mirrored, capture]): indices of byte masks (a list) by the entries samo_count_flags_batched
// and samo_fill_index_batched at the addresses `count` and `fill`; stream() is the handle of the stream to launch on, scratch(nbytes) a
// uint8 tensor for the flag bits or None.  With `mirrored` (samo_count_flags_mirrored_batched) and `capture` (hipStreamIsCapturing) the
// counts are polled instead of read back: a stream synchronisation and a copy between the two launches are 10 to 15 us.  Not on a
// stream under capture: its graph may be launched after the page-locked counts have gone back to their cache.
// A list of (idx, seg_ptr, nnz, n); a status other than SAMO_OK as an int; None where the
// caller has to go another way: a mask is no plain tensor, or there is no scratch memory.
PyObject *build_indices(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    HANDLE_TH_ERRORS
    typedef samo_status (*Entry)(const samo_index_job *, void *const *, int32_t, void *);
    typedef samo_status (*Mirrored)(const samo_index_job *, void *const *, int64_t *, int32_t, void *);
    if ((nargs != 5 && nargs != 7) || !PyList_Check(args[0]) || PyList_GET_SIZE(args[0]) == 0) {
        PyErr_SetString(PyExc_TypeError, "build_indices(masks, stream, scratch, count, fill[, mirrored, capture])");
        return nullptr;
    }
    const Entry count = reinterpret_cast<Entry>(PyLong_AsVoidPtr(args[3])), fill = reinterpret_cast<Entry>(PyLong_AsVoidPtr(args[4]));
    typedef int (*Capture)(void *, int *);
    Mirrored mirrored = reinterpret_cast<Mirrored>(nargs > 5 ? PyLong_AsVoidPtr(args[5]) : nullptr);
    const Capture capture = reinterpret_cast<Capture>(nargs > 5 ? PyLong_AsVoidPtr(args[6]) : nullptr);
    if (PyErr_Occurred()) return nullptr;
    const size_t k = (size_t)PyList_GET_SIZE(args[0]);
    std::vector<at::Tensor> masks(k), seg_ptrs(k), idxs(k);              // they hold the masks whatever happens to the list
    std::vector<samo_index_job> jobs(k);
    std::vector<void *> flags(k);
    int64_t flag_bytes = 0, elements = 0;
    for (size_t i = 0; i < k; ++i) {
        PyObject *m = PyList_GET_ITEM(args[0], (Py_ssize_t)i);
        if (!THPVariable_CheckExact(m)) Py_RETURN_NONE;
        masks[i] = THPVariable_Unpack(m);
        if (!masks[i].is_cuda() || masks[i].scalar_type() != at::kByte || masks[i].dim() != 1 || !masks[i].is_contiguous()) Py_RETURN_NONE;
        const int64_t n = masks[i].numel();
        if (n > INT32_MAX) return PyLong_FromLong(SAMO_ERR_SIZE);
        flag_bytes += (n + 8 * SAMO_SEG_ELEMS - 1) / (8 * SAMO_SEG_ELEMS) * 1024;
        elements += n;
    }
    THPObjectPtr handle(PyObject_CallNoArgs(args[1]));
    if (!handle) return nullptr;
    void *stream = PyLong_AsVoidPtr(handle.get());
    if (PyErr_Occurred()) return nullptr;
    int capturing = 1;
    if (mirrored && (!capture || capture(stream, &capturing) != 0 || capturing != 0)) mirrored = nullptr;
    THPObjectPtr bytes(PyLong_FromLongLong(flag_bytes > 0 ? flag_bytes : 1));
    THPObjectPtr scratch(bytes ? PyObject_CallOneArg(args[2], bytes) : nullptr);
    if (!scratch) return nullptr;
    if (!THPVariable_Check(scratch.get())) Py_RETURN_NONE;
    char *flags_at = static_cast<char *>(THPVariable_Unpack(scratch.get()).data_ptr());
    const at::TensorOptions ints = masks[0].options().dtype(at::kInt).requires_grad(false);
    at::Tensor counts;                       // in host memory
    samo_status status;
    {
        WithoutGil gil;
        at::Tensor nnz = at::empty({(int64_t)k}, ints.dtype(at::kLong));
        CountsAwaited awaited{nnz};
        for (size_t i = 0; i < k; ++i) {
            const int64_t n = masks[i].numel();
            seg_ptrs[i] = at::empty({(n + SAMO_SEG_ELEMS - 1) / SAMO_SEG_ELEMS + 1}, ints);
            jobs[i] = {n ? static_cast<const uint8_t *>(masks[i].data_ptr()) : nullptr, n, nullptr, 0,
                       static_cast<int32_t *>(seg_ptrs[i].data_ptr()), static_cast<int64_t *>(nnz.data_ptr()) + i};
            flags[i] = flags_at;
            flags_at += (n + 8 * SAMO_SEG_ELEMS - 1) / (8 * SAMO_SEG_ELEMS) * 1024;
        }
        if (mirrored) {
            counts = at::empty({(int64_t)k}, at::TensorOptions().dtype(at::kLong).pinned_memory(true));
            int64_t *there = counts.data_ptr<int64_t>();
            for (size_t i = 0; i < k; ++i) there[i] = kNoCount;
            size_t part = k;
            if (elements >= kCountInParts)
                for (int64_t sum = part = 0; 2 * sum < elements; ++part) sum += jobs[part].n;
            status = mirrored(jobs.data(), flags.data(), there, (int32_t)part, stream);
            awaited.counts = there;
            // a call that failed at a launch may have launched others before it, any other failure has launched nothing
            if (status == SAMO_OK || status == SAMO_ERR_HIP) awaited.k = part;
            if (status == SAMO_OK && part < k) {
                status = mirrored(jobs.data() + part, flags.data() + part, there + part, (int32_t)(k - part), stream);
                if (status == SAMO_OK || status == SAMO_ERR_HIP) awaited.k = k;
            }
        } else {
            status = count(jobs.data(), flags.data(), (int32_t)k, stream);
            if (status == SAMO_OK) counts = nnz.cpu();
        }
        bool polled = mirrored != nullptr;
        int64_t waiting = 0, enough = kFirstFill;
        for (size_t i = 0, first = 0; status == SAMO_OK && i < k; ++i) {
            if (polled && !seen(counts.data_ptr<int64_t>() + i)) {
                at::Tensor read = nnz.cpu();     // waits for the stream
                awaited.k = 0;
                counts = std::move(read);
                polled = false;
            }
            const int64_t found = counts.data_ptr<int64_t>()[i];
            idxs[i] = at::empty({found}, ints);
            jobs[i].idx = found ? static_cast<int32_t *>(idxs[i].data_ptr()) : nullptr;
            jobs[i].idx_capacity = found;
            waiting += jobs[i].n;
            if (waiting < enough && i + 1 < k) continue;
            status = fill(jobs.data() + first, flags.data() + first, (int32_t)(i + 1 - first), stream);
            first = i + 1;
            waiting = 0;
            enough *= 2;
        }
    }
    if (status != SAMO_OK) return PyLong_FromLong(status);
    THPObjectPtr out(PyList_New((Py_ssize_t)k));
    if (!out) return nullptr;
    for (size_t i = 0; i < k; ++i) {
        PyObject *item = Py_BuildValue("NNLL", THPVariable_Wrap(idxs[i]), THPVariable_Wrap(seg_ptrs[i]), (long long)jobs[i].idx_capacity, (long long)jobs[i].n);
        if (!item) return nullptr;
        PyList_SET_ITEM(out.get(), (Py_ssize_t)i, item);
    }
    return out.release();
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
    {"build_indices", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(build_indices)), METH_FASTCALL, nullptr},
    {"use", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(use)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) { return PyModule_Create(&module); }
