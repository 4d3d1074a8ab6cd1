// The operations of binding.py in their ordinary form, as native calls: plain tensors on the current device, the current stream, results
// new or given.  What costs a small call its time is the host -- 5.3 us through Python, of which the launch is 2.85 -- and most of the
// rest was Python's: torch.empty 1.35, attribute look-ups and checks 0.6, ctypes 0.4.  us, through Python / native, in most runs (some hosts
// are faster: the last figure): scan of 65541 elements 5.5 / 4.9, 4.3 (4.1 are the kernel), sums of 2^20 elements in segments of 256 5.3 / 4.4, 3.9, moments
// of 6.4 million in segments of 784 6.3 / 5.4, 4.9 (the last with smaller shares than before too).
// Everything else is left to binding.py: a function here returns None, before it has done anything, where an argument is not what
// is expected (subclasses and wrapped tensors, modes, other devices, wrong types and sizes), and binding.py goes on to its own
// checks and errors.  Nothing is computed here; libtcr.so's functions come as addresses from binding.py, which has loaded it.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/ops/empty.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/tcr.h"

namespace {

decltype(&tcr_segmented_reduce) g_segmented_reduce;
decltype(&tcr_segmented_scan_ex) g_segmented_scan_ex;
decltype(&tcr_scan_ex) g_scan_ex;
decltype(&tcr_reduce) g_reduce;
decltype(&tcr_segmented_moments) g_segmented_moments;
decltype(&tcr_irregular_reduce) g_irregular_reduce;
decltype(&tcr_irregular_scan_ex) g_irregular_scan_ex;
decltype(&tcr_irregular_scan_filled) g_irregular_scan_filled;
decltype(&tcr_irregular_moments) g_irregular_moments;
PyObject* g_error;                              // binding.TcrError(status, where)

// A contiguous tensor of `type` in this process's GPU memory and nothing more special than that.
const at::Tensor* plain(PyObject* o, at::ScalarType type) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    constexpr c10::DispatchKeySet usual({c10::DispatchKey::CUDA, c10::DispatchKey::ADInplaceOrView, c10::DispatchKey::AutogradCUDA, c10::DispatchKey::AutocastCUDA});
    const c10::DispatchKeySet keys = t.key_set();
    if (!keys.has(c10::DispatchKey::CUDA) || (keys.raw_repr() & ~usual.raw_repr()) != 0 || t.scalar_type() != type || !t.is_contiguous()) return nullptr;
    return &t;
}
// The input: one dimension, on the current device; no mode wants to see what is called.
const at::Tensor* input(PyObject* o) {
    const at::Tensor* x = plain(o, at::kHalf);
    if (x == nullptr || x->dim() != 1 || at::impl::torch_function_mode_enabled() || c10::impl::TorchDispatchModeTLS::any_modes_set()) return nullptr;
    c10::DeviceIndex device = -1;
    if (c10::hip::GetDevice(&device) != hipSuccess || device != x->device().index()) return nullptr;
    return x;
}
const at::Tensor* entries(PyObject* o, const at::Tensor& x) {
    const at::Tensor* t = plain(o, at::kLong);
    return t != nullptr && t->dim() == 1 && t->numel() >= 1 && t->device() == x.device() ? t : nullptr;
}
bool number(PyObject* o, uint64_t least, uint64_t most, uint64_t& v) {
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    const long long got = PyLong_AsLongLongAndOverflow(o, &overflow);
    if (overflow != 0 || got < 0 || (uint64_t)got < least || (uint64_t)got > most) return false;
    v = (uint64_t)got;
    return true;
}

// Gives the interpreter up, as torch.empty does around the allocation too: one that grows, or frees what is cached, may wait for the device, and
// the device for Python.
struct WithoutInterpreter {
    PyThreadState* const state = PyEval_SaveThread();
    ~WithoutInterpreter() { PyEval_RestoreThread(state); }
};

// The results: given and then of the right size, or new, which is for later (ready).
struct Results {
    at::Tensor made;
    PyObject* given = nullptr;
    void* data = nullptr;
    int64_t count = 0;
    at::ScalarType type = at::kFloat;
    bool set(PyObject* out, uint64_t size, at::ScalarType dtype, const at::Tensor& x) {
        count = (int64_t)size;
        type = dtype;
        if (out == Py_None) return true;
        const at::Tensor* t = plain(out, type);
        if (t == nullptr || (uint64_t)t->numel() != size || t->device() != x.device()) return false;
        given = out;
        data = t->data_ptr();
        return true;
    }
    void ready(const at::Tensor& x) {
        if (given != nullptr) return;
        made = at::empty({count}, x.options().dtype(type).requires_grad(false));
        data = made.data_ptr();
    }
    PyObject* take() {
        if (given == nullptr) return THPVariable_Wrap(std::move(made));
        Py_INCREF(given);
        return given;
    }
};

void* stream_of(const at::Tensor& x) { return c10::hip::getCurrentHIPStream(x.device().index()).stream(); }

PyObject* failed(tcr_status st, const char* where) {
    PyObject* e = PyObject_CallFunction(g_error, "is", (int)st, where);
    if (e != nullptr) {
        PyErr_SetObject(g_error, e);
        Py_DECREF(e);
    }
    return nullptr;
}
// Allocation and call, with the interpreter given up once for both.
#define TCR_CALL(allocate, expression)      \
    tcr_status st;                          \
    {                                       \
        const WithoutInterpreter released;  \
        allocate;                           \
        st = (expression);                  \
    }

// segmented_reduce(x, seg_len, out)
PyObject* segmented_reduce(PyObject*, PyObject* const* args, Py_ssize_t count) {
    HANDLE_TH_ERRORS
    const at::Tensor* x = count == 3 ? input(args[0]) : nullptr;
    uint64_t seg_len = 0;
    if (x == nullptr || !number(args[1], 1, INT64_MAX, seg_len)) Py_RETURN_NONE;
    const uint64_t n = (uint64_t)x->numel();
    Results out;
    if (n % seg_len != 0 || !out.set(args[2], n / seg_len, at::kFloat, *x)) Py_RETURN_NONE;
    const void* in = x->data_ptr();
    void* const stream = stream_of(*x);
    TCR_CALL(out.ready(*x), g_segmented_reduce(in, static_cast<float*>(out.data), n, seg_len, stream))
    return st == TCR_OK ? out.take() : failed(st, "tcr_segmented_reduce");
    END_HANDLE_TH_ERRORS
}

// x in segments of seg_len, or as one (seg_len 0)
PyObject* scan_in(const at::Tensor& x, uint64_t seg_len, uint64_t flags, PyObject* given, PyObject* where) {
    const uint64_t n = (uint64_t)x.numel();
    Results out;
    if ((seg_len != 0 && n % seg_len != 0) || !out.set(given, n, flags & TCR_OUT_F16 ? at::kHalf : at::kFloat, x)) Py_RETURN_NONE;
    const void* in = x.data_ptr();
    void* const stream = stream_of(x);
    TCR_CALL(out.ready(x), seg_len != 0 ? g_segmented_scan_ex(in, out.data, n, seg_len, (uint32_t)flags, stream) : g_scan_ex(in, out.data, n, (uint32_t)flags, stream))
    return st == TCR_OK ? out.take() : failed(st, PyUnicode_AsUTF8(where));
}
// segmented_scan(x, seg_len, flags, out, where)
PyObject* segmented_scan(PyObject*, PyObject* const* args, Py_ssize_t count) {
    HANDLE_TH_ERRORS
    const at::Tensor* x = count == 5 ? input(args[0]) : nullptr;
    uint64_t seg_len = 0, flags = 0;
    if (x == nullptr || !number(args[1], 1, INT64_MAX, seg_len) || !number(args[2], 0, 7, flags)) Py_RETURN_NONE;
    return scan_in(*x, seg_len, flags, args[3], args[4]);
    END_HANDLE_TH_ERRORS
}
// scan(x, flags, out, where)
PyObject* scan(PyObject*, PyObject* const* args, Py_ssize_t count) {
    HANDLE_TH_ERRORS
    const at::Tensor* x = count == 4 ? input(args[0]) : nullptr;
    uint64_t flags = 0;
    if (x == nullptr || !number(args[1], 0, 7, flags)) Py_RETURN_NONE;
    return scan_in(*x, 0, flags, args[2], args[3]);
    END_HANDLE_TH_ERRORS
}

// reduce(x, out)
PyObject* reduce(PyObject*, PyObject* const* args, Py_ssize_t count) {
    HANDLE_TH_ERRORS
    const at::Tensor* x = count == 2 ? input(args[0]) : nullptr;
    Results out;
    if (x == nullptr || !out.set(args[1], 1, at::kFloat, *x)) Py_RETURN_NONE;
    const void* in = x->data_ptr();
    const uint64_t n = (uint64_t)x->numel();
    void* const stream = stream_of(*x);
    TCR_CALL(out.ready(*x), g_reduce(in, static_cast<float*>(out.data), n, stream))
    return st == TCR_OK ? out.take() : failed(st, "tcr_reduce");
    END_HANDLE_TH_ERRORS
}

// segmented_moments(x, seg_len)
PyObject* segmented_moments(PyObject*, PyObject* const* args, Py_ssize_t count) {
    HANDLE_TH_ERRORS
    const at::Tensor* x = count == 2 ? input(args[0]) : nullptr;
    uint64_t seg_len = 0;
    if (x == nullptr || !number(args[1], 1, INT64_MAX, seg_len)) Py_RETURN_NONE;
    const uint64_t n = (uint64_t)x->numel();
    Results a, q;
    a.set(Py_None, n / seg_len, at::kFloat, *x);
    q.set(Py_None, n / seg_len, at::kFloat, *x);
    const void* in = x->data_ptr();
    void* const stream = stream_of(*x);
    TCR_CALL((a.ready(*x), q.ready(*x)), g_segmented_moments(in, static_cast<float*>(a.data), static_cast<float*>(q.data), n, seg_len, stream))
    return st == TCR_OK ? Py_BuildValue("NN", a.take(), q.take()) : failed(st, "tcr_segmented_moments");
    END_HANDLE_TH_ERRORS
}

// irregular_reduce(x, offsets, out)
PyObject* irregular_reduce(PyObject*, PyObject* const* args, Py_ssize_t count) {
    HANDLE_TH_ERRORS
    const at::Tensor* x = count == 3 ? input(args[0]) : nullptr;
    const at::Tensor* offsets = x != nullptr ? entries(args[1], *x) : nullptr;
    Results out;
    if (offsets == nullptr || !out.set(args[2], (uint64_t)offsets->numel() - 1, at::kFloat, *x)) Py_RETURN_NONE;
    const void* in = x->data_ptr();
    const uint64_t* off = static_cast<const uint64_t*>(offsets->data_ptr());
    const uint64_t n = (uint64_t)x->numel(), nseg = (uint64_t)offsets->numel() - 1;
    void* const stream = stream_of(*x);
    TCR_CALL(out.ready(*x), g_irregular_reduce(in, off, static_cast<float*>(out.data), n, nseg, stream))
    return st == TCR_OK ? out.take() : failed(st, "tcr_irregular_reduce");
    END_HANDLE_TH_ERRORS
}

// irregular_moments(x, offsets)
PyObject* irregular_moments(PyObject*, PyObject* const* args, Py_ssize_t count) {
    HANDLE_TH_ERRORS
    const at::Tensor* x = count == 2 ? input(args[0]) : nullptr;
    const at::Tensor* offsets = x != nullptr ? entries(args[1], *x) : nullptr;
    if (offsets == nullptr) Py_RETURN_NONE;
    const uint64_t n = (uint64_t)x->numel(), nseg = (uint64_t)offsets->numel() - 1;
    Results a, q;
    a.set(Py_None, nseg, at::kFloat, *x);
    q.set(Py_None, nseg, at::kFloat, *x);
    const void* in = x->data_ptr();
    const uint64_t* off = static_cast<const uint64_t*>(offsets->data_ptr());
    void* const stream = stream_of(*x);
    TCR_CALL((a.ready(*x), q.ready(*x)), g_irregular_moments(in, off, static_cast<float*>(a.data), static_cast<float*>(q.data), n, nseg, stream))
    return st == TCR_OK ? Py_BuildValue("NN", a.take(), q.take()) : failed(st, "tcr_irregular_moments");
    END_HANDLE_TH_ERRORS
}

// irregular_scan(x, offsets, flags, out, where); new results are 0 where no segment lies
PyObject* irregular_scan(PyObject*, PyObject* const* args, Py_ssize_t count) {
    HANDLE_TH_ERRORS
    const at::Tensor* x = count == 5 ? input(args[0]) : nullptr;
    const at::Tensor* offsets = x != nullptr ? entries(args[1], *x) : nullptr;
    uint64_t flags = 0;
    if (offsets == nullptr || !number(args[2], 0, 7, flags)) Py_RETURN_NONE;
    const uint64_t n = (uint64_t)x->numel(), nseg = (uint64_t)offsets->numel() - 1;
    Results out;
    if (!out.set(args[3], n, flags & TCR_OUT_F16 ? at::kHalf : at::kFloat, *x)) Py_RETURN_NONE;
    const void* in = x->data_ptr();
    const uint64_t* off = static_cast<const uint64_t*>(offsets->data_ptr());
    void* const stream = stream_of(*x);
    TCR_CALL(out.ready(*x), (out.given == nullptr ? g_irregular_scan_filled : g_irregular_scan_ex)(in, off, out.data, n, nseg, (uint32_t)flags, stream))
    return st == TCR_OK ? out.take() : failed(st, PyUnicode_AsUTF8(args[4]));
    END_HANDLE_TH_ERRORS
}

// bind(error class, addresses): in the order of the variables above
PyObject* bind(PyObject*, PyObject* args) {
    unsigned long long a[9];
    PyObject* error = nullptr;
    if (!PyArg_ParseTuple(args, "OKKKKKKKKK", &error, &a[0], &a[1], &a[2], &a[3], &a[4], &a[5], &a[6], &a[7], &a[8])) return nullptr;
    g_segmented_reduce = reinterpret_cast<decltype(g_segmented_reduce)>(a[0]);
    g_segmented_scan_ex = reinterpret_cast<decltype(g_segmented_scan_ex)>(a[1]);
    g_scan_ex = reinterpret_cast<decltype(g_scan_ex)>(a[2]);
    g_reduce = reinterpret_cast<decltype(g_reduce)>(a[3]);
    g_segmented_moments = reinterpret_cast<decltype(g_segmented_moments)>(a[4]);
    g_irregular_reduce = reinterpret_cast<decltype(g_irregular_reduce)>(a[5]);
    g_irregular_scan_ex = reinterpret_cast<decltype(g_irregular_scan_ex)>(a[6]);
    g_irregular_scan_filled = reinterpret_cast<decltype(g_irregular_scan_filled)>(a[7]);
    g_irregular_moments = reinterpret_cast<decltype(g_irregular_moments)>(a[8]);
    Py_INCREF(error);
    Py_XSETREF(g_error, error);
    Py_RETURN_NONE;
}

#define TCR_FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {TCR_FAST(segmented_reduce), TCR_FAST(segmented_scan), TCR_FAST(scan), TCR_FAST(reduce), TCR_FAST(segmented_moments),
                           TCR_FAST(irregular_reduce), TCR_FAST(irregular_moments), TCR_FAST(irregular_scan),
                           {"bind", bind, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_native", "The ordinary calls of binding.py (see there).", -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() { return PyModule_Create(&g_module); }
