// The per-iteration calls from Python, for the ordinary case: checks the tensors, makes the output and
// calls the C entry point, without a Python object in between.  What this leaves (subclasses and wrapped
// tensors, anything that is not as the call wants it, modes that watch torch's functions) returns None, and
// the caller goes through binding.py's own checks, which say what is wrong.
//
// A minibatch of a small graph is two kernels of 4 us; through ctypes a call took 7.2 and 8.2 us of the host,
// of which the launch is 3: 1.7 for torch.empty from Python, 1.0 for ctypes, the rest attributes and checks.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <torch/csrc/autograd/generated/variable_factories.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/jit/frontend/tracer.h>

#include <cstdint>
#include <string>

namespace {

using DequantFn = int (*)(void *, const uint8_t *, int64_t, const int64_t *, int64_t, float *, void *);
using AggregateFn = int (*)(void *, const uint8_t *, int64_t, const int64_t *, const void *, int64_t, int64_t, float *,
                            void *);

PyObject *g_device = nullptr, *g_stream = nullptr;  // torch._C._cuda_getDevice, ._cuda_getCurrentRawStream

const at::Tensor *tensor(PyObject *o, at::ScalarType a, at::ScalarType b) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.dim() < 1 || t.layout() != at::kStrided) return nullptr;
    if (!t.unsafeGetTensorImpl()->has_storage() || !t.is_contiguous()) return nullptr;
    return t.scalar_type() == a || t.scalar_type() == b ? &t : nullptr;
}

bool watched() {
    return at::impl::torch_function_mode_enabled() || c10::impl::TorchDispatchModeTLS::any_modes_set() ||
           torch::jit::tracer::isTracing();
}

// the current stream's handle, as binding.py asks for it; false with a Python error set
bool stream(void **out) {
    PyObject *device = PyObject_CallNoArgs(g_device);
    if (!device) return false;
    PyObject *handle = PyObject_CallOneArg(g_stream, device);
    Py_DECREF(device);
    if (!handle) return false;
    *out = PyLong_AsVoidPtr(handle);
    Py_DECREF(handle);
    return !(*out == nullptr && PyErr_Occurred());
}

// The interpreter runs other threads while this lives: an allocation may wait for the device, or for a lock that
// another thread holds.
struct Released {
    PyThreadState *state = PyEval_SaveThread();
    ~Released() { PyEval_RestoreThread(state); }
    Released() = default;
    Released(const Released &) = delete;
};

at::Tensor rows(const at::Tensor &like, int64_t n, int64_t D) {
    return torch::empty({n, D}, at::TensorOptions().dtype(at::kFloat).device(like.device()));
}

// Returns the output tensor, an error status as an integer, or None (see the top).
PyObject *finish(int status, const at::Tensor &out) {
    return status == 0 ? THPVariable_Wrap(out) : PyLong_FromLong(status);
}

// gather_dequant(address of the entry point, handle, codes, idx, D)
PyObject *gather_dequant(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (n != 5) Py_RETURN_NONE;
    try {
        const at::Tensor *codes = tensor(a[2], at::kByte, at::kByte), *idx = tensor(a[3], at::kLong, at::kLong);
        if (!codes || !idx || watched()) Py_RETURN_NONE;
        auto fn = reinterpret_cast<DequantFn>(PyLong_AsVoidPtr(a[0]));
        void *handle = PyLong_AsVoidPtr(a[1]), *s = nullptr;
        const int64_t D = PyLong_AsLongLong(a[4]);
        if (!fn || !handle || D <= 0 || PyErr_Occurred() || !stream(&s)) {
            PyErr_Clear();
            Py_RETURN_NONE;
        }
        const int64_t M = idx->size(0), N = codes->size(0);
        const auto *pc = static_cast<const uint8_t *>(codes->data_ptr());
        const auto *pi = static_cast<const int64_t *>(idx->data_ptr());
        at::Tensor out;
        int status;
        {
            Released interpreter;
            out = rows(*codes, M, D);
            status = fn(handle, pc, N, pi, M, static_cast<float *>(out.data_ptr()), s);
        }
        return finish(status, out);
    } catch (...) {
        Py_RETURN_NONE;
    }
}

// aggregate(address for 64-bit entries, for 32-bit ones, handle, codes, indptr, indices, D)
PyObject *aggregate(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (n != 7) Py_RETURN_NONE;
    try {
        const at::Tensor *codes = tensor(a[3], at::kByte, at::kByte), *indptr = tensor(a[4], at::kLong, at::kLong),
                         *indices = tensor(a[5], at::kLong, at::kInt);
        if (!codes || !indptr || !indices || indptr->size(0) < 1 || watched()) Py_RETURN_NONE;
        auto fn = reinterpret_cast<AggregateFn>(PyLong_AsVoidPtr(a[indices->scalar_type() == at::kInt ? 1 : 0]));
        void *handle = PyLong_AsVoidPtr(a[2]), *s = nullptr;
        const int64_t D = PyLong_AsLongLong(a[6]);
        if (!fn || !handle || D <= 0 || PyErr_Occurred() || !stream(&s)) {
            PyErr_Clear();
            Py_RETURN_NONE;
        }
        const int64_t V = indptr->size(0) - 1, E = indices->size(0), N = codes->size(0);
        const auto *pc = static_cast<const uint8_t *>(codes->data_ptr());
        const auto *pp = static_cast<const int64_t *>(indptr->data_ptr());
        const void *pi = indices->data_ptr();
        at::Tensor out;
        int status;
        {
            Released interpreter;
            out = rows(*codes, V, D);
            status = fn(handle, pc, N, pp, pi, V, E, static_cast<float *>(out.data_ptr()), s);
        }
        return finish(status, out);
    } catch (...) {
        Py_RETURN_NONE;
    }
}

PyMethodDef methods[] = {
    {"gather_dequant", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(gather_dequant)), METH_FASTCALL, nullptr},
    {"aggregate", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(aggregate)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls() {
    PyObject *c = PyImport_ImportModule("torch._C");
    if (!c) return nullptr;
    g_device = PyObject_GetAttrString(c, "_cuda_getDevice");
    g_stream = g_device ? PyObject_GetAttrString(c, "_cuda_getCurrentRawStream") : nullptr;
    Py_DECREF(c);
    // (tensors are taken apart by their layout in the torch that this was compiled against)
    PyObject *torch = PyImport_ImportModule("torch");
    PyObject *version = torch ? PyObject_GetAttrString(torch, "__version__") : nullptr;
    PyObject *text = version ? PyObject_Str(version) : nullptr;
    const char *now = text ? PyUnicode_AsUTF8(text) : nullptr;
    const std::string python = std::to_string(PY_MAJOR_VERSION) + "." + std::to_string(PY_MINOR_VERSION) + ".";
    if (now && (std::string(now) != BF_TORCH_VERSION || std::string(Py_GetVersion()).rfind(python, 0) != 0))
        PyErr_Format(PyExc_ImportError, "_calls.so was built for torch %s and Python %sx", BF_TORCH_VERSION, python.c_str());
    Py_XDECREF(text);
    Py_XDECREF(version);
    Py_XDECREF(torch);
    if (PyErr_Occurred()) return nullptr;
    return g_stream ? PyModule_Create(&module) : nullptr;
}
