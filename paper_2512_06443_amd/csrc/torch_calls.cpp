// The binding's frequent calls as native code: arguments out of torch tensors, outputs and workspaces from torch's allocator, the
// call of the C ABI on the current stream.  binding.py has each of them in Python too and takes that form whenever a function
// here returns None, which it does for every argument it does not know to be ordinary, before anything has been launched: a
// tensor subclass or one without plain storage, another number type, an active torch-function mode, a failed check.  So errors
// are always raised there, and this file decides nothing but speed.
// Why: a launch takes 2.2 us of the host, the Python form of a call 2.5 to 5 us around it (torch.empty 1.8 us each, ctypes with
// 15 arguments 0.6, attribute reads and checks), this one 0.7 to 2.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstring>

#include "vlut.h"

namespace {

struct Api {                                   // addresses inside the loaded libvlut.so, in the order of binding._NATIVE_ORDER
    decltype(&vlut_quantize_act) quantize_act;
    decltype(&vlut_mpgemm_lean) mpgemm;
    decltype(&vlut_workspace_used) workspace;
    decltype(&vlut_mpgemm_f32) mpgemm_f32;
    decltype(&vlut_workspace_bytes_f32) workspace_bytes_f32;
    decltype(&vlut_mpgemm_g5_lean) mpgemm_g5;
    decltype(&vlut_workspace_used_g5) workspace_g5;
    decltype(&vlut_mpgemm_mixed_lean) mpgemm_mixed;
    decltype(&vlut_workspace_used_mixed) workspace_mixed;
    decltype(&vlut_pack_weights) pack_weights;
    decltype(&vlut_packed_weight_bytes) packed_weight_bytes;
    decltype(&vlut_pack_weights_g5) pack_weights_g5;
    decltype(&vlut_packed_weight_bytes_g5) packed_weight_bytes_g5;
    decltype(&vlut_pack_weights_mixed) pack_weights_mixed;
    decltype(&vlut_packed_weight_bytes_mixed) packed_weight_bytes_mixed;
};
constexpr int kApiCount = (int)(sizeof(Api) / sizeof(void*));
Api g_api;                                     // written once, by bind()
bool g_bound = false;

// The object as a tensor that a kernel can be given: exactly a Tensor (or Parameter) on the GPU with storage of its own and no wrapper
// around it.  Null otherwise.
const at::Tensor* plain(PyObject* o) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    constexpr c10::DispatchKeySet odd({c10::DispatchKey::Python, c10::DispatchKey::PythonTLSSnapshot, c10::DispatchKey::FuncTorchBatched,
                                       c10::DispatchKey::FuncTorchGradWrapper, c10::DispatchKey::Functionalize, c10::DispatchKey::Conjugate,
                                       c10::DispatchKey::Negative, c10::DispatchKey::ZeroTensor});
    if (!t.defined() || !t.is_cuda() || t.layout() != c10::kStrided || !t.has_storage() || t.key_set().has_any(odd)) return nullptr;
    return &t;
}
bool matrix(const at::Tensor* t, c10::ScalarType type) { return t && t->scalar_type() == type && t->dim() == 2 && t->stride(1) == 1; }
bool whole(PyObject* o, int64_t& v) {
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    v = PyLong_AsLongLongAndOverflow(o, &overflow);
    return overflow == 0;
}
bool real(PyObject* o, float& v) {
    if (!PyFloat_CheckExact(o)) return false;
    v = (float)PyFloat_AS_DOUBLE(o);
    return true;
}
// None, or an ordinary tensor
bool optional(PyObject* o, const at::Tensor*& t) {
    t = nullptr;
    return o == Py_None || (t = plain(o)) != nullptr;
}
bool output(PyObject* o, const at::Tensor*& t) { return optional(o, t) && (!t || t->dim() >= 1); }

at::Tensor make(c10::IntArrayRef size, c10::ScalarType type, c10::Device dev) {
    return at::empty(size, at::TensorOptions().dtype(type).device(dev));
}
size_t bytes_of(const at::Tensor& t) { return (size_t)t.numel() * t.element_size(); }
void* stream() { return (void*)c10::hip::getCurrentHIPStream().stream(); }
template <class T>
T* ptr(const at::Tensor& t) { return t.defined() ? (T*)t.data_ptr() : nullptr; }

PyObject* wrapped(const at::Tensor& t) {
    if (t.defined()) return THPVariable_Wrap(t);
    Py_RETURN_NONE;
}
// The outputs as a tuple; the status of the call as a whole number if it is not VLUT_OK.
template <class... T>
PyObject* result(int rc, const T&... t) {
    if (rc != VLUT_OK) return PyLong_FromLong(rc);
    PyObject* const items[] = {wrapped(t)...};
    PyObject* tuple = PyTuple_New(sizeof...(T));
    bool ok = tuple != nullptr;
    for (size_t i = 0; i < sizeof...(T); ++i) {
        ok = ok && items[i];
        if (tuple) PyTuple_SET_ITEM(tuple, i, items[i]);       // (owned by the tuple from here, also if null)
        else Py_XDECREF(items[i]);
    }
    if (ok) return tuple;
    Py_XDECREF(tuple);
    return nullptr;
}
// Ordinary situation: the functions are known, the argument count fits, and no torch-function mode wants to see the calls.
bool ordinary(Py_ssize_t n, Py_ssize_t want) { return g_bound && n == want && !at::impl::torch_function_mode_enabled(); }

// What is allocated in here throws as torch does (out of memory, say): the Python form then meets the same and raises it.
template <class F>
PyObject* guarded(F f) {
    try {
        return f();
    } catch (...) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}
// Other threads run Python during the allocations and the call of the library, as they do during torch.empty and a ctypes call: an
// allocation may wait for the device.  Taken back on the way out of an exception too.
struct WithoutGil {
    PyThreadState* const state = PyEval_SaveThread();
    ~WithoutGil() { PyEval_RestoreThread(state); }
};
template <class F>
void without_gil(F f) {
    const WithoutGil released;
    f();
}

// quantize_act(x, a_q, a_scale)
PyObject* py_quantize_act(PyObject*, PyObject* const* o, Py_ssize_t n) {
    return guarded([&]() -> PyObject* {
        const at::Tensor *x, *given_q, *given_s;
        if (!ordinary(n, 3) || !matrix(x = plain(o[0]), at::kFloat) || !optional(o[1], given_q) || !optional(o[2], given_s)) Py_RETURN_NONE;
        const int64_t N = x->size(0), K = x->size(1);
        at::Tensor a_q, a_s;
        if (given_q) a_q = *given_q;
        if (given_s) a_s = *given_s;
        int rc;
        without_gil([&] {
            if (!given_q) a_q = make({(N + 7) / 8, K, 8}, at::kChar, x->device());
            if (!given_s) a_s = make({N}, at::kFloat, x->device());
            rc = g_api.quantize_act(ptr<float>(*x), N, K, x->stride(0), ptr<int8_t>(a_q), ptr<float>(a_s), stream());
        });
        return result(rc, a_q, a_s);
    });
}

// What mpgemm, mpgemm_g5 and mpgemm_mixed have in common: (packed, w_scale, a_q, a_scale, M, y, acc or None, want_acc, workspace or None).
// `used` tells what the call needs of operands aligned to 16 bytes; others are left to the Python form, and so is a workspace without
// memory, which the lean call would take for one that was not given.
template <class Bytes, class Call>
PyObject* product(PyObject* const* o, Bytes used, Call call) {
    return guarded([&]() -> PyObject* {
        const at::Tensor *packed = plain(o[0]), *q = plain(o[2]), *s = plain(o[3]), *gy, *gacc, *gws;
        float w_scale;
        int64_t M;
        if (!packed || !q || !s || q->dim() < 2 || s->dim() < 1 || !real(o[1], w_scale) || !whole(o[4], M) || M < 0 || !output(o[5], gy) ||
            !optional(o[6], gacc) || !optional(o[8], gws) || (gws && !gws->data_ptr()) || ((uintptr_t)packed->data_ptr() | (uintptr_t)q->data_ptr()) % 16 != 0)
            Py_RETURN_NONE;
        const int64_t K = q->size(1), N = s->size(0);
        const int want = PyObject_IsTrue(o[7]);
        if (want < 0) { PyErr_Clear(); Py_RETURN_NONE; }
        at::Tensor y, acc, ws;
        if (gy) y = *gy;
        if (gacc) acc = *gacc;
        if (gws) ws = *gws;
        int rc;
        without_gil([&] {
            if (!gy) y = make({N, M}, at::kFloat, q->device());
            if (!gacc && want) acc = make({M, N}, at::kInt, q->device());
            if (!gws) {
                const size_t need = used(M, K, N);
                if (need) ws = make({(int64_t)need}, at::kByte, q->device());
            }
            rc = call(ptr<uint8_t>(*packed), w_scale, ptr<int8_t>(*q), ptr<float>(*s), M, K, N, ptr<float>(y), y.stride(0), ptr<int32_t>(acc),
                      ptr<void>(ws), ws.defined() ? bytes_of(ws) : 0, stream());
        });
        return result(rc, y, acc);
    });
}

PyObject* py_mpgemm(PyObject*, PyObject* const* o, Py_ssize_t n) {
    if (!ordinary(n, 9)) Py_RETURN_NONE;
    return product(o, g_api.workspace, [](const uint8_t* p, float w, const int8_t* q, const float* s, int64_t M, int64_t K, int64_t N, float* y,
                                                   int64_t ldy, int32_t* acc, void* ws, size_t bytes, void* st) {
        return g_api.mpgemm(p, w, q, s, nullptr, M, K, N, y, ldy, acc, ws, bytes, st);
    });
}
PyObject* py_mpgemm_g5(PyObject*, PyObject* const* o, Py_ssize_t n) {
    if (!ordinary(n, 9)) Py_RETURN_NONE;
    return product(o, g_api.workspace_g5, g_api.mpgemm_g5);
}
PyObject* py_mpgemm_mixed(PyObject*, PyObject* const* o, Py_ssize_t n) {
    if (!ordinary(n, 9)) Py_RETURN_NONE;
    return product(o, g_api.workspace_mixed, g_api.mpgemm_mixed);
}

// mpgemm_f32(packed, w_scale, x, M, y, want_acc, want_scales, workspace)
PyObject* py_mpgemm_f32(PyObject*, PyObject* const* o, Py_ssize_t n) {
    return guarded([&]() -> PyObject* {
        const at::Tensor *packed, *x, *gy, *gws, *rows = nullptr;
        float w_scale = 1.0f;
        int64_t M;
        if (!ordinary(n, 8) || !(packed = plain(o[0])) || !matrix(x = plain(o[2]), at::kFloat) || !whole(o[3], M) || M < 0 || !output(o[4], gy) ||
            !optional(o[7], gws))
            Py_RETURN_NONE;
        if (!real(o[1], w_scale) && (!(rows = plain(o[1])) || rows->scalar_type() != at::kFloat || rows->numel() != M)) Py_RETURN_NONE;
        const int want_acc = PyObject_IsTrue(o[5]), want_scales = PyObject_IsTrue(o[6]);
        if (want_acc < 0 || want_scales < 0) { PyErr_Clear(); Py_RETURN_NONE; }
        const int64_t N = x->size(0), K = x->size(1);
        at::Tensor y, acc, scales, ws, w_rows;
        if (gy) y = *gy;
        if (gws) ws = *gws;
        if (rows) w_rows = *rows;
        int rc;
        without_gil([&] {
            if (!gy) y = make({N, M}, at::kFloat, x->device());
            if (want_acc) acc = make({M, N}, at::kInt, x->device());
            if (want_scales) scales = make({N}, at::kFloat, x->device());
            size_t bytes = 0;
            if (gws) bytes = bytes_of(ws);
            else if ((bytes = g_api.workspace_bytes_f32(M, K, N)) != 0) ws = make({(int64_t)bytes}, at::kByte, x->device());
            rc = g_api.mpgemm_f32(ptr<uint8_t>(*packed), w_scale, ptr<float>(w_rows), ptr<float>(*x), x->stride(0), M, K, N, ptr<float>(y), y.stride(0),
                                  ptr<int32_t>(acc), ptr<float>(scales), ptr<void>(ws), bytes, stream());
        });
        return result(rc, y, acc, scales);
    });
}

// pack_weights*(w): a tuple of the blob
template <class Bytes, class Call>
PyObject* pack(PyObject* const* o, Py_ssize_t n, Bytes packed_bytes, Call call) {
    return guarded([&]() -> PyObject* {
        const at::Tensor* w;
        if (!ordinary(n, 1) || !(w = plain(o[0])) || w->scalar_type() != at::kChar || w->dim() != 2 || !w->is_contiguous()) Py_RETURN_NONE;
        const int64_t M = w->size(0), K = w->size(1);
        const size_t bytes = packed_bytes(M, K);
        if (bytes == 0) Py_RETURN_NONE;
        at::Tensor packed;
        int rc;
        without_gil([&] {
            packed = make({(int64_t)bytes}, at::kByte, w->device());
            rc = call(ptr<int8_t>(*w), M, K, ptr<uint8_t>(packed), bytes, stream());
        });
        return result(rc, packed);
    });
}
PyObject* py_pack_weights(PyObject*, PyObject* const* o, Py_ssize_t n) { return pack(o, n, g_api.packed_weight_bytes, g_api.pack_weights); }
PyObject* py_pack_weights_g5(PyObject*, PyObject* const* o, Py_ssize_t n) { return pack(o, n, g_api.packed_weight_bytes_g5, g_api.pack_weights_g5); }
PyObject* py_pack_weights_mixed(PyObject*, PyObject* const* o, Py_ssize_t n) {
    return pack(o, n, g_api.packed_weight_bytes_mixed, g_api.pack_weights_mixed);
}

// bind(addresses): the functions of the loaded library, as whole numbers in the order of Api
PyObject* py_bind(PyObject*, PyObject* const* o, Py_ssize_t n) {
    void* address[kApiCount];
    if (n != kApiCount) {
        PyErr_SetString(PyExc_TypeError, "bind: one address for each function");
        return nullptr;
    }
    for (int i = 0; i < kApiCount; ++i) {
        address[i] = PyLong_AsVoidPtr(o[i]);
        if (!address[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "bind: null address");
            return nullptr;
        }
    }
    std::memcpy((void*)&g_api, address, sizeof(g_api));
    g_bound = true;
    Py_RETURN_NONE;
}

PyMethodDef kMethods[] = {
    {"bind", (PyCFunction)(void (*)(void))py_bind, METH_FASTCALL, nullptr},
    {"quantize_act", (PyCFunction)(void (*)(void))py_quantize_act, METH_FASTCALL, nullptr},
    {"mpgemm", (PyCFunction)(void (*)(void))py_mpgemm, METH_FASTCALL, nullptr},
    {"mpgemm_f32", (PyCFunction)(void (*)(void))py_mpgemm_f32, METH_FASTCALL, nullptr},
    {"mpgemm_g5", (PyCFunction)(void (*)(void))py_mpgemm_g5, METH_FASTCALL, nullptr},
    {"mpgemm_mixed", (PyCFunction)(void (*)(void))py_mpgemm_mixed, METH_FASTCALL, nullptr},
    {"pack_weights", (PyCFunction)(void (*)(void))py_pack_weights, METH_FASTCALL, nullptr},
    {"pack_weights_g5", (PyCFunction)(void (*)(void))py_pack_weights_g5, METH_FASTCALL, nullptr},
    {"pack_weights_mixed", (PyCFunction)(void (*)(void))py_pack_weights_mixed, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_vlut_torch", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// built_for: the torch and the Python of the headers above (binding.built_for); binding.py uses no module that was built for others
PyMODINIT_FUNC PyInit__vlut_torch(void) {
    PyObject* m = PyModule_Create(&kModule);
    if (m && PyModule_AddStringConstant(m, "built_for", VLUT_BUILT_FOR) != 0) Py_CLEAR(m);
    return m;
}
