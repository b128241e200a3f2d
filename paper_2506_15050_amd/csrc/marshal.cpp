// Python side of the C ABI (tppo.h), native: turns a call's tensors into pointers, allocates its results, and calls.  The
// smallest passes are bound by what happens here, once a call: through ctypes and torch's Python functions a token filter
// with its plan took 18.8 us of host time, log-probs 10.6, EGAE 5.7 and losses 6.0; here 9.1, 8.7, 3.6 and 3.9.
// What is taken and what is refused is what ctypes and the binding's own assertions take and refuse; sizes, ranges and NULLs are
// the C entry points' own business.
#include <Python.h>
#include <ATen/Context.h>
#include <ATen/ops/empty.h>
#include <c10/core/DeviceGuard.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <torch/csrc/Device.h>
#include <torch/csrc/DynamicTypes.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <exception>
#include <utility>

#include "tppo.h"

namespace {

struct Raised {};                                                   // a Python exception is set

[[noreturn]] void raise(PyObject* type, const char* text) {
    PyErr_SetString(type, text);
    throw Raised{};
}

// a new reference, or the exception that is there instead
class Held {
  public:
    explicit Held(PyObject* o) : o_(o) {
        if (!o) throw Raised{};
    }
    ~Held() { Py_DECREF(o_); }
    Held(const Held&) = delete;
    PyObject* get() const { return o_; }

  private:
    PyObject* o_;
};

// The arguments of one call, in order.
class Args {
  public:
    Args(PyObject* const* args, Py_ssize_t n, Py_ssize_t want) : at_(args) {
        if (n != want) raise(PyExc_TypeError, "wrong number of arguments");
    }
    // a tensor's memory; None: NULL.  Anything but a plain tensor is asked through Python, where a subclass or another
    // library's array has its own say.
    void* any() {
        PyObject* o = *at_++;
        if (o == Py_None) return nullptr;
        if (THPVariable_CheckExact(o)) return THPVariable_Unpack(o).data_ptr();
        const Held p(PyObject_CallMethod(o, "data_ptr", nullptr));
        if (p.get() == Py_None) return nullptr;
        void* v = PyLong_AsVoidPtr(p.get());
        if (PyErr_Occurred()) throw Raised{};
        return v;
    }
    template <typename T>
    T* ptr() { return static_cast<T*>(any()); }
    int32_t* dev_i32() { return static_cast<int32_t*>(checked(at::kInt)); }
    float* dev_f32() { return static_cast<float*>(checked(at::kFloat)); }
    // a buffer and its size in bytes; None: NULL and 0
    void* buffer(size_t& bytes) {
        bytes = 0;
        PyObject* o = *at_;
        if (o == Py_None) return any();
        if (THPVariable_CheckExact(o)) {
            bytes = (size_t)THPVariable_Unpack(o).numel();
        } else {
            const Held n(PyObject_CallMethod(o, "numel", nullptr));
            bytes = (size_t)PyLong_AsUnsignedLongLongMask(n.get());
            if (PyErr_Occurred()) throw Raised{};
        }
        return any();
    }
    int64_t i64() {
        PyObject* o = *at_++;
        const unsigned long long v = PyLong_AsUnsignedLongLongMask(o);
        if (v == ~0ull && PyErr_Occurred()) refuse(o);
        return (int64_t)v;
    }
    int32_t i32() { return (int32_t)i64(); }
    float f32() {
        const double v = PyFloat_AsDouble(*at_++);
        if (v == -1.0 && PyErr_Occurred()) throw Raised{};
        return (float)v;
    }
    void* stream() {
        void* s = PyLong_AsVoidPtr(*at_++);
        if (PyErr_Occurred()) throw Raised{};
        return s;
    }

  private:
    // what is no whole number: ctypes' own exception
    [[noreturn]] static void refuse(PyObject* o) {
        PyErr_Clear();
        const Held ctypes(PyImport_ImportModule("ctypes")), error(PyObject_GetAttrString(ctypes.get(), "ArgumentError"));
        PyErr_Format(error.get(), "int expected instead of %.200s instance", Py_TYPE(o)->tp_name);
        throw Raised{};
    }
    void* checked(at::ScalarType type) {
        PyObject* o = *at_;
        if (o == Py_None) raise(PyExc_AssertionError, "a tensor is required");
        bool good;
        if (THPVariable_CheckExact(o)) {
            const at::Tensor& t = THPVariable_Unpack(o);
            good = t.is_cuda() && t.scalar_type() == type && t.is_contiguous();
        } else {
            const Held cuda(PyObject_GetAttrString(o, "is_cuda")), dtype(PyObject_GetAttrString(o, "dtype"));
            const Held dense(PyObject_CallMethod(o, "is_contiguous", nullptr));
            good = truth(PyObject_IsTrue(cuda.get())) && truth(PyObject_IsTrue(dense.get())) &&
                   truth(PyObject_RichCompareBool(dtype.get(), reinterpret_cast<PyObject*>(torch::getTHPDtype(type)), Py_EQ));
        }
        if (!good) raise(PyExc_AssertionError, "a contiguous device tensor of the documented type is required");
        return any();
    }
    static bool truth(int answer) {
        if (answer < 0) throw Raised{};
        return answer != 0;
    }
    PyObject* const* at_;
};

// What torch raises passes as from its own functions: an allocation that fails is torch.OutOfMemoryError, an exception of a
// Python dispatch mode is that exception.
template <class F>
PyObject* guarded(F&& f) {
    try {
        return f();
    } catch (const Raised&) {
    } catch (...) {
        torch::translate_exception_to_python(std::current_exception());
    }
    return nullptr;
}

// other Python threads run while one of these lives
class NoInterpreter {
  public:
    NoInterpreter() : state_(PyEval_SaveThread()) {}
    ~NoInterpreter() { PyEval_RestoreThread(state_); }
    NoInterpreter(const NoInterpreter&) = delete;

  private:
    PyThreadState* state_;
};

// the call itself, with the interpreter free as it is under ctypes
template <class F>
PyObject* status_of(F&& call) {
    int rc;
    {
        NoInterpreter other_threads_run;
        rc = call();
    }
    return PyLong_FromLong(rc);
}

// a call of `want` arguments
template <PyObject* (*call)(Args&), int want>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t n) {
    return guarded([&] {
        Args x(args, n, want);
        return call(x);
    });
}

PyObject* select(Args& x) {
    auto *cu = x.dev_i32(), *ctx = x.dev_i32(), *done = x.dev_i32(), *ids = x.ptr<int32_t>();
    const int64_t B = x.i64(), n_tok = x.i64();
    const int32_t drop = x.i32();
    auto *resp = x.ptr<int32_t>(), *sel = x.ptr<int32_t>(), *keep = x.ptr<int32_t>(), *rows = x.ptr<int32_t>();
    auto *targets = x.ptr<int32_t>(), *idx = x.ptr<int32_t>();
    const int64_t cap = x.i64();
    auto* counts = x.ptr<int64_t>();
    size_t ws_bytes, plan_bytes;
    void *ws = x.buffer(ws_bytes), *plan = x.buffer(plan_bytes);
    auto* status = x.ptr<int32_t>();
    void* s = x.stream();
    return status_of([&] {
        return tppo_select(cu, ctx, done, ids, B, n_tok, drop, resp, sel, keep, rows, targets, idx, cap, counts, ws, ws_bytes,
                           plan, plan_bytes, status, s);
    });
}

PyObject* token_logprobs(Args& x) {
    const void* hidden = x.any();
    const int64_t n_rows = x.i64(), H = x.i64(), ld_h = x.i64();
    const void* w = x.any();
    const int64_t V = x.i64(), ld_w = x.i64();
    const auto dt = (tppo_dtype)x.i32();
    auto *rows = x.dev_i32(), *targets = x.dev_i32();
    const int64_t M = x.i64();
    auto* m_actual = x.ptr<int64_t>();
    auto* out_index = x.ptr<int32_t>();
    auto *logp = x.ptr<float>(), *lse = x.ptr<float>();
    size_t bytes;
    void* ws = x.buffer(bytes);
    auto* status = x.ptr<int32_t>();
    void* s = x.stream();
    return status_of([&] {
        return tppo_token_logprobs(hidden, n_rows, H, ld_h, w, V, ld_w, dt, rows, targets, M, m_actual, out_index, logp, lse, ws,
                                   bytes, status, s);
    });
}

// tppo_egae, tppo_egae_terminal
template <decltype(tppo_egae)* entry_point>
PyObject* egae(Args& x) {
    auto *rewards = x.dev_f32(), *values = x.dev_f32();
    auto *resp = x.dev_i32(), *done = x.dev_i32();
    auto* boot = x.ptr<float>();
    const int64_t B = x.i64(), n_resp = x.i64();
    const float gamma = x.f32(), lam = x.f32();
    auto *adv = x.ptr<float>(), *ret = x.ptr<float>();
    size_t bytes;
    void *ws = x.buffer(bytes), *plan = x.any();
    auto* status = x.ptr<int32_t>();
    void* s = x.stream();
    return status_of([&] {
        return entry_point(rewards, values, resp, done, boot, B, n_resp, gamma, lam, adv, ret, ws, bytes, plan, status, s);
    });
}

PyObject* ppo_losses(Args& x) {
    const float* in[6];
    for (auto& p : in) p = x.ptr<float>();
    auto *resp = x.dev_i32(), *keep = x.dev_i32(), *done = x.dev_i32();
    const int64_t B = x.i64(), n_resp = x.i64();
    const float el = x.f32(), eh = x.f32(), xl = x.f32(), xh = x.f32();
    auto* out = x.ptr<tppo_loss_out>();
    size_t bytes;
    void *ws = x.buffer(bytes), *plan = x.any();
    auto* status = x.ptr<int32_t>();
    void* s = x.stream();
    return status_of([&] {
        return tppo_ppo_losses(in[0], in[1], in[2], in[3], in[4], in[5], resp, keep, done, B, n_resp, el, eh, xl, xh, out, ws, bytes,
                               plan, status, s);
    });
}

PyObject* ppo_losses_backward(Args& x) {
    const float* in[6];
    for (auto& p : in) p = x.ptr<float>();
    auto *resp = x.dev_i32(), *keep = x.dev_i32(), *done = x.dev_i32();
    const int64_t B = x.i64(), n_resp = x.i64();
    const float el = x.f32(), eh = x.f32(), xl = x.f32(), xh = x.f32(), ps = x.f32(), vs = x.f32();
    const int64_t pd = x.i64(), vd = x.i64();
    auto *g_logp = x.ptr<float>(), *g_v = x.ptr<float>();
    auto* out = x.ptr<tppo_loss_out>();
    auto* stats = x.ptr<tppo_loss_stats>();
    size_t bytes;
    void *ws = x.buffer(bytes), *plan = x.any();
    auto* status = x.ptr<int32_t>();
    void* s = x.stream();
    return status_of([&] {
        return tppo_ppo_losses_backward(in[0], in[1], in[2], in[3], in[4], in[5], resp, keep, done, B, n_resp, el, eh, xl, xh, ps, vs,
                                        pd, vd, g_logp, g_v, out, stats, ws, bytes, plan, status, s);
    });
}

PyObject* value_head(Args& x) {
    const void* hidden = x.any();
    const int64_t n_rows = x.i64(), H = x.i64(), ld = x.i64();
    const void* w = x.any();
    const float bias = x.f32();
    const auto dt = (tppo_dtype)x.i32();
    auto *rows = x.ptr<int32_t>(), *out_index = x.ptr<int32_t>();
    const int64_t M = x.i64();
    auto* m_actual = x.ptr<int64_t>();
    auto* v = x.ptr<float>();
    auto* status = x.ptr<int32_t>();
    void* s = x.stream();
    return status_of([&] { return tppo_value_head(hidden, n_rows, H, ld, w, bias, dt, rows, out_index, M, m_actual, v, status, s); });
}

// sizes of buffers that a caller did not bring
PyObject* select_workspace_bytes(Args& x) {
    const int64_t B = x.i64(), capacity = x.i64();
    return PyLong_FromSize_t(tppo_select_workspace_bytes(B, capacity));
}
PyObject* plan_bytes(Args& x) {
    const int64_t n_resp = x.i64(), B = x.i64();
    return PyLong_FromSize_t(tppo_plan_bytes(n_resp, B));
}

// empties(like, kinds, n0, n1, ...): one-dimensional uninitialised tensors on `like`'s device, kinds[i] in "ilfb" (int32, int64,
// float32, bytes).  The interpreter is free meanwhile, as it is in torch.empty: an allocator that has to ask the driver, or that
// waits for another thread's call into it, must not hold up the other Python threads.
constexpr Py_ssize_t kMostBuffers = 16;

// Each buffer is an allocation of its own, as torch.empty's: a caller may resize it, give it as `out`, save it, keep it, and record a
// stream's use of it without the others.  (Pieces of one allocation are cheaper still and allow none of these: what grows runs into the
// next piece, and storages of their own over one block are none that the device's allocator knows to record a stream for.)  The first
// is at::empty's; the others are made here from its storage's allocator, past the dispatcher, whose way costs more than the allocation
// (a token filter's nine: 7.3 us of host time, so 4.4; pieces of one block 2.15), unless a dispatch mode, a transform, a trace or the
// fill of deterministic runs has its own say about allocations.
const c10::DispatchKeySet kPlainKeys({c10::DispatchKey::CPU, c10::DispatchKey::CUDA, c10::DispatchKey::ADInplaceOrView,
                                      c10::DispatchKey::AutogradCPU, c10::DispatchKey::AutogradCUDA, c10::DispatchKey::AutocastCPU,
                                      c10::DispatchKey::AutocastCUDA});
bool undisturbed() {                                               // nothing beyond the usual takes part in this thread's calls
    return !c10::impl::dispatch_mode_enabled() && c10::default_included_set.has_all(c10::impl::tls_local_dispatch_key_set().included_) &&
           !at::globalContext().deterministicAlgorithms();         // (which fills what is allocated, by type)
}
void allocate(const at::TensorOptions& on, const at::ScalarType* types, const int64_t* sizes, Py_ssize_t count, at::Tensor* made) {
    if (count == 0) return;
    made[0] = at::empty({sizes[0]}, on.dtype(types[0]));
    Py_ssize_t i = 1;
    const auto keys = made[0].key_set();
    if (count > 1 && undisturbed() && kPlainKeys.has_all(keys) && made[0].has_storage() && made[0].storage().allocator()) {
        const c10::DeviceGuard there(made[0].device());
        // (sizes that are none, or too many bytes for a number, are at::empty's to refuse)
        for (; i < count && sizes[i] >= 0 && sizes[i] <= INT64_MAX / 8; ++i) {
            c10::Storage own(c10::Storage::use_byte_size_t(), (size_t)sizes[i] * c10::elementSize(types[i]), made[0].storage().allocator(), true);
            made[i] = at::detail::make_tensor<c10::TensorImpl>(std::move(own), keys, c10::scalarTypeToTypeMeta(types[i]));
            made[i].unsafeGetTensorImpl()->set_sizes_contiguous({sizes[i]});
        }
    }
    for (; i < count; ++i) made[i] = at::empty({sizes[i]}, on.dtype(types[i]));
}
at::Device device_of(PyObject* like) {
    if (THPVariable_CheckExact(like)) return THPVariable_Unpack(like).device();
    const Held device(PyObject_GetAttrString(like, "device"));
    if (!THPDevice_Check(device.get())) raise(PyExc_TypeError, "a torch.device is required");
    return reinterpret_cast<THPDevice*>(device.get())->device;
}
PyObject* empties(PyObject*, PyObject* const* args, Py_ssize_t n) {
    HANDLE_TH_ERRORS                                                // (the allocator's warnings are Python's)
    try {
        if (n < 2 || args[0] == Py_None) raise(PyExc_TypeError, "empties(tensor, kinds, sizes...)");
        Py_ssize_t count = 0;
        const char* kinds = PyUnicode_AsUTF8AndSize(args[1], &count);
        if (!kinds) throw Raised{};
        if (count != n - 2) raise(PyExc_TypeError, "a size for each kind");
        const auto on = at::TensorOptions().device(device_of(args[0]));
        int64_t sizes[kMostBuffers];
        at::Tensor made[kMostBuffers];
        if (count > kMostBuffers) raise(PyExc_TypeError, "too many buffers");
        for (Py_ssize_t i = 0; i < count; ++i) {
            sizes[i] = PyLong_AsLongLong(args[2 + i]);
            if (sizes[i] == -1 && PyErr_Occurred()) throw Raised{};
        }
        {
            NoInterpreter other_threads_run;
            at::ScalarType types[kMostBuffers];
            for (Py_ssize_t i = 0; i < count; ++i)
                types[i] = kinds[i] == 'i' ? at::kInt : kinds[i] == 'l' ? at::kLong : kinds[i] == 'f' ? at::kFloat : at::kByte;
            allocate(on, types, sizes, count, made);
        }
        PyObject* out = PyTuple_New(count);
        if (!out) throw Raised{};
        for (Py_ssize_t i = 0; i < count; ++i) {
            PyObject* t = THPVariable_Wrap(made[i]);
            if (!t) {
                Py_DECREF(out);
                throw Raised{};
            }
            PyTuple_SET_ITEM(out, i, t);
        }
        return out;
    } catch (const Raised&) {
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}

template <PyObject* (*f)(PyObject*, PyObject* const*, Py_ssize_t)>
PyMethodDef method(const char* name) {
    return {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr};
}
PyMethodDef methods[] = {method<entry<select, 19>>("select"),
                         method<entry<token_logprobs, 18>>("token_logprobs"),
                         method<entry<egae<tppo_egae>, 15>>("egae"),
                         method<entry<egae<tppo_egae_terminal>, 15>>("egae_terminal"),
                         method<entry<ppo_losses, 20>>("ppo_losses"),
                         method<entry<ppo_losses_backward, 27>>("ppo_losses_backward"),
                         method<entry<value_head, 14>>("value_head"),
                         method<entry<select_workspace_bytes, 2>>("select_workspace_bytes"),
                         method<entry<plan_bytes, 2>>("plan_bytes"),
                         method<empties>("empties"),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) { return PyModule_Create(&module); }
