// Marshalling of the layer's calls in C++ (module paper_2309_16119_amd._marshal): what binding.py and nn.py do
// in Python for tensors as they are met in earnest -- plain, contiguous, on the GPU, of the types the calls
// take, outputs not given -- and nothing else.  Every function returns None for anything it does not take, and
// the Python code, which stays the definition of checks, conversions and errors, does the call.  No
// arithmetic here: the entry points of libmodulora.so are handed over as addresses by binding.py.
//
// Why: on a small layer the host is slower than the GPU.  256 x 256, 16 tokens, forward and backward in three
// calls: 38 us of Python against 23 us of kernels; through the autograd module 155 us, of which torch's own
// engine with its hand-over to another thread is 46 (forward 21, and a Python backward on that thread the rest).
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/anomaly_mode.h>
#include <torch/csrc/autograd/custom_function.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/jit/frontend/tracer.h>
#include <torch/custom_class.h>
#include <ATen/ATen.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>

#include <cstdint>
#include <map>
#include <mutex>
#include <optional>
#include <utility>
#include <vector>

#include "modulora.h"

namespace {

using at::Tensor;

// ---- the library's entry points ---------------------------------------------------------------
using fwd_fn = int (*)(const void *, const uint16_t *, int32_t, const float *, const float *, int32_t, float, uint16_t *, float *, void *, size_t, void *);
using grad_fn = decltype(&modulora_bwd_lora);
using bytes_fn = size_t (*)(const void *, int32_t, int32_t);
struct Library {
    fwd_fn product[2][2];      // [binary16][backward]
    grad_fn grad[2];
    bytes_fn bytes[2];
} lib{};

struct ReleaseGil {            // as ctypes does around a library call
    PyThreadState *state = PyGILState_Check() ? PyEval_SaveThread() : nullptr;
    ~ReleaseGil() { if (state) PyEval_RestoreThread(state); }
};

// ---- scratch memory: one buffer per (device, stream), see binding._workspace() --------------------
// A call is several launches that hand data over through the scratch memory of their stream, so a call has to be on its
// stream whole before another host thread's on the same stream begins: `order` is held from before the library call
// until it has returned.  (Recursive: what Python runs on its own account, a finalizer say, may call in between.)
struct Scratch {
    std::recursive_mutex order;                             // of `held` too
    std::vector<Tensor> held;
};
struct Scratches {
    std::mutex mutex;
    std::map<std::pair<int, int64_t>, Scratch> of;          // entries stay where they are
};
Scratches &scratches() {
    static auto *s = new Scratches;        // never destroyed: the buffers outlive the GPU runtime's own end otherwise
    return *s;
}
Scratch &scratch_of(int device, int64_t stream) {
    static thread_local std::pair<int, int64_t> last_key;
    static thread_local Scratch *last = nullptr;
    const std::pair<int, int64_t> key(device, stream);
    if (!last || last_key != key) {
        std::lock_guard<std::mutex> lock(scratches().mutex);
        last = &scratches().of[key];
        last_key = key;
    }
    return *last;
}
// A call's turn on its stream: holds `order`, and a buffer of at least `nbytes`.  No thread waits for `order` with
// Python's lock in hand.  A request larger than the held buffer gets a new one; the old ones stay, because a HIP graph
// captured earlier may still hold their addresses.
struct Turn {
    Scratch *scratch = nullptr;            // none for no bytes
    Turn(int device, int64_t stream, size_t nbytes) {
        if (nbytes == 0) return;
        Scratch *s = &scratch_of(device, stream);
        take(s);
        if (s->held.empty() || (size_t)s->held.back().numel() < nbytes) {
            s->order.unlock();             // (the allocator may run Python of its own)
            Tensor t = at::empty({(int64_t)nbytes}, at::TensorOptions().dtype(at::kByte).device(at::kCUDA, device));
            take(s);
            if (s->held.empty() || s->held.back().numel() < t.numel()) s->held.push_back(t);
        }
        scratch = s;
    }
    ~Turn() { if (scratch) scratch->order.unlock(); }
    Turn(const Turn &) = delete;
    void *memory() const { return scratch ? scratch->held.back().data_ptr() : nullptr; }

private:
    static void take(Scratch *s) {
        if (s->order.try_lock()) return;
        ReleaseGil release;
        s->order.lock();
    }
};

// ---- the weight, as the attributes of a QWeight / QWeightF16 say at the time of the call -----------------
struct Weight {
    int32_t d_in, d_out, bits, group;
    Tensor qweight, scales, zeros, bias;
    bool f16;
};
PyObject *names[8];
enum { D_IN, D_OUT, BITS, GROUP, QWEIGHT, SCALES, ZEROS, BIAS };
bool read_int(PyObject *w, int name, int32_t &out) {
    PyObject *v = PyObject_GetAttr(w, names[name]);
    if (!v) return false;
    const bool ok = PyLong_CheckExact(v);
    const long value = ok ? PyLong_AsLong(v) : -1;
    Py_DECREF(v);
    out = (int32_t)value;
    return ok && value == out && !PyErr_Occurred();
}
bool read_tensor(PyObject *w, int name, Tensor &out, bool optional = false) {
    PyObject *v = PyObject_GetAttr(w, names[name]);
    if (!v) return false;
    const bool none = optional && v == Py_None, ok = none || THPVariable_CheckExact(v);
    if (ok && !none) out = THPVariable_Unpack(v);
    Py_DECREF(v);
    return ok;
}

// A tensor whose memory is what it says: no wrapper of a transform, no lazily negated or virtual data.
bool plain(const Tensor &t) {
    if (!t.defined() || !t.is_cuda() || !t.has_storage() || !t.is_contiguous() || t.is_neg()) return false;
    const auto keys = t.key_set();
    return !keys.has(c10::DispatchKey::Python) && !keys.has(c10::DispatchKey::FuncTorchBatched) && !keys.has(c10::DispatchKey::FuncTorchGradWrapper) &&
           !keys.has(c10::DispatchKey::Functionalize) && !keys.has(c10::DispatchKey::Batched) && !keys.has(c10::DispatchKey::ZeroTensor);
}
bool read_weight(PyObject *w, bool f16, Weight &out) {
    out.f16 = f16;
    const bool ok = read_int(w, D_IN, out.d_in) && read_int(w, D_OUT, out.d_out) && read_int(w, BITS, out.bits) && read_int(w, GROUP, out.group) &&
                    read_tensor(w, QWEIGHT, out.qweight) && read_tensor(w, SCALES, out.scales) && read_tensor(w, ZEROS, out.zeros) &&
                    (!f16 || read_tensor(w, BIAS, out.bias, true));
    if (!ok) { PyErr_Clear(); return false; }
    return plain(out.qweight) && plain(out.scales) && plain(out.zeros) && (!out.bias.defined() || plain(out.bias));
}

// Modes under which a call is more than a call: left to Python.
bool special_mode() {
    return c10::impl::TorchDispatchModeTLS::any_modes_set() || torch::jit::tracer::isTracing() ||
           c10::impl::tls_is_dispatch_key_included(c10::DispatchKey::FuncTorchDynamicLayerFrontMode) ||
           c10::impl::tls_is_dispatch_key_included(c10::DispatchKey::Functionalize);
}
bool unpack(PyObject *o, Tensor &t) {
    if (!THPVariable_CheckExact(o)) return false;
    t = THPVariable_Unpack(o);
    return true;
}
template <typename T>
T *ptr(const Tensor &t) { return t.defined() ? static_cast<T *>(t.data_ptr()) : nullptr; }

// The adapter's factors: both or neither.
bool factors_fit(const Tensor &A, const Tensor &B, int64_t d_in, int64_t d_out) {
    if (A.defined() != B.defined()) return false;
    if (!A.defined()) return true;
    return plain(A) && plain(B) && A.scalar_type() == at::kFloat && B.scalar_type() == at::kFloat && A.dim() == 2 && B.dim() == 2 &&
           A.size(0) == d_in && B.size(1) == d_out && A.size(1) == B.size(0) && A.size(1) > 0;
}

struct Where {                 // what a call is launched on, and its turn there
    void *stream;
    Turn turn;
    Where(int device, size_t nbytes) : Where(device, nbytes, c10::hip::current_device()) {}

private:
    Where(int device, size_t nbytes, int current) : Where(device, nbytes, current, c10::hip::getCurrentHIPStream(current)) {}
    Where(int device, size_t nbytes, int current, c10::hip::HIPStream s)
        : stream(s.stream()), turn(device, (int64_t)(intptr_t)(device == current ? s : c10::hip::getCurrentHIPStream(device)).stream(), nbytes) {}
};

// One forward or input-gradient call; returns the library's status.
int product(const Weight &w, bool backward, const Tensor &act, const Tensor &A, const Tensor &B, float scale, bool want_P, Tensor &out, Tensor &P) {
    const int64_t M = act.size(0), r = A.defined() ? A.size(1) : 0;
    out = at::empty({M, backward ? w.d_in : w.d_out}, act.options().requires_grad(false));
    if (want_P && r) P = at::empty({M, r}, act.options().dtype(at::kFloat).requires_grad(false));
    modulora_qweight q{w.d_in, w.d_out, w.bits, w.group, ptr<uint32_t>(w.qweight), ptr<uint16_t>(w.scales), ptr<uint8_t>(w.zeros)};
    modulora_qweight_f16 h{w.d_in, w.d_out, w.bits, w.group, ptr<uint32_t>(w.qweight), ptr<uint16_t>(w.scales), ptr<uint16_t>(w.zeros), ptr<uint16_t>(w.bias)};
    const void *layer = w.f16 ? static_cast<const void *>(&h) : static_cast<const void *>(&q);
    const size_t nbytes = lib.bytes[w.f16](layer, (int32_t)M, (int32_t)r);
    const Where at(act.get_device(), nbytes);
    ReleaseGil release;
    return lib.product[w.f16][backward](layer, ptr<uint16_t>(act), (int32_t)M, ptr<float>(A), ptr<float>(B), (int32_t)r, scale, ptr<uint16_t>(out),
                                        ptr<float>(P), at.turn.memory(), nbytes, at.stream);
}
int gradients(bool f16, const Tensor &X, const Tensor &dY, const Tensor &A, const Tensor &B, float scale, const Tensor &XA, const Tensor &T, Tensor &dA, Tensor &dB) {
    const int64_t M = X.size(0), r = A.size(1);
    const int32_t d_in = (int32_t)X.size(1), d_out = (int32_t)dY.size(1);
    const auto opt = X.options().dtype(at::kFloat).requires_grad(false);
    dA = at::empty({d_in, r}, opt);
    dB = at::empty({r, d_out}, opt);
    modulora_qweight q{d_in, d_out, 4, 32, nullptr, nullptr, nullptr};
    modulora_qweight_f16 h{d_in, d_out, 4, 32, nullptr, nullptr, nullptr, nullptr};
    const size_t nbytes = lib.bytes[f16](f16 ? static_cast<const void *>(&h) : static_cast<const void *>(&q), (int32_t)M, (int32_t)r);
    const Where at(X.get_device(), nbytes);
    ReleaseGil release;
    return lib.grad[f16](d_in, d_out, (int32_t)M, (int32_t)r, scale, ptr<uint16_t>(X), ptr<uint16_t>(dY), ptr<float>(A), ptr<float>(B), ptr<float>(XA), ptr<float>(T),
                         ptr<float>(dA), ptr<float>(dB), 0, at.turn.memory(), nbytes, at.stream);
}
at::ScalarType act_type(bool f16) { return f16 ? at::kHalf : at::kBFloat16; }

// ---- calls from binding.py ----------------------------------------------------------------------
// product(f16, backward, w, act, A, B, lora_scale, want_P) -> (out, P or None), a status, or None
PyObject *py_product(PyObject *, PyObject *const *args, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 8 || special_mode()) Py_RETURN_NONE;
    const bool f16 = args[0] == Py_True, backward = args[1] == Py_True;
    Weight w;
    Tensor act, A, B, out, P;
    if (!unpack(args[3], act) || !plain(act) || !read_weight(args[2], f16, w)) Py_RETURN_NONE;
    if ((args[4] != Py_None && !unpack(args[4], A)) || (args[5] != Py_None && !unpack(args[5], B))) Py_RETURN_NONE;
    if (act.scalar_type() != act_type(f16) || act.dim() != 2 || act.size(1) != (backward ? w.d_out : w.d_in) || act.size(0) >= INT32_MAX) Py_RETURN_NONE;
    if (!factors_fit(A, B, w.d_in, w.d_out)) Py_RETURN_NONE;
    const double scale = PyFloat_AsDouble(args[6]);
    if (scale == -1.0 && PyErr_Occurred()) { PyErr_Clear(); Py_RETURN_NONE; }
    const int want = PyObject_IsTrue(args[7]);
    if (want < 0) { PyErr_Clear(); Py_RETURN_NONE; }
    at::NoGradGuard no_grad;
    const int status = product(w, backward, act, A, B, (float)scale, want != 0, out, P);
    if (status != MODULORA_OK) return PyLong_FromLong(status);
    PyObject *o = THPVariable_Wrap(out), *p = P.defined() ? THPVariable_Wrap(P) : (Py_INCREF(Py_None), Py_None);
    PyObject *pair = o && p ? PyTuple_Pack(2, o, p) : nullptr;
    Py_XDECREF(o);
    Py_XDECREF(p);
    return pair;
    END_HANDLE_TH_ERRORS
}
// gradients(f16, X, dY, A, B, lora_scale, XA, dYBt) -> (dA, dB), a status, or None
PyObject *py_gradients(PyObject *, PyObject *const *args, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 8 || special_mode()) Py_RETURN_NONE;
    const bool f16 = args[0] == Py_True;
    Tensor X, dY, A, B, XA, T, dA, dB;
    if (!unpack(args[1], X) || !unpack(args[2], dY) || !unpack(args[3], A) || !unpack(args[4], B)) Py_RETURN_NONE;
    if ((args[6] != Py_None && !unpack(args[6], XA)) || (args[7] != Py_None && !unpack(args[7], T))) Py_RETURN_NONE;
    if (!plain(X) || !plain(dY) || X.scalar_type() != act_type(f16) || dY.scalar_type() != act_type(f16) || X.dim() != 2 || dY.dim() != 2 ||
        X.size(0) != dY.size(0) || X.size(0) >= INT32_MAX || X.size(1) >= INT32_MAX || dY.size(1) >= INT32_MAX || !factors_fit(A, B, X.size(1), dY.size(1)))
        Py_RETURN_NONE;
    for (const Tensor *t : {&XA, &T})
        if (t->defined() && !plain(*t)) Py_RETURN_NONE;
    const double scale = PyFloat_AsDouble(args[5]);
    if (scale == -1.0 && PyErr_Occurred()) { PyErr_Clear(); Py_RETURN_NONE; }
    at::NoGradGuard no_grad;
    const int status = gradients(f16, X, dY, A, B, (float)scale, XA, T, dA, dB);
    if (status != MODULORA_OK) return PyLong_FromLong(status);
    PyObject *a = THPVariable_Wrap(dA), *b = THPVariable_Wrap(dB), *pair = a && b ? PyTuple_Pack(2, a, b) : nullptr;
    Py_XDECREF(a);
    Py_XDECREF(b);
    return pair;
    END_HANDLE_TH_ERRORS
}

// ---- the autograd function of nn.LPLoRAFunction ----------------------------------------------------
struct WeightObject : torch::CustomClassHolder {      // the Python weight, read anew by the backward pass
    PyObject *w;
    explicit WeightObject(PyObject *o) : w(o) { Py_INCREF(w); }
    ~WeightObject() override {
        if (!Py_IsInitialized()) return;
        const PyGILState_STATE g = PyGILState_Ensure();
        Py_DECREF(w);
        PyGILState_Release(g);
    }
};
// A backward call that the library refused before it launched anything: binding.ModuloraError, as Python raises it.
PyObject *refusal;
[[noreturn]] void raise_refusal(int status, const char *where) {
    python_error raised;
    {
        pybind11::gil_scoped_acquire gil;
        PyObject *error = PyObject_CallFunction(refusal, "is", status, where);
        if (error) PyErr_SetObject(refusal, error);
        Py_XDECREF(error);
        raised.persist();
    }
    throw std::move(raised);
}
struct Refused {};             // the library refused a forward call before it launched anything: Python names the error

struct Layer : torch::autograd::Function<Layer> {
    static Tensor forward(torch::autograd::AutogradContext *ctx, const Tensor &x, const std::optional<Tensor> &A_, const std::optional<Tensor> &B_,
                          const Weight &w, const c10::intrusive_ptr<WeightObject> &object, double scale) {
        const Tensor A = A_.value_or(Tensor()), B = B_.value_or(Tensor());
        const Tensor x2 = x.reshape({-1, w.d_in}).contiguous();
        Tensor y, xa;
        if (product(w, false, x2, A, B, (float)scale, true, y, xa) != MODULORA_OK) throw Refused();
        ctx->saved_data["w"] = c10::IValue::make_capsule(object);
        ctx->saved_data["scale"] = scale;
        ctx->saved_data["f16"] = w.f16;
        ctx->saved_data["shape"] = x.sizes().vec();
        ctx->save_for_backward({x2, A, B, xa});
        auto shape = x.sizes().vec();
        shape.back() = w.d_out;
        return y.view(shape);
    }
    static torch::autograd::variable_list backward(torch::autograd::AutogradContext *ctx, const torch::autograd::variable_list &grads) {
        const auto saved = ctx->get_saved_variables();
        const Tensor &x2 = saved[0], &A = saved[1], &B = saved[2], &xa = saved[3];
        const bool f16 = ctx->saved_data["f16"].toBool();
        const double scale = ctx->saved_data["scale"].toDouble();
        const auto shape = ctx->saved_data["shape"].toIntVector();
        Weight w;
        {
            const PyGILState_STATE g = PyGILState_Ensure();
            const auto object = c10::static_intrusive_pointer_cast<WeightObject>(ctx->saved_data["w"].toCapsule());
            const bool ok = read_weight(object->w, f16, w);
            PyGILState_Release(g);
            TORCH_CHECK(ok, "the frozen weight is no longer what the forward pass saw");
        }
        Tensor dy = grads[0].defined() ? grads[0] : at::zeros({x2.size(0), w.d_out}, x2.options());
        dy = dy.detach().reshape({-1, w.d_out}).to(act_type(f16)).contiguous();
        Tensor dx, t, dA, dB;
        at::NoGradGuard no_grad;
        // (saved-tensor hooks may have brought back other tensors than were saved, and the weight may be another one)
        const bool factors = A.defined() && (ctx->needs_input_grad(1) || ctx->needs_input_grad(2));
        TORCH_CHECK(plain(dy) && factors_fit(A, B, w.d_in, w.d_out), "the adapter or the weight is no longer what the forward pass saw");
        TORCH_CHECK(!factors || (plain(x2) && x2.scalar_type() == act_type(f16) && x2.dim() == 2 && x2.size(0) == dy.size(0) && x2.size(1) == w.d_in &&
                                 (!xa.defined() || (plain(xa) && xa.scalar_type() == at::kFloat && xa.numel() == dy.size(0) * A.size(1)))),
                    "the saved activations are no longer what the forward pass saw");
        int status = product(w, true, dy, A, B, (float)scale, true, dx, t);
        if (status != MODULORA_OK) raise_refusal(status, f16 ? "modulora_f16_bwd_input" : "modulora_bwd_input");
        if (factors) status = gradients(f16, x2, dy, A, B, (float)scale, xa, t, dA, dB);
        if (status != MODULORA_OK) raise_refusal(status, f16 ? "modulora_f16_bwd_lora" : "modulora_bwd_lora");
        return {dx.view(shape), dA, dB, Tensor(), Tensor(), Tensor()};
    }
};
// layer(f16, x, A, B, w, lora_scale) -> y with its place in the autograd graph, or None
PyObject *py_layer(PyObject *, PyObject *const *args, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 6 || special_mode() || torch::autograd::AnomalyMode::is_enabled()) Py_RETURN_NONE;
    const bool f16 = args[0] == Py_True;
    Weight w;
    Tensor x, A, B;
    if (!unpack(args[1], x) || !plain(x) || !read_weight(args[4], f16, w)) Py_RETURN_NONE;
    if ((args[2] != Py_None && !unpack(args[2], A)) || (args[3] != Py_None && !unpack(args[3], B))) Py_RETURN_NONE;
    if (x.scalar_type() != act_type(f16) || x.dim() < 1 || x.size(-1) != w.d_in || x.numel() == 0 || x.numel() / w.d_in >= INT32_MAX) Py_RETURN_NONE;
    for (const Tensor *t : {&x, &A, &B})      // forward-mode tangents: Python says that there is no rule for them
        if (t->defined() && t->_fw_grad(0).defined()) Py_RETURN_NONE;
    if (!factors_fit(A, B, w.d_in, w.d_out)) Py_RETURN_NONE;
    const double scale = PyFloat_AsDouble(args[5]);
    if (scale == -1.0 && PyErr_Occurred()) { PyErr_Clear(); Py_RETURN_NONE; }
    const auto opt = [](const Tensor &t) { return t.defined() ? std::optional<Tensor>(t) : std::nullopt; };
    Tensor y;
    try {
        y = Layer::apply(x, opt(A), opt(B), w, c10::make_intrusive<WeightObject>(args[4]), scale);
    } catch (const Refused &) {
        Py_RETURN_NONE;
    }
    return THPVariable_Wrap(y);
    END_HANDLE_TH_ERRORS
}

// workspace(device index, stream, bytes) -> uint8 tensor or None; forget_workspaces()
PyObject *py_workspace(PyObject *, PyObject *args) {
    HANDLE_TH_ERRORS
    int device;
    long long stream, nbytes;
    if (!PyArg_ParseTuple(args, "iLL", &device, &stream, &nbytes)) return nullptr;
    at::NoGradGuard no_grad;
    const Turn turn(device, stream, (size_t)nbytes);
    if (!turn.scratch) Py_RETURN_NONE;
    return THPVariable_Wrap(turn.scratch->held.back());
    END_HANDLE_TH_ERRORS
}
PyObject *py_forget(PyObject *, PyObject *) {
    HANDLE_TH_ERRORS
    std::vector<Tensor> gone;
    std::vector<Scratch *> all;
    {
        std::lock_guard<std::mutex> lock(scratches().mutex);
        for (auto &entry : scratches().of) all.push_back(&entry.second);
    }
    Py_BEGIN_ALLOW_THREADS
    for (Scratch *s : all) {
        std::lock_guard<std::recursive_mutex> lock(s->order);
        gone.insert(gone.end(), s->held.begin(), s->held.end());
        s->held.clear();
    }
    Py_END_ALLOW_THREADS
    Py_RETURN_NONE;
    END_HANDLE_TH_ERRORS
}
// lock(device index, stream), unlock(device index, stream): Scratch::order for a call that Python makes
PyObject *py_lock(PyObject *, PyObject *args) {
    HANDLE_TH_ERRORS
    int device;
    long long stream;
    if (!PyArg_ParseTuple(args, "iL", &device, &stream)) return nullptr;
    Scratch &s = scratch_of(device, stream);
    Py_BEGIN_ALLOW_THREADS
    s.order.lock();
    Py_END_ALLOW_THREADS
    Py_RETURN_NONE;
    END_HANDLE_TH_ERRORS
}
PyObject *py_unlock(PyObject *, PyObject *args) {
    HANDLE_TH_ERRORS
    int device;
    long long stream;
    if (!PyArg_ParseTuple(args, "iL", &device, &stream)) return nullptr;
    scratch_of(device, stream).order.unlock();
    Py_RETURN_NONE;
    END_HANDLE_TH_ERRORS
}
// use(addresses of fwd, bwd_input, bwd_lora, workspace_bytes, and of the four f16 ones, ModuloraError)
PyObject *py_use(PyObject *, PyObject *args) {
    unsigned long long p[8];
    PyObject *error;
    if (!PyArg_ParseTuple(args, "KKKKKKKKO", &p[0], &p[1], &p[2], &p[3], &p[4], &p[5], &p[6], &p[7], &error)) return nullptr;
    if (!refusal) refusal = Py_NewRef(error);      // of the first binding: another copy of the module changes nothing
    for (int f = 0; f < 2; ++f) {
        lib.product[f][0] = reinterpret_cast<fwd_fn>(p[4 * f]);
        lib.product[f][1] = reinterpret_cast<fwd_fn>(p[4 * f + 1]);
        lib.grad[f] = reinterpret_cast<grad_fn>(p[4 * f + 2]);
        lib.bytes[f] = reinterpret_cast<bytes_fn>(p[4 * f + 3]);
    }
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"product", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_product)), METH_FASTCALL, nullptr},
    {"gradients", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_gradients)), METH_FASTCALL, nullptr},
    {"layer", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_layer)), METH_FASTCALL, nullptr},
    {"workspace", py_workspace, METH_VARARGS, nullptr},
    {"forget_workspaces", py_forget, METH_NOARGS, nullptr},
    {"lock", py_lock, METH_VARARGS, nullptr},
    {"unlock", py_unlock, METH_VARARGS, nullptr},
    {"use", py_use, METH_VARARGS, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// Tensors are read through torch's C++ classes, whose layout is that of one build of torch: no other one loads this
// module (MARSHAL_TORCH: the version and commit it was compiled for), not even one with the same symbols.
static bool is_this_torch() {
    PyObject *module = PyImport_ImportModule("torch.version");
    PyObject *version = module ? PyObject_GetAttrString(module, "__version__") : nullptr;
    PyObject *commit = version ? PyObject_GetAttrString(module, "git_version") : nullptr;
    PyObject *found = commit ? PyUnicode_FromFormat("%S %S", version, commit) : nullptr;
    const bool same = found && PyUnicode_CompareWithASCIIString(found, MARSHAL_TORCH) == 0;
    if (!same) {
        PyErr_Clear();
        PyErr_Format(PyExc_ImportError, "compiled for torch %s, not %V", MARSHAL_TORCH, found, "this one");
    }
    Py_XDECREF(found);
    Py_XDECREF(commit);
    Py_XDECREF(version);
    Py_XDECREF(module);
    return same;
}

PyMODINIT_FUNC PyInit__marshal() {
    if (!is_this_torch()) return nullptr;
    const char *attr[8] = {"d_in", "d_out", "bits", "group_size", "qweight", "scales", "zeros", "bias"};
    for (int i = 0; i < 8; ++i)
        if (!(names[i] = PyUnicode_InternFromString(attr[i]))) return nullptr;
    return PyModule_Create(&module_def);
}
