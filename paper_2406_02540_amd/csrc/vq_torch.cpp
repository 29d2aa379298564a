// The torch side of the C-ABI library: tensors to device pointers, the current stream, output
// allocation.  No arithmetic and no HIP call of its own: the entry points of libvidiq.so are
// handed over as addresses (bind()), checked arguments go straight to them.
//
// Why this is native: a layer on a few hundred tokens runs for about 10 us on the device, and
// marshalling the same ten arguments in Python (attribute checks, ctypes conversions, the stream
// object) kept the host longer than that: a vq_linear call took 13.4 us of host time, both
// kernels' launches included, and takes 6.4 here (15.1 and 7.1 where it allocates its output);
// the 256 x 1152 -> 1152 layer went from 15.1 to 10.0 us, and takes 7.3 to 8.3 with the kernels as they
// are, 7.0 of them on the device.
//
// Conventions: a Python exception that has been set travels as the C++ exception Raised;
// messages and exception types are part of the package's interface.
#include <Python.h>

#include <climits>
#include <type_traits>

#include <ATen/ATen.h>
#include <ATen/hip/impl/HIPStreamMasqueradingAsCUDA.h>
#include <c10/core/StreamGuard.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/Stream.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/version.h>

#include "vq.h"

namespace {

struct Raised {};

PyObject* g_vq_error = nullptr;  // the package's VqError(status, where)

// The library's entry points, in the order binding.py passes their addresses.
struct Entries {
    decltype(&::vq_quantize_per_token) quantize_per_token;
    decltype(&::vq_gelu_quantize) gelu_quantize;
    decltype(&::vq_layernorm_quantize) layernorm_quantize;
    decltype(&::vq_residual_quantize) residual_quantize;
    decltype(&::vq_hadamard_quantize) hadamard_quantize;
    decltype(&::vq_quantize_static) quantize_static;
    decltype(&::vq_channel_absmax) channel_absmax;
    decltype(&::vq_balance_mask) balance_mask;
    decltype(&::vq_rotate_weight) rotate_weight;
    decltype(&::vq_quantize_weight) quantize_weight;
    decltype(&::vq_gemm_f16) gemm_f16;
    decltype(&::vq_gemm_w8a8) gemm_w8a8;
    decltype(&::vq_gemm_w4a8) gemm_w4a8;
    decltype(&::vq_linear_workspace_bytes) linear_workspace_bytes;
    decltype(&::vq_linear) linear;
    decltype(&::vq_linear_static) linear_static;
    decltype(&::vq_layernorm_linear) layernorm_linear;
    decltype(&::vq_gelu_linear) gelu_linear;
    decltype(&::vq_residual_linear) residual_linear;
    decltype(&::vq_hadamard_linear) hadamard_linear;
} g_lib;
static_assert(sizeof(Entries) % sizeof(void*) == 0, "a plain array of addresses");
constexpr Py_ssize_t kEntries = sizeof(Entries) / sizeof(void*);

[[noreturn]] void fail(PyObject* type, const char* text) {
    PyErr_SetString(type, text);
    throw Raised{};
}

const char* dtype_name(at::ScalarType t) {
    switch (t) {
        case at::kHalf: return "torch.float16";
        case at::kFloat: return "torch.float32";
        case at::kDouble: return "torch.float64";
        case at::kBFloat16: return "torch.bfloat16";
        case at::kByte: return "torch.uint8";
        case at::kChar: return "torch.int8";
        case at::kShort: return "torch.int16";
        case at::kInt: return "torch.int32";
        case at::kLong: return "torch.int64";
        case at::kBool: return "torch.bool";
        default: return c10::toString(t);
    }
}

// A dense device tensor of the given type; None gives a null pointer.
const at::Tensor* device_tensor(PyObject* o, at::ScalarType dtype, const char* name) {
    if (o == Py_None) return nullptr;
    if (!THPVariable_Check(o) || !THPVariable_Unpack(o).is_cuda()) {
        PyErr_Format(PyExc_TypeError, "%s: expected a device tensor", name);
        throw Raised{};
    }
    const at::Tensor& t = THPVariable_Unpack(o);
    if (t.scalar_type() != dtype) {
        PyErr_Format(PyExc_TypeError, "%s: expected %s, got %s", name, dtype_name(dtype), dtype_name(t.scalar_type()));
        throw Raised{};
    }
    if (!t.is_contiguous()) {
        PyErr_Format(PyExc_ValueError, "%s: must be contiguous (dense row-major)", name);
        throw Raised{};
    }
    return &t;
}

// The same for an argument that cannot be left out.
const at::Tensor& required(PyObject* o, at::ScalarType dtype, const char* name) {
    const at::Tensor* t = device_tensor(o, dtype, name);
    if (!t) fail(PyExc_AttributeError, "'NoneType' object has no attribute 'shape'");
    return *t;
}

struct Rows {
    int64_t n, k;
};
Rows matrix(const at::Tensor& t) {
    if (t.dim() < 2) {
        PyErr_Format(PyExc_ValueError, "not enough values to unpack (expected 2, got %d)", (int)t.dim());
        throw Raised{};
    }
    if (t.dim() > 2) fail(PyExc_ValueError, "too many values to unpack (expected 2)");
    return {t.size(0), t.size(1)};
}
int64_t first_size(const at::Tensor& t) {
    if (t.dim() == 0) fail(PyExc_IndexError, "tuple index out of range");
    return t.size(0);
}

bool is_vector(const at::Tensor& t, int64_t n) { return t.dim() == 1 && t.size(0) == n; }
bool is_matrix(const at::Tensor& t, int64_t n, int64_t k) { return t.dim() == 2 && t.size(0) == n && t.size(1) == k; }

void* ptr(const at::Tensor& t) { return t.data_ptr(); }
void* ptr(const at::Tensor* t) { return t ? t->data_ptr() : nullptr; }
template <class T, class A>
T* as(const A& a) { return static_cast<T*>(ptr(a)); }

// The stream that a call enqueues on: the argument, or the current one.  Memory that the call allocates
// comes from that stream's: the caching allocator hands memory of the current stream out again without
// waiting for work on another, so scratch taken there would be given to the next allocation while this
// call's kernels still use it, and what it held before would be overwritten ahead of its readers.
class CallStream {
    PyObject* given_;

    void* given_handle() const {
        PyObject* raw = PyObject_GetAttrString(given_, "cuda_stream");
        if (!raw) throw Raised{};
        void* s = PyLong_AsVoidPtr(raw);
        Py_DECREF(raw);
        if (!s && PyErr_Occurred()) throw Raised{};
        return s;
    }
    c10::Stream given_stream(void* handle, c10::DeviceIndex device) const {
        if (THPStream_Check(given_)) {
            const THPStream* s = (const THPStream*)given_;
            return c10::Stream::unpack3(s->stream_id, (c10::DeviceIndex)s->device_index, (c10::DeviceType)s->device_type);
        }
        return c10::hip::getStreamFromExternalMasqueradingAsCUDA((hipStream_t)handle, device).unwrap();
    }

  public:
    explicit CallStream(PyObject* given) : given_(given) {}
    void* handle() const { return given_ == Py_None ? c10::hip::getCurrentHIPStream().stream() : given_handle(); }

    // `for_caller`: the current stream reads it next (behind whatever orders the two streams), and may
    // still do so when the caller lets go of it.
    at::Tensor empty(at::IntArrayRef shape, at::ScalarType dtype, const at::Tensor& like, bool for_caller) const {
        const auto options = like.options().dtype(dtype).requires_grad(false);
        if (given_ == Py_None) return at::empty(shape, options);
        void* const handle = given_handle();
        const auto current = c10::hip::getCurrentHIPStreamMasqueradingAsCUDA(like.device().index());
        if (current.stream() == handle) return at::empty(shape, options);
        at::Tensor t;
        {
            const c10::StreamGuard guard(given_stream(handle, like.device().index()));
            t = at::empty(shape, options);
        }
        if (for_caller) t.record_stream(current.unwrap());
        return t;
    }
};

// An output: the caller's tensor (checked), or a new one.
struct Output {
    PyObject* given = nullptr;
    at::Tensor t;
    Output() = default;
    Output(PyObject* o, at::IntArrayRef shape, at::ScalarType dtype, const char* name, const char* shape_error,
           const at::Tensor& like, const CallStream& stream) {
        if (o == Py_None) {
            t = stream.empty(shape, dtype, like, true);
        } else {
            given = o;
            t = *device_tensor(o, dtype, name);
            if (t.sizes() != shape) fail(PyExc_ValueError, shape_error);
        }
    }
    PyObject* release() {
        if (given) {
            Py_INCREF(given);
            return given;
        }
        return THPVariable_Wrap(std::move(t));
    }
};

[[noreturn]] void raise_status(int status, const char* where) {
    PyObject* e = PyObject_CallFunction(g_vq_error, "is", status, where);
    if (e) {
        PyErr_SetObject(g_vq_error, e);
        Py_DECREF(e);
    }
    throw Raised{};
}

// The interpreter lock is given up while this lives, and taken back however its scope is left.
struct Unlocked {
    PyThreadState* state = PyEval_SaveThread();
    Unlocked() = default;
    Unlocked(const Unlocked&) = delete;
    ~Unlocked() { PyEval_RestoreThread(state); }
};

// Enqueues without the interpreter lock (other threads go on, as under ctypes) and turns a
// status into VqError.  The arguments are plain values, all taken before the lock is given up: a
// tensor without storage (under a functorch transform, say) throws where its address is asked for.
template <class... P, class... A>
void enqueue(const char* where, int (*entry)(P...), A... args) {
    static_assert(sizeof...(P) == sizeof...(A));
    static_assert((std::is_scalar_v<A> && ...), "addresses and numbers");
    int status;
    {
        Unlocked unlocked;
        status = entry(static_cast<P>(args)...);
    }
    if (status != VQ_OK) raise_status(status, where);
}

// What float() takes, texts included.
double number(PyObject* o) {
    PyObject* f = PyNumber_Float(o);
    if (!f) throw Raised{};
    const double v = PyFloat_AS_DOUBLE(f);
    Py_DECREF(f);
    return v;
}

// 8 or 4; anything else is VQ_ERR_BITS.
int weight_bits(PyObject* o, const char* where) {
    const double v = PyFloat_AsDouble(o);
    if (PyErr_Occurred()) PyErr_Clear();
    if (v == 8.0) return 8;
    if (v == 4.0) return 4;
    raise_status(VQ_ERR_BITS, where);
}

bool truth(PyObject* o) {
    const int t = PyObject_IsTrue(o);
    if (t < 0) throw Raised{};
    return t != 0;
}

// Tokens that share a row of the per-sample arrays: all of them if not given.  What does not fit the
// library's int is VQ_ERR_SHAPE here: narrowed, it would be another length, or 0.
int tokens_per_sample(PyObject* o, int64_t M, const char* where) {
    if (!truth(o)) return (int)std::max<int64_t>(M, 1);
    PyObject* l = PyNumber_Long(o);
    if (!l) throw Raised{};
    int overflow = 0;
    const long v = PyLong_AsLongAndOverflow(l, &overflow);
    Py_DECREF(l);
    if (v == -1 && PyErr_Occurred()) throw Raised{};
    if (overflow || v < INT_MIN || v > INT_MAX) raise_status(VQ_ERR_SHAPE, where);
    return (int)v;
}

const at::Tensor* per_sample(PyObject* o, int64_t M, int64_t K, int T, const char* name) {
    const at::Tensor* t = device_tensor(o, at::kFloat, name);
    if (!t) return nullptr;   // (a length that is not positive is left to the library's check)
    if (T == 0) fail(PyExc_ZeroDivisionError, "integer division or modulo by zero");   // (0.5, say)
    const int64_t up = M + T - 1, q = up / T, rows = q - (up % T != 0 && (up < 0) != (T < 0));  // floor
    if (!is_matrix(*t, rows, K)) {
        PyErr_Format(PyExc_ValueError, "%s must have shape [ceil(M / tokens_per_sample), K]", name);
        throw Raised{};
    }
    return t;
}

const at::Tensor* channel_vector(PyObject* o, int64_t K, const char* name) {
    const at::Tensor* t = device_tensor(o, at::kFloat, name);
    if (t && !is_vector(*t, K)) {
        PyErr_Format(PyExc_ValueError, "%s must have shape [K]", name);
        throw Raised{};
    }
    return t;
}

PyObject* tuple_of(PyObject* a, PyObject* b, PyObject* c = nullptr) {
    PyObject* t = c ? PyTuple_Pack(3, a, b, c) : PyTuple_Pack(2, a, b);
    Py_XDECREF(a);
    Py_XDECREF(b);
    Py_XDECREF(c);
    return t;
}

// What every quantizer returns: codes and token scales.
struct Codes {
    const at::Tensor* chan_mul;
    Output xq, x_scale;
    Codes(const at::Tensor& x, Rows r, PyObject* cm, PyObject* xq_o, PyObject* xs_o, const CallStream& st) {
        chan_mul = channel_vector(cm, r.k, "chan_mul");
        xq = Output(xq_o, {r.n, r.k}, at::kChar, "xq", "output shapes", x, st);
        x_scale = Output(xs_o, {r.n}, at::kFloat, "x_scale", "output shapes", x, st);
    }
    const float* cm() const { return as<float>(chan_mul); }
    int8_t* q() const { return as<int8_t>(xq.t); }
    float* s() const { return as<float>(x_scale.t); }
};

// ---- entry points: positional arguments only, as binding.py passes them -----------------------

PyObject* quantize_per_token(PyObject* const* a) {  // x chan_mul xq x_scale stream
    const CallStream st(a[4]);
    const at::Tensor& x = required(a[0], at::kHalf, "x");
    const Rows r = matrix(x);
    Codes c(x, r, a[1], a[2], a[3], st);
    enqueue("vq_quantize_per_token", g_lib.quantize_per_token, ptr(x), c.cm(), c.q(), c.s(), (int)r.n, (int)r.k,
            st.handle());
    return tuple_of(c.xq.release(), c.x_scale.release());
}

PyObject* gelu_quantize(PyObject* const* a) {  // h approximate chan_mul xq x_scale stream
    const CallStream st(a[5]);
    const at::Tensor& x = required(a[0], at::kHalf, "h");
    const Rows r = matrix(x);
    Codes c(x, r, a[2], a[3], a[4], st);
    const int approximate = truth(a[1]);
    enqueue("vq_gelu_quantize", g_lib.gelu_quantize, ptr(x), approximate, c.cm(), c.q(), c.s(), (int)r.n, (int)r.k,
            st.handle());
    return tuple_of(c.xq.release(), c.x_scale.release());
}

PyObject* layernorm_quantize(PyObject* const* a) {  // x mod_scale mod_shift T eps chan_mul xq x_scale stream
    const CallStream st(a[8]);
    const at::Tensor& x = required(a[0], at::kHalf, "x");
    const Rows r = matrix(x);
    const int T = tokens_per_sample(a[3], r.n, "vq_layernorm_quantize");
    const at::Tensor* scale = per_sample(a[1], r.n, r.k, T, "mod_scale");
    const at::Tensor* shift = per_sample(a[2], r.n, r.k, T, "mod_shift");
    Codes c(x, r, a[5], a[6], a[7], st);
    const float eps = (float)number(a[4]);
    enqueue("vq_layernorm_quantize", g_lib.layernorm_quantize, ptr(x), as<float>(scale), as<float>(shift), T, eps, c.cm(),
            c.q(), c.s(), (int)r.n, (int)r.k, st.handle());
    return tuple_of(c.xq.release(), c.x_scale.release());
}

PyObject* residual_quantize(PyObject* const* a) {  // x y gate T r chan_mul xq x_scale stream
    const CallStream st(a[8]);
    const at::Tensor& x = required(a[0], at::kHalf, "x");
    const at::Tensor* y = device_tensor(a[1], at::kHalf, "y");
    if (!y || y->sizes() != x.sizes()) fail(PyExc_ValueError, "y must have the shape of x");
    const Rows r = matrix(x);
    const int T = tokens_per_sample(a[3], r.n, "vq_residual_quantize");
    const at::Tensor* gate = per_sample(a[2], r.n, r.k, T, "gate");
    Output res(a[4], {r.n, r.k}, at::kHalf, "r", "r must have the shape of x", x, st);
    Codes c(x, r, a[5], a[6], a[7], st);
    enqueue("vq_residual_quantize", g_lib.residual_quantize, ptr(x), ptr(y), as<float>(gate), T, ptr(res.t), c.cm(), c.q(),
            c.s(), (int)r.n, (int)r.k, st.handle());
    return tuple_of(res.release(), c.xq.release(), c.x_scale.release());
}

PyObject* hadamard_quantize(PyObject* const* a) {  // x chan_mul xq x_scale stream
    const CallStream st(a[4]);
    const at::Tensor& x = required(a[0], at::kHalf, "x");
    const Rows r = matrix(x);
    Codes c(x, r, a[1], a[2], a[3], st);
    enqueue("vq_hadamard_quantize", g_lib.hadamard_quantize, ptr(x), c.cm(), c.q(), c.s(), (int)r.n, (int)r.k, st.handle());
    return tuple_of(c.xq.release(), c.x_scale.release());
}

PyObject* quantize_static(PyObject* const* a) {  // x scale chan_mul xq stream
    const CallStream st(a[4]);
    const at::Tensor& x = required(a[0], at::kHalf, "x");
    const Rows r = matrix(x);
    const at::Tensor* cm = channel_vector(a[2], r.k, "chan_mul");
    Output xq(a[3], {r.n, r.k}, at::kChar, "xq", "xq must have shape [M,K]", x, st);
    const float scale = (float)number(a[1]);
    enqueue("vq_quantize_static", g_lib.quantize_static, ptr(x), as<float>(cm), scale, as<int8_t>(xq.t), (int)r.n,
            (int)r.k, st.handle());
    return xq.release();
}

PyObject* channel_absmax(PyObject* const* a) {  // a amax accumulate stream
    const CallStream st(a[3]);
    if (!THPVariable_Check(a[0]) || (THPVariable_Unpack(a[0]).scalar_type() != at::kHalf &&
                                     THPVariable_Unpack(a[0]).scalar_type() != at::kFloat))
        fail(PyExc_TypeError, "a: expected a float16 or float32 device tensor");
    const at::ScalarType dtype = THPVariable_Unpack(a[0]).scalar_type();
    const at::Tensor& m = required(a[0], dtype, "a");
    const Rows r = matrix(m);
    const int accumulate = truth(a[2]);
    if (a[1] == Py_None && accumulate) fail(PyExc_ValueError, "accumulate needs the running amax");
    Output amax(a[1], {r.k}, at::kFloat, "amax", "amax must have shape [K]", m, st);
    enqueue("vq_channel_absmax", g_lib.channel_absmax, ptr(m), (int)(dtype == at::kFloat), as<float>(amax.t), (int)r.n,
            (int)r.k, accumulate, st.handle());
    return amax.release();
}

PyObject* balance_mask(PyObject* const* a) {  // amax_x amax_w alpha stream
    const CallStream st(a[3]);
    const at::Tensor& ax = required(a[0], at::kFloat, "amax_x");
    const at::Tensor& aw = required(a[1], at::kFloat, "amax_w");
    const int64_t K = first_size(ax);
    if (!is_vector(ax, K) || !is_vector(aw, K)) fail(PyExc_ValueError, "statistics must have shape [K]");
    Output s(Py_None, {K}, at::kFloat, "s", "", ax, st), cm(Py_None, {K}, at::kFloat, "chan_mul", "", ax, st);
    const float alpha = (float)number(a[2]);
    enqueue("vq_balance_mask", g_lib.balance_mask, as<float>(ax), as<float>(aw), alpha, as<float>(s.t), as<float>(cm.t),
            (int)K, st.handle());
    return tuple_of(s.release(), cm.release());
}

PyObject* rotate_weight(PyObject* const* a) {  // w chan_s out stream
    const CallStream st(a[3]);
    const at::Tensor& w = required(a[0], at::kFloat, "w");
    const Rows r = matrix(w);
    const at::Tensor* s = channel_vector(a[1], r.k, "chan_s");
    Output out(a[2], {r.n, r.k}, at::kFloat, "out", "out must have the shape of w", w, st);
    enqueue("vq_rotate_weight", g_lib.rotate_weight, as<float>(w), as<float>(s), as<float>(out.t), (int)r.n, (int)r.k,
            st.handle());
    return out.release();
}

PyObject* quantize_weight(PyObject* const* a) {  // w chan_s w_bits stream
    const CallStream st(a[3]);
    const at::Tensor& w = required(a[0], at::kFloat, "w");
    const Rows r = matrix(w);
    const at::Tensor* s = channel_vector(a[1], r.k, "chan_s");
    const int bits = weight_bits(a[2], "vq_quantize_weight");
    Output wq = bits == 8 ? Output(Py_None, {r.n, r.k}, at::kChar, "wq", "", w, st)
                          : Output(Py_None, {r.n, r.k / 2}, at::kByte, "wq", "", w, st);
    Output ws(Py_None, {r.n}, at::kFloat, "w_scale", "", w, st);
    enqueue("vq_quantize_weight", g_lib.quantize_weight, as<float>(w), as<float>(s), bits, ptr(wq.t), as<float>(ws.t),
            (int)r.n, (int)r.k, st.handle());
    return tuple_of(wq.release(), ws.release());
}

PyObject* gemm_f16(PyObject* const* a) {  // x w bias y stream
    const CallStream st(a[4]);
    const at::Tensor& x = required(a[0], at::kHalf, "x");
    const at::Tensor& w = required(a[1], at::kHalf, "w");
    const Rows r = matrix(x);
    const int64_t N = first_size(w);
    if (!is_matrix(w, N, r.k)) fail(PyExc_ValueError, "weight shape does not match K");
    const at::Tensor* bias = device_tensor(a[2], at::kHalf, "bias");
    if (bias && !is_vector(*bias, N)) fail(PyExc_ValueError, "bias must have shape [N]");
    Output y(a[3], {r.n, N}, at::kHalf, "y", "y must have shape [M,N]", x, st);
    enqueue("vq_gemm_f16", g_lib.gemm_f16, ptr(x), ptr(w), ptr(bias), ptr(y.t), (int)r.n, (int)N, (int)r.k, st.handle());
    return y.release();
}

PyObject* gemm(PyObject* const* a, int bits) {  // xq x_scale w w_scale bias y return_acc stream
    const CallStream st(a[7]);
    const at::Tensor& xq = required(a[0], at::kChar, "xq");
    const Rows r = matrix(xq);
    const at::Tensor& w = required(a[2], bits == 8 ? at::kChar : at::kByte, "w");
    const int64_t N = first_size(w), div = bits == 8 ? 1 : 2;
    if (!is_matrix(w, N, r.k / div) || r.k % div) fail(PyExc_ValueError, "weight shape does not match K");
    const at::Tensor* x_scale = device_tensor(a[1], at::kFloat, "x_scale");
    const at::Tensor* w_scale = device_tensor(a[3], at::kFloat, "w_scale");
    const at::Tensor* bias = device_tensor(a[4], at::kHalf, "bias");
    if (!x_scale || !w_scale) fail(PyExc_AttributeError, "'NoneType' object has no attribute 'shape'");
    if (!is_vector(*x_scale, r.n) || !is_vector(*w_scale, N) || (bias && !is_vector(*bias, N)))
        fail(PyExc_ValueError, "scale / bias shapes");
    Output y(a[5], {r.n, N}, at::kHalf, "y", "y shape", xq, st);
    const bool want_acc = truth(a[6]);
    Output acc;
    if (want_acc) acc = Output(Py_None, {r.n, N}, at::kInt, "acc", "", xq, st);
    int32_t* acc_ptr = want_acc ? as<int32_t>(acc.t) : nullptr;
    if (bits == 8)
        enqueue("vq_gemm_w8a8", g_lib.gemm_w8a8, as<int8_t>(xq), as<float>(x_scale), as<int8_t>(w), as<float>(w_scale),
                ptr(bias), ptr(y.t), acc_ptr, (int)r.n, (int)N, (int)r.k, st.handle());
    else
        enqueue("vq_gemm_w4a8", g_lib.gemm_w4a8, as<int8_t>(xq), as<float>(x_scale), as<uint8_t>(w), as<float>(w_scale),
                ptr(bias), ptr(y.t), acc_ptr, (int)r.n, (int)N, (int)r.k, st.handle());
    return want_acc ? tuple_of(y.release(), acc.release()) : y.release();
}
PyObject* gemm_w8a8(PyObject* const* a) { return gemm(a, 8); }
PyObject* gemm_w4a8(PyObject* const* a) { return gemm(a, 4); }

// What every layer call takes.
struct Layer {
    const at::Tensor* x;
    const at::Tensor* chan_mul;
    const at::Tensor* w;
    const at::Tensor* w_scale;
    const at::Tensor* bias;
    Output y;
    int bits, M, N, K;
    at::Tensor workspace;
    Layer(PyObject* x_o, PyObject* cm_o, PyObject* w_o, PyObject* bits_o, PyObject* ws_o, PyObject* bias_o, PyObject* y_o,
          const CallStream& st, const char* where) {
        x = &required(x_o, at::kHalf, "x");
        const Rows r = matrix(*x);
        bits = weight_bits(bits_o, where);
        w = &required(w_o, bits == 8 ? at::kChar : at::kByte, "w");
        if (w->dim() != 2 || (bits == 4 && r.k % 2) || w->size(1) != (bits == 8 ? r.k : r.k / 2))
            fail(PyExc_ValueError, "weight shape does not match K");
        const int64_t n = w->size(0);
        chan_mul = device_tensor(cm_o, at::kFloat, "chan_mul");
        w_scale = &required(ws_o, at::kFloat, "w_scale");
        bias = device_tensor(bias_o, at::kHalf, "bias");
        if ((chan_mul && !is_vector(*chan_mul, r.k)) || !is_vector(*w_scale, n) || (bias && !is_vector(*bias, n)))
            fail(PyExc_ValueError, "chan_mul / scale / bias shapes");
        y = Output(y_o, {r.n, n}, at::kHalf, "y", "y shape", *x, st);
        M = (int)r.n, N = (int)n, K = (int)r.k;
    }
    void take_workspace(PyObject* o, const CallStream& st) {
        if (o == Py_None) {
            const int64_t need = (int64_t)g_lib.linear_workspace_bytes(M, N, K, bits);
            workspace = st.empty({std::max<int64_t>(need, 16)}, at::kByte, *x, false);
        } else {
            workspace = *device_tensor(o, at::kByte, "workspace");
        }
    }
    const float* cm() const { return as<float>(chan_mul); }
    const float* ws() const { return as<float>(w_scale); }
    size_t workspace_bytes() const { return (size_t)workspace.numel(); }
};

PyObject* linear(PyObject* const* a) {  // x chan_mul w w_bits w_scale bias y workspace stream
    const CallStream st(a[8]);
    Layer l(a[0], a[1], a[2], a[3], a[4], a[5], a[6], st, "vq_linear");
    l.take_workspace(a[7], st);
    enqueue("vq_linear", g_lib.linear, ptr(l.x), l.cm(), ptr(l.w), l.bits, l.ws(), ptr(l.bias), ptr(l.y.t),
            ptr(l.workspace), l.workspace_bytes(), l.M, l.N, l.K, st.handle());
    return l.y.release();
}

PyObject* linear_static(PyObject* const* a) {  // x chan_mul w w_bits w_scale bias y stream
    const CallStream st(a[7]);
    Layer l(a[0], a[1], a[2], a[3], a[4], a[5], a[6], st, "vq_linear_static");
    enqueue("vq_linear_static", g_lib.linear_static, ptr(l.x), l.cm(), ptr(l.w), l.bits, l.ws(), ptr(l.bias), ptr(l.y.t),
            l.M, l.N, l.K, st.handle());
    return l.y.release();
}

PyObject* layernorm_linear(PyObject* const* a) {  // x w w_bits w_scale mod_scale mod_shift T eps chan_mul bias y workspace stream
    const CallStream st(a[12]);
    Layer l(a[0], a[8], a[1], a[2], a[3], a[9], a[10], st, "vq_layernorm_linear");
    const int T = tokens_per_sample(a[6], l.M, "vq_layernorm_linear");
    const at::Tensor* scale = per_sample(a[4], l.M, l.K, T, "mod_scale");
    const at::Tensor* shift = per_sample(a[5], l.M, l.K, T, "mod_shift");
    l.take_workspace(a[11], st);
    const float eps = (float)number(a[7]);
    enqueue("vq_layernorm_linear", g_lib.layernorm_linear, ptr(l.x), as<float>(scale), as<float>(shift), T, eps, l.cm(),
            ptr(l.w), l.bits, l.ws(), ptr(l.bias), ptr(l.y.t), ptr(l.workspace), l.workspace_bytes(), l.M, l.N, l.K, st.handle());
    return l.y.release();
}

PyObject* gelu_linear(PyObject* const* a) {  // h w w_bits w_scale approximate chan_mul bias y workspace stream
    const CallStream st(a[9]);
    Layer l(a[0], a[5], a[1], a[2], a[3], a[6], a[7], st, "vq_gelu_linear");
    l.take_workspace(a[8], st);
    const int approximate = truth(a[4]);
    enqueue("vq_gelu_linear", g_lib.gelu_linear, ptr(l.x), approximate, l.cm(), ptr(l.w), l.bits, l.ws(), ptr(l.bias),
            ptr(l.y.t), ptr(l.workspace), l.workspace_bytes(), l.M, l.N, l.K, st.handle());
    return l.y.release();
}

PyObject* residual_linear(PyObject* const* a) {  // x y_in w w_bits w_scale gate T r chan_mul bias y workspace stream
    const CallStream st(a[12]);
    Layer l(a[0], a[8], a[2], a[3], a[4], a[9], a[10], st, "vq_residual_linear");
    const at::Tensor* y_in = device_tensor(a[1], at::kHalf, "y_in");
    if (!y_in || !is_matrix(*y_in, l.M, l.K)) fail(PyExc_ValueError, "y_in must have the shape of x");
    const int T = tokens_per_sample(a[6], l.M, "vq_residual_linear");
    const at::Tensor* gate = per_sample(a[5], l.M, l.K, T, "gate");
    Output r(a[7], {l.M, l.K}, at::kHalf, "r", "r must have the shape of x", *l.x, st);
    l.take_workspace(a[11], st);
    enqueue("vq_residual_linear", g_lib.residual_linear, ptr(l.x), ptr(y_in), as<float>(gate), T, ptr(r.t), l.cm(),
            ptr(l.w), l.bits, l.ws(), ptr(l.bias), ptr(l.y.t), ptr(l.workspace), l.workspace_bytes(), l.M, l.N, l.K, st.handle());
    return tuple_of(r.release(), l.y.release());
}

PyObject* hadamard_linear(PyObject* const* a) {  // x chan_mul w w_bits w_scale bias y workspace stream
    const CallStream st(a[8]);
    Layer l(a[0], a[1], a[2], a[3], a[4], a[5], a[6], st, "vq_hadamard_linear");
    l.take_workspace(a[7], st);
    enqueue("vq_hadamard_linear", g_lib.hadamard_linear, ptr(l.x), l.cm(), ptr(l.w), l.bits, l.ws(), ptr(l.bias),
            ptr(l.y.t), ptr(l.workspace), l.workspace_bytes(), l.M, l.N, l.K, st.handle());
    return l.y.release();
}

// ---- module ------------------------------------------------------------------------------------

// bind(vq_error, addresses): the exception class and the entry points' addresses in Entries' order.
PyObject* bind(PyObject*, PyObject* args) {
    PyObject *error, *list;
    if (!PyArg_ParseTuple(args, "OO!", &error, &PyTuple_Type, &list)) return nullptr;
    if (PyTuple_GET_SIZE(list) != kEntries) {
        PyErr_SetString(PyExc_ValueError, "one address per entry point");
        return nullptr;
    }
    void* addresses[kEntries];
    for (Py_ssize_t i = 0; i < kEntries; ++i) {
        addresses[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(list, i));
        if (!addresses[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null entry point");
            return nullptr;
        }
    }
    memcpy(&g_lib, addresses, sizeof(g_lib));
    Py_INCREF(error);
    Py_XDECREF(g_vq_error);
    g_vq_error = error;
    Py_RETURN_NONE;
}

template <PyObject* (*F)(PyObject* const*), Py_ssize_t ARGS>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t n) {
    if (n != ARGS) {
        PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", ARGS, n);
        return nullptr;
    }
    try {
        return F(args);
    } catch (const Raised&) {
    } catch (const std::exception&) {  // torch's own (out of memory, ...)
        torch::translate_exception_to_python(std::current_exception());
    } catch (...) {
        PyErr_SetString(PyExc_RuntimeError, "unknown C++ exception");
    }
    return nullptr;
}

#define VQ_ENTRY(name, args) {#name, (PyCFunction)(void (*)(void))entry<name, args>, METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {
    {"bind", bind, METH_VARARGS, nullptr},
    VQ_ENTRY(quantize_per_token, 5),
    VQ_ENTRY(gelu_quantize, 6),
    VQ_ENTRY(layernorm_quantize, 9),
    VQ_ENTRY(residual_quantize, 9),
    VQ_ENTRY(hadamard_quantize, 5),
    VQ_ENTRY(quantize_static, 5),
    VQ_ENTRY(channel_absmax, 4),
    VQ_ENTRY(balance_mask, 4),
    VQ_ENTRY(rotate_weight, 4),
    VQ_ENTRY(quantize_weight, 4),
    VQ_ENTRY(gemm_f16, 5),
    VQ_ENTRY(gemm_w8a8, 8),
    VQ_ENTRY(gemm_w4a8, 8),
    VQ_ENTRY(linear, 9),
    VQ_ENTRY(linear_static, 8),
    VQ_ENTRY(layernorm_linear, 13),
    VQ_ENTRY(gelu_linear, 10),
    VQ_ENTRY(residual_linear, 13),
    VQ_ENTRY(hadamard_linear, 9),
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_vq_torch", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__vq_torch(void) {
    PyObject* m = PyModule_Create(&g_module);
    if (m && PyModule_AddStringConstant(m, "TORCH_VERSION", TORCH_VERSION) < 0) Py_CLEAR(m);
    return m;
}
