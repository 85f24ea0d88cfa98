// The argument marshalling of binding.py's hot entry points, in C++: tensor checks, output allocation, the current HIP stream
// and the call through the C ABI.  A decode launch on a small layer takes the GPU four to five microseconds; done in Python
// (a dozen attribute reads, two torch calls and the ctypes conversion) the marshalling took six and a half of the 10.7 us
// that linear_fused on 1536 -> 4096 took per call; now the call takes 5.0, of which the launch itself is 4.3.
//
// binding.load() hands over the C ABI's function addresses (bind) -- the library stays whichever one it loaded -- and its
// BitnetError class.  The checks, their order and their messages are those of binding.py's own helpers.  The GIL is released
// around the call, as ctypes does.
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "bitnet.h"

namespace {

struct Abi {
    decltype(&bitnet_quantize_acts) quantize_acts;
    decltype(&bitnet_rmsnorm_quantize) rmsnorm_quantize;
    decltype(&bitnet_swiglu_quantize) swiglu_quantize;
    decltype(&bitnet_linear) linear;
    decltype(&bitnet_linear_variant) linear_variant;
    decltype(&bitnet_linear_segmented) linear_segmented;
    decltype(&bitnet_linear_ws) linear_ws;
    decltype(&bitnet_linear_fused) linear_fused;
    decltype(&bitnet_linear_fused_segmented) linear_fused_segmented;
    decltype(&bitnet_rmsnorm_linear_fused) rmsnorm_linear_fused;
    decltype(&bitnet_rmsnorm_linear_fused_segmented) rmsnorm_linear_fused_segmented;
    decltype(&bitnet_swiglu_linear_fused) swiglu_linear_fused;
    decltype(&bitnet_ffn_gate_up_fused) ffn_gate_up_fused;
} abi;
PyObject* error_class = nullptr;

// A Python exception is set: unwinds to the entry point, which returns NULL.
struct Raised {};
template <typename... A>
[[noreturn]] void raise(PyObject* type, const char* fmt, A... a) {
    PyErr_Format(type, fmt, a...);
    throw Raised();
}

const char* dtype_name(at::ScalarType t) {
    switch (t) {
        case at::kFloat: return "torch.float32";
        case at::kDouble: return "torch.float64";
        case at::kHalf: return "torch.float16";
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

const at::Tensor& tensor(PyObject* o, const char* name) {
    if (!THPVariable_Check(o)) raise(PyExc_TypeError, "%s must be a CUDA/HIP tensor", name);
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_cuda()) raise(PyExc_TypeError, "%s must be a CUDA/HIP tensor", name);
    if (!t.is_contiguous()) raise(PyExc_ValueError, "%s must be contiguous", name);
    return t;
}
const at::Tensor& tensor(PyObject* o, const char* name, at::ScalarType dt) {
    const at::Tensor& t = tensor(o, name);
    if (t.scalar_type() != dt) raise(PyExc_TypeError, "%s has dtype %s", name, dtype_name(t.scalar_type()));
    return t;
}
void two_d(const at::Tensor& t, const char* name) {
    if (t.dim() != 2) raise(PyExc_ValueError, "%s must be 2-D", name);
}
// a float matrix: fp32 or bf16, two dimensions
const at::Tensor& matrix(PyObject* o, const char* name, bitnet_dtype* dt) {
    const at::Tensor& t = tensor(o, name);
    if (t.scalar_type() == at::kFloat) *dt = BITNET_F32;
    else if (t.scalar_type() == at::kBFloat16) *dt = BITNET_BF16;
    else raise(PyExc_TypeError, "%s has dtype %s", name, dtype_name(t.scalar_type()));
    two_d(t, name);
    return t;
}
const at::Tensor& int8_matrix(PyObject* o, const char* name) {
    const at::Tensor& t = tensor(o, name, at::kChar);
    two_d(t, name);
    return t;
}

int64_t integer(PyObject* o) {
    PyObject* i = PyNumber_Index(o);
    if (!i) throw Raised();
    const unsigned long long v = PyLong_AsUnsignedLongLongMask(i);
    Py_DECREF(i);
    if (v == (unsigned long long)-1 && PyErr_Occurred()) throw Raised();
    return (int64_t)v;
}
float real(PyObject* o) {
    PyObject* f = PyNumber_Float(o);
    if (!f) throw Raised();
    const double v = PyFloat_AS_DOUBLE(f);
    Py_DECREF(f);
    return (float)v;
}
bool truth(PyObject* o) {
    const int v = PyObject_IsTrue(o);
    if (v < 0) throw Raised();
    return v != 0;
}

at::ScalarType out_type(PyObject* code) {
    if (PyIndex_Check(code)) {
        switch (integer(code)) {
            case BITNET_F32: return at::kFloat;
            case BITNET_BF16: return at::kBFloat16;
            case BITNET_I32: return at::kInt;
            default: break;
        }
    }
    PyErr_SetObject(PyExc_KeyError, code);
    throw Raised();
}
// the caller's output tensor, or a new one on x's device
at::Tensor output(PyObject* given, const char* name, at::IntArrayRef shape, at::ScalarType dt, const at::Tensor& x) {
    if (given == Py_None) return at::empty(shape, at::TensorOptions().dtype(dt).device(x.device()));
    return tensor(given, name, dt);
}
const float* gain(PyObject* g, int64_t K, bool check_shape) {
    if (g == Py_None) return nullptr;
    const at::Tensor& t = tensor(g, "g", at::kFloat);
    if (check_shape && (t.dim() != 1 || t.size(0) != K)) raise(PyExc_ValueError, "g must have one entry per column");
    return static_cast<const float*>(t.const_data_ptr());
}
const float* floats(PyObject* o, const char* name) { return static_cast<const float*>(tensor(o, name, at::kFloat).const_data_ptr()); }
const float* per_block(PyObject* o, const char* name, int64_t N) {
    const at::Tensor& t = tensor(o, name, at::kFloat);
    if (t.numel() < (N + 15) / 16) raise(PyExc_ValueError, "%s needs one entry per 16-row block", name);
    return static_cast<const float*>(t.const_data_ptr());
}

void* stream() { return c10::hip::getCurrentHIPStream().stream(); }

// other threads may run until it goes out of scope, however that happens
struct GilReleased {
    PyThreadState* state = PyEval_SaveThread();
    ~GilReleased() { PyEval_RestoreThread(state); }
};

template <typename F>
void call(const char* where, F&& f) {
    const bitnet_status st = [&] { GilReleased released; return f(); }();
    if (st == BITNET_OK) return;
    PyObject* e = PyObject_CallFunction(error_class, "is", (int)st, where);
    if (e) {
        PyErr_SetObject(error_class, e);
        Py_DECREF(e);
    }
    throw Raised();
}

// Every entry point: a fixed number of positional arguments; C++ exceptions become Python ones.
template <typename F>
PyObject* entry(Py_ssize_t n, Py_ssize_t want, F&& f) {
    HANDLE_TH_ERRORS
    if (!error_class) {
        PyErr_SetString(PyExc_RuntimeError, "bind() has not been called");
        return nullptr;
    }
    if (n != want) {
        PyErr_Format(PyExc_TypeError, "%zd arguments expected", want);
        return nullptr;
    }
    try {
        return f();
    } catch (const Raised&) {
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}
PyObject* pair(const at::Tensor& a, const at::Tensor& b) {
    PyObject* pa = THPVariable_Wrap(a);
    PyObject* pb = pa ? THPVariable_Wrap(b) : nullptr;
    PyObject* t = pb ? PyTuple_Pack(2, pa, pb) : nullptr;
    Py_XDECREF(pa);
    Py_XDECREF(pb);
    return t;
}

#define ENTRY(name_) PyObject* name_(PyObject*, PyObject* const* a, Py_ssize_t n)

ENTRY(quantize_acts) {      // x, xq, sx
    return entry(n, 3, [&] {
        bitnet_dtype dt;
        const at::Tensor& x = matrix(a[0], "x", &dt);
        const int64_t M = x.size(0), K = x.size(1);
        at::Tensor xq = output(a[1], "xq", {M, K}, at::kChar, x), sx = output(a[2], "sx", {M}, at::kFloat, x);
        const void* xp = x.const_data_ptr();
        int8_t* qp = static_cast<int8_t*>(xq.mutable_data_ptr());
        float* sp = static_cast<float*>(sx.mutable_data_ptr());
        void* st = stream();
        call("bitnet_quantize_acts", [&] { return abi.quantize_acts(xp, dt, M, K, qp, sp, st); });
        return pair(xq, sx);
    });
}

ENTRY(rmsnorm_quantize) {      // x, g, eps, xq, sx
    return entry(n, 5, [&] {
        bitnet_dtype dt;
        const at::Tensor& x = matrix(a[0], "x", &dt);
        const int64_t M = x.size(0), K = x.size(1);
        at::Tensor xq = output(a[3], "xq", {M, K}, at::kChar, x), sx = output(a[4], "sx", {M}, at::kFloat, x);
        const float* g = gain(a[1], K, true);
        const float eps = real(a[2]);
        const void* xp = x.const_data_ptr();
        int8_t* qp = static_cast<int8_t*>(xq.mutable_data_ptr());
        float* sp = static_cast<float*>(sx.mutable_data_ptr());
        void* st = stream();
        call("bitnet_rmsnorm_quantize", [&] { return abi.rmsnorm_quantize(xp, dt, g, eps, M, K, qp, sp, st); });
        return pair(xq, sx);
    });
}

ENTRY(swiglu_quantize) {      // gu, hq, sh
    return entry(n, 3, [&] {
        bitnet_dtype dt;
        const at::Tensor& gu = matrix(a[0], "gu", &dt);
        const int64_t M = gu.size(0);
        if (gu.size(1) % 2) raise(PyExc_ValueError, "gu must have an even number of columns");
        const int64_t F = gu.size(1) / 2;
        at::Tensor hq = output(a[1], "hq", {M, F}, at::kChar, gu), sh = output(a[2], "sh", {M}, at::kFloat, gu);
        const void* gp = gu.const_data_ptr();
        int8_t* qp = static_cast<int8_t*>(hq.mutable_data_ptr());
        float* sp = static_cast<float*>(sh.mutable_data_ptr());
        void* st = stream();
        call("bitnet_swiglu_quantize", [&] { return abi.swiglu_quantize(gp, dt, M, F, qp, sp, st); });
        return pair(hq, sh);
    });
}

// the product's operands that every linear entry point shares
struct Product {
    const at::Tensor& xq;
    int64_t M, K, N;
    at::Tensor y;
    const int8_t* xp;
    const float* sx;
    const void* packed;
    void* yp;
    bitnet_format f;
    bitnet_dtype yt;
    Product(PyObject* oxq, PyObject* osx, PyObject* opacked, PyObject* oN, PyObject* ofmt, PyObject* oyt, PyObject* oy)
        : xq(int8_matrix(oxq, "xq")), M(xq.size(0)), K(xq.size(1)), N(integer(oN)), y(output(oy, "y", {M, N}, out_type(oyt), xq)),
          xp(static_cast<const int8_t*>(xq.const_data_ptr())), sx(floats(osx, "sx")),
          packed(tensor(opacked, "packed").const_data_ptr()), yp(y.mutable_data_ptr()), f((bitnet_format)(int)integer(ofmt)),
          yt((bitnet_dtype)(int)integer(oyt)) {}
};

ENTRY(linear) {      // xq, sx, packed, gamma, N, fmt, y_dtype, y, kernel
    return entry(n, 9, [&] {
        Product p(a[0], a[1], a[2], a[4], a[5], a[6], a[7]);
        const float* gamma = floats(a[3], "gamma");
        const bitnet_kernel which = (bitnet_kernel)(int)integer(a[8]);
        void* st = stream();
        if (which == BITNET_KERNEL_AUTO)
            call("bitnet_linear", [&] { return abi.linear(p.xp, p.sx, p.packed, gamma, p.M, p.N, p.K, p.f, p.yp, p.yt, st); });
        else
            call("bitnet_linear_variant", [&] { return abi.linear_variant(p.xp, p.sx, p.packed, gamma, p.M, p.N, p.K, p.f, p.yp, p.yt, which, st); });
        return THPVariable_Wrap(p.y);
    });
}

ENTRY(linear_segmented) {      // xq, sx, packed, gamma_rb, N, fmt, y_dtype, y, kernel
    return entry(n, 9, [&] {
        Product p(a[0], a[1], a[2], a[4], a[5], a[6], a[7]);
        const float* gamma = per_block(a[3], "gamma_rb", p.N);
        const bitnet_kernel which = (bitnet_kernel)(int)integer(a[8]);
        void* st = stream();
        call("bitnet_linear_segmented", [&] { return abi.linear_segmented(p.xp, p.sx, p.packed, gamma, p.M, p.N, p.K, p.f, p.yp, p.yt, which, st); });
        return THPVariable_Wrap(p.y);
    });
}

ENTRY(linear_ws) {      // xq, sx, packed, gamma, N, fmt, y_dtype, y, kernel, workspace, gamma_per_block
    return entry(n, 11, [&] {
        Product p(a[0], a[1], a[2], a[4], a[5], a[6], a[7]);
        const float* gamma = floats(a[3], "gamma");
        const bitnet_kernel which = (bitnet_kernel)(int)integer(a[8]);
        void* ws = nullptr;
        size_t bytes = 0;
        if (a[9] != Py_None) {
            const at::Tensor& w = tensor(a[9], "workspace");
            ws = w.mutable_data_ptr();
            bytes = (size_t)w.numel() * w.element_size();
        }
        const int per = truth(a[10]) ? 1 : 0;
        void* st = stream();
        call("bitnet_linear_ws", [&] { return abi.linear_ws(p.xp, p.sx, p.packed, gamma, per, p.M, p.N, p.K, p.f, p.yp, p.yt, which, ws, bytes, st); });
        return THPVariable_Wrap(p.y);
    });
}

ENTRY(linear_fused) {      // x, packed, gamma, N, fmt, y_dtype, y, segmented
    return entry(n, 8, [&] {
        bitnet_dtype dt;
        const at::Tensor& x = matrix(a[0], "x", &dt);
        const int64_t M = x.size(0), K = x.size(1), N = integer(a[3]);
        at::Tensor y = output(a[6], "y", {M, N}, out_type(a[5]), x);
        const bool seg = truth(a[7]);
        const float* gamma = seg ? per_block(a[2], "gamma_rb", N) : floats(a[2], "gamma");
        const void *xp = x.const_data_ptr(), *w = tensor(a[1], "packed").const_data_ptr();
        const bitnet_format f = (bitnet_format)(int)integer(a[4]);
        const bitnet_dtype yt = (bitnet_dtype)(int)integer(a[5]);
        void *yp = y.mutable_data_ptr(), *st = stream();
        call(seg ? "bitnet_linear_fused_segmented" : "bitnet_linear_fused",
             [&] { return (seg ? abi.linear_fused_segmented : abi.linear_fused)(xp, dt, w, gamma, M, N, K, f, yp, yt, st); });
        return THPVariable_Wrap(y);
    });
}

ENTRY(rmsnorm_linear_fused) {      // x, g, eps, packed, gamma, N, fmt, y_dtype, y, segmented
    return entry(n, 10, [&] {
        bitnet_dtype dt;
        const at::Tensor& x = matrix(a[0], "x", &dt);
        const int64_t M = x.size(0), K = x.size(1), N = integer(a[5]);
        at::Tensor y = output(a[8], "y", {M, N}, out_type(a[7]), x);
        const float* g = gain(a[1], K, true);
        const float eps = real(a[2]);
        const bool seg = truth(a[9]);
        const float* gamma = seg ? per_block(a[4], "gamma", N) : floats(a[4], "gamma");
        const void *xp = x.const_data_ptr(), *w = tensor(a[3], "packed").const_data_ptr();
        const bitnet_format f = (bitnet_format)(int)integer(a[6]);
        const bitnet_dtype yt = (bitnet_dtype)(int)integer(a[7]);
        void *yp = y.mutable_data_ptr(), *st = stream();
        call(seg ? "bitnet_rmsnorm_linear_fused_segmented" : "bitnet_rmsnorm_linear_fused", [&] {
            return (seg ? abi.rmsnorm_linear_fused_segmented : abi.rmsnorm_linear_fused)(xp, dt, g, eps, w, gamma, M, N, K, f, yp, yt, st);
        });
        return THPVariable_Wrap(y);
    });
}

ENTRY(swiglu_linear_fused) {      // gu, packed, gamma, N, fmt, y_dtype, y
    return entry(n, 7, [&] {
        bitnet_dtype dt;
        const at::Tensor& gu = matrix(a[0], "gu", &dt);
        const int64_t M = gu.size(0), N = integer(a[3]);
        if (gu.size(1) % 2) raise(PyExc_ValueError, "gu must hold a gate and an up half");
        const int64_t F = gu.size(1) / 2;
        at::Tensor y = output(a[6], "y", {M, N}, out_type(a[5]), gu);
        const float* gamma = floats(a[2], "gamma");
        const void *gp = gu.const_data_ptr(), *w = tensor(a[1], "packed").const_data_ptr();
        const bitnet_format f = (bitnet_format)(int)integer(a[4]);
        const bitnet_dtype yt = (bitnet_dtype)(int)integer(a[5]);
        void *yp = y.mutable_data_ptr(), *st = stream();
        call("bitnet_swiglu_linear_fused", [&] { return abi.swiglu_linear_fused(gp, dt, w, gamma, M, N, F, f, yp, yt, st); });
        return THPVariable_Wrap(y);
    });
}

ENTRY(ffn_gate_up_fused) {      // x, packed, gamma, F, norm, g, eps, gamma_per_block, fmt, h_dtype, h
    return entry(n, 11, [&] {
        bitnet_dtype dt;
        const at::Tensor& x = matrix(a[0], "x", &dt);
        const int64_t M = x.size(0), K = x.size(1), F = integer(a[3]);
        at::Tensor h = output(a[10], "h", {M, F}, out_type(a[9]), x);
        const int norm = truth(a[4]) ? 1 : 0, per = truth(a[7]) ? 1 : 0;
        const float* g = gain(a[5], K, false);
        const float eps = real(a[6]);
        const float* gamma = floats(a[2], "gamma");
        const void *xp = x.const_data_ptr(), *w = tensor(a[1], "packed").const_data_ptr();
        const bitnet_format f = (bitnet_format)(int)integer(a[8]);
        const bitnet_dtype ht = (bitnet_dtype)(int)integer(a[9]);
        void *hp = h.mutable_data_ptr(), *st = stream();
        call("bitnet_ffn_gate_up_fused", [&] { return abi.ffn_gate_up_fused(xp, dt, norm, g, eps, w, gamma, per, M, F, K, f, hp, ht, st); });
        return THPVariable_Wrap(h);
    });
}

// bind({name: address}, BitnetError)
PyObject* bind(PyObject*, PyObject* args) {
    PyObject *addresses, *cls;
    if (!PyArg_ParseTuple(args, "O!O", &PyDict_Type, &addresses, &cls)) return nullptr;
    Abi got;
#define TAKE(field_)                                                                                    \
    do {                                                                                                \
        PyObject* v = PyDict_GetItemString(addresses, "bitnet_" #field_);                               \
        void* p = v ? PyLong_AsVoidPtr(v) : nullptr;                                                    \
        if (!p) {                                                                                       \
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "no address for bitnet_" #field_); \
            return nullptr;                                                                             \
        }                                                                                               \
        got.field_ = reinterpret_cast<decltype(got.field_)>(p);                                         \
    } while (0)
    TAKE(quantize_acts); TAKE(rmsnorm_quantize); TAKE(swiglu_quantize); TAKE(linear); TAKE(linear_variant); TAKE(linear_segmented);
    TAKE(linear_ws); TAKE(linear_fused); TAKE(linear_fused_segmented); TAKE(rmsnorm_linear_fused);
    TAKE(rmsnorm_linear_fused_segmented); TAKE(swiglu_linear_fused); TAKE(ffn_gate_up_fused);
#undef TAKE
    abi = got;
    Py_INCREF(cls);
    Py_XDECREF(error_class);
    error_class = cls;
    Py_RETURN_NONE;
}

#define FAST(name_) {#name_, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name_)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"bind", bind, METH_VARARGS, nullptr},
    FAST(quantize_acts), FAST(rmsnorm_quantize), FAST(swiglu_quantize), FAST(linear), FAST(linear_segmented), FAST(linear_ws),
    FAST(linear_fused), FAST(rmsnorm_linear_fused), FAST(swiglu_linear_fused), FAST(ffn_gate_up_fused),
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__call() { return PyModule_Create(&module); }
