// Python side of the convenience functions in attn.py: check the tensors, allocate the outputs, find the
// stream, call the C ABI.  No arithmetic of the method.
//
// A small call is bound by what happens on the host: through ctypes and torch's Python functions a forward
// took 12.5 us (5 of them to find the current stream, 4 to marshal the arguments), longer than its kernel.
// Every function here takes the positional arguments its wrapper in attn.py passes, raises ValueError for
// tensors that do not fit, and returns either the outputs or the negative status of the C call.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/core/LegacyTypeDispatch.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <dlfcn.h>

#include <exception>
#include <initializer_list>

#include "../../include/tk_attn.h"

namespace {

struct Raised {};       // a Python exception is set

// The functions of the library that load_library() in attn.py opened, which need not be the one next to this module.
#define TK_FUNCTIONS(F) \
    F(tk_attn_fwd_scratch_bytes) F(tk_attn_fwd_rect_scratch) F(tk_attn_bwd_scratch_bytes) F(tk_attn_bwd_rect_scratch) \
    F(tk_attn_decode_workspace_bytes) F(tk_attn_decode) F(tk_rotary) F(tk_gemm)
struct Library {
#define TK_MEMBER(name) decltype(&::name) name = nullptr;
    TK_FUNCTIONS(TK_MEMBER)
#undef TK_MEMBER
    bool bound = false;
} lib;

[[noreturn]] void value_error(const char* format, const char* name) {
    PyErr_Format(PyExc_ValueError, format, name);
    throw Raised();
}

const at::Tensor& tensor(PyObject* o, const char* name) {
    if (!THPVariable_Check(o)) {
        PyErr_Format(PyExc_TypeError, "%s must be a tensor", name);
        throw Raised();
    }
    return THPVariable_Unpack(o);
}

const at::Tensor& typed(PyObject* o, const char* name, at::ScalarType type, const char* type_name) {
    const at::Tensor& t = tensor(o, name);
    if (!(t.is_cuda() && t.scalar_type() == type && t.is_contiguous())) {
        PyErr_Format(PyExc_ValueError, "%s must be a contiguous CUDA %s tensor", name, type_name);
        throw Raised();
    }
    return t;
}

void shape(const at::Tensor& t, const char* name, std::initializer_list<int64_t> want) {
    if (t.sizes() != at::IntArrayRef(want)) {
        PyObject* text = PyUnicode_FromString("");
        for (int64_t n : want) {
            PyObject* more = PyUnicode_FromFormat("%U%s%lld", text, PyUnicode_GetLength(text) ? ", " : "", (long long)n);
            Py_DECREF(text);
            text = more;
        }
        PyErr_Format(PyExc_ValueError, "%s has another shape than the expected (%U)", name, text);
        Py_DECREF(text);
        throw Raised();
    }
}

const at::Tensor& bf16(PyObject* o, const char* name) { return typed(o, name, at::kBFloat16, "bf16"); }

const at::Tensor& bf16(PyObject* o, const char* name, std::initializer_list<int64_t> want) {
    const at::Tensor& t = bf16(o, name);
    shape(t, name, want);
    return t;
}

const at::Tensor& f32(PyObject* o, const char* name, std::initializer_list<int64_t> want) {
    const at::Tensor& t = typed(o, name, at::kFloat, "fp32");
    shape(t, name, want);
    return t;
}

void rank(const at::Tensor& t, const char* name, int64_t want) {
    if (t.dim() != want) value_error("%s has the wrong number of dimensions", name);
}

// a size as the C ABI takes it
int narrow(int64_t n, const char* name) {
    if (n > 0x7fffffff) value_error("%s has a dimension beyond 31 bits", name);
    return (int)n;
}

// memory that the call may write from end to end
const at::Tensor& buffer(PyObject* o, const char* name) {
    const at::Tensor& t = tensor(o, name);
    if (!(t.is_cuda() && t.is_contiguous())) value_error("%s must be a contiguous CUDA tensor", name);
    return t;
}

// the tensors of out=
class Outputs {
public:
    Outputs(PyObject* out, Py_ssize_t n) : items_(PySequence_Fast(out, "out must be a sequence of tensors")) {
        if (!items_) throw Raised();
        if (PySequence_Fast_GET_SIZE(items_) != n) {
            Py_DECREF(items_);
            PyErr_Format(PyExc_ValueError, "out must hold %zd tensors", n);
            throw Raised();
        }
    }
    ~Outputs() { Py_DECREF(items_); }
    Outputs(const Outputs&) = delete;
    Outputs& operator=(const Outputs&) = delete;
    PyObject* operator[](Py_ssize_t i) const { return PySequence_Fast_GET_ITEM(items_, i); }

private:
    PyObject* items_;
};

bool truth(PyObject* o) {
    const int v = PyObject_IsTrue(o);
    if (v < 0) throw Raised();
    return v != 0;
}

float number(PyObject* o) {
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) throw Raised();
    return (float)v;
}

// the raw stream an int names, or the current stream of the current device
struct Stream {
    void* raw;
    bool given;
};
Stream stream_of(PyObject* o) {
    if (o == Py_None) return {(void*)c10::hip::getCurrentHIPStream().stream(), false};
    void* s = PyLong_AsVoidPtr(o);
    if (PyErr_Occurred()) throw Raised();
    return {s, true};
}

// The interpreter lock is released while this lives: an allocation may wait for the device and a launch for room in the
// stream's queue, possibly behind a host callback that needs the lock itself.  No Python object is touched meanwhile.
class Unlocked {
public:
    Unlocked() : state_(PyEval_SaveThread()) {}
    ~Unlocked() { PyEval_RestoreThread(state_); }
    Unlocked(const Unlocked&) = delete;
    Unlocked& operator=(const Unlocked&) = delete;

private:
    PyThreadState* state_;
};

// Makes `stream` the current one of `device` for a while.  Scratch that a call takes and gives back must come from the
// pool of the stream it runs on: only there is the memory's next use ordered behind this one, and this one behind its last.
class OnStream {
public:
    OnStream(void* stream, c10::DeviceIndex device) : before_(c10::hip::getCurrentHIPStream(device)), changed_(stream != (void*)before_.stream()) {
        if (changed_) c10::hip::setCurrentHIPStream(c10::hip::getStreamFromExternal((hipStream_t)stream, device));
    }
    ~OnStream() { if (changed_) c10::hip::setCurrentHIPStream(before_); }
    OnStream(const OnStream&) = delete;
    OnStream& operator=(const OnStream&) = delete;

private:
    c10::hip::HIPStream before_;
    bool changed_;
};

// The device is that of the stream: the current one, or with a stream of the caller's the one its tensors are on, which
// need not be the current.
at::Tensor scratch_on(Stream stream, size_t bytes, const at::Tensor& like) {
    at::AutoDispatchBelowADInplaceOrView plain;
    const c10::DeviceIndex device = stream.given ? like.device().index() : c10::hip::current_device();
    OnStream on(stream.raw, device);
    return at::empty({(int64_t)bytes}, like.options().dtype(at::kByte).device(at::kCUDA, device));
}

// Scratch that only makes a call faster: where there is no memory for it the call does without (n becomes 0).
at::Tensor optional_scratch(Stream stream, size_t& n, const at::Tensor& like) {
    if (n == 0) return {};
    try {
        return scratch_on(stream, n, like);
    } catch (const c10::OutOfMemoryError&) {
        n = 0;
        return {};
    }
}

PyObject* status(int rc) { return PyLong_FromLong(rc); }

PyObject* give(std::initializer_list<const at::Tensor*> outs) {
    PyObject* tuple = PyTuple_New((Py_ssize_t)outs.size());
    if (!tuple) throw Raised();
    Py_ssize_t i = 0;
    for (const at::Tensor* t : outs) {
        PyObject* o = THPVariable_Wrap(*t);
        if (!o) { Py_DECREF(tuple); throw Raised(); }
        PyTuple_SET_ITEM(tuple, i++, o);
    }
    return tuple;
}

struct Sizes {
    int B, Hq, Hkv, Nq, Nk, D;
};

// q [B,Hq,Nq,D], k and v [B,Hkv,Nk,D]; same_heads / same_length: the calls that do not take others
Sizes qkv(PyObject* const* a, bool same_heads, bool same_length) {
    const at::Tensor& q = bf16(a[0], "q");
    rank(q, "q", 4);
    const at::Tensor& k = bf16(a[1], "k");
    rank(k, "k", 4);
    const int64_t B = q.size(0), Hq = q.size(1), Nq = q.size(2), D = q.size(3);
    const int64_t Hkv = same_heads ? Hq : k.size(1), Nk = same_length ? Nq : k.size(2);
    shape(k, "k", {B, Hkv, Nk, D});
    bf16(a[2], "v", {B, Hkv, Nk, D});
    return {narrow(B, "q"), narrow(Hq, "q"), narrow(Hkv, "k"), narrow(Nq, "q"), narrow(Nk, "k"), narrow(D, "q")};
}

// fwd(q, k, v, causal, scale, stream, same_heads, same_length, out): out None, or (o, lse) to write to
PyObject* fwd(PyObject* const* a) {
    const Sizes s = qkv(a, truth(a[6]), truth(a[7]));
    const at::Tensor &q = THPVariable_Unpack(a[0]), &k = THPVariable_Unpack(a[1]), &v = THPVariable_Unpack(a[2]);
    const bool causal = truth(a[3]);
    const float scale = number(a[4]);
    const Stream stream = stream_of(a[5]);
    at::Tensor o, lse;
    if (a[8] != Py_None) {
        const Outputs out(a[8], 2);
        o = bf16(out[0], "o", {s.B, s.Hq, s.Nq, s.D});
        lse = f32(out[1], "lse", {s.B, s.Hq, s.Nq});
    }
    int rc;
    {
        Unlocked unlocked;
        if (!o.defined()) {
            at::AutoDispatchBelowADInplaceOrView plain;
            o = at::empty(q.sizes(), q.options());
            lse = at::empty({s.B, s.Hq, s.Nq}, q.options().dtype(at::kFloat));
        }
        size_t n = s.Nq < s.Nk ? lib.tk_attn_fwd_scratch_bytes(s.B, s.Hq, s.Hkv, s.Nq, s.Nk, s.D, causal) : 0;
        const at::Tensor scratch = optional_scratch(stream, n, q);
        rc = lib.tk_attn_fwd_rect_scratch(q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(), (float*)lse.data_ptr(),
                                          s.B, s.Hq, s.Hkv, s.Nq, s.Nk, s.D, causal, scale, n ? scratch.data_ptr() : nullptr, n, stream.raw);
    }
    return rc != TK_OK ? status(rc) : give({&o, &lse});
}

// bwd(q, k, v, o, d_o, lse, causal, scale, workspace, own_bytes, stream, same_heads, same_length, out): workspace None: the
// call takes own_bytes and gives them back; out None, or (dq, dk, dv) to write to
PyObject* bwd(PyObject* const* a) {
    const Sizes s = qkv(a, truth(a[11]), truth(a[12]));
    const at::Tensor &q = THPVariable_Unpack(a[0]), &k = THPVariable_Unpack(a[1]), &v = THPVariable_Unpack(a[2]);
    const at::Tensor& o = bf16(a[3], "o", {s.B, s.Hq, s.Nq, s.D});
    const at::Tensor& d_o = bf16(a[4], "d_o", {s.B, s.Hq, s.Nq, s.D});
    const at::Tensor& lse = f32(a[5], "lse", {s.B, s.Hq, s.Nq});
    const bool causal = truth(a[6]);
    const float scale = number(a[7]);
    at::Tensor workspace;
    if (a[8] != Py_None) workspace = buffer(a[8], "workspace");
    const size_t own_bytes = PyLong_AsSize_t(a[9]);
    if (PyErr_Occurred()) throw Raised();
    const Stream stream = stream_of(a[10]);
    at::Tensor dq, dk, dv;
    if (a[13] != Py_None) {
        const Outputs out(a[13], 3);
        dq = bf16(out[0], "dq", {s.B, s.Hq, s.Nq, s.D});
        dk = bf16(out[1], "dk", {s.B, s.Hkv, s.Nk, s.D});
        dv = bf16(out[2], "dv", {s.B, s.Hkv, s.Nk, s.D});
    }
    int rc;
    {
        Unlocked unlocked;
        if (!workspace.defined()) workspace = scratch_on(stream, own_bytes, q);
        if (!dq.defined()) {
            at::AutoDispatchBelowADInplaceOrView plain;
            dq = at::empty(q.sizes(), q.options());
            dk = at::empty(k.sizes(), k.options());
            dv = at::empty(k.sizes(), k.options());
        }
        const size_t workspace_bytes = (size_t)workspace.numel() * workspace.element_size();
        size_t n = s.Hq != s.Hkv || s.Nq != s.Nk ? lib.tk_attn_bwd_scratch_bytes(s.B, s.Hq, s.Hkv, s.Nq, s.Nk, s.D, causal, workspace_bytes) : 0;
        const at::Tensor scratch = optional_scratch(stream, n, q);
        rc = lib.tk_attn_bwd_rect_scratch(q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(), d_o.data_ptr(), (const float*)lse.data_ptr(),
                                          dq.data_ptr(), dk.data_ptr(), dv.data_ptr(), s.B, s.Hq, s.Hkv, s.Nq, s.Nk, s.D, causal, scale,
                                          workspace.data_ptr(), workspace_bytes, n ? scratch.data_ptr() : nullptr, n, stream.raw);
    }
    return rc != TK_OK ? status(rc) : give({&dq, &dk, &dv});
}

// decode(q, k, v, scale, workspace or None, stream)
PyObject* decode(PyObject* const* a) {
    const at::Tensor& q = bf16(a[0], "q");
    rank(q, "q", 4);
    if (q.size(2) != 1) value_error("%s takes exactly one query per head", "decode");
    const Sizes s = qkv(a, false, false);
    const at::Tensor &k = THPVariable_Unpack(a[1]), &v = THPVariable_Unpack(a[2]);
    const float scale = number(a[3]);
    at::Tensor workspace;
    if (a[4] != Py_None) workspace = buffer(a[4], "workspace");
    const Stream stream = stream_of(a[5]);
    at::Tensor o, lse;
    int rc;
    {
        Unlocked unlocked;
        at::AutoDispatchBelowADInplaceOrView plain;
        if (!workspace.defined()) {
            const size_t n = lib.tk_attn_decode_workspace_bytes(s.B, s.Hq, s.Hkv, s.Nk, s.D);
            workspace = scratch_on(stream, n < 16 ? 16 : n, q);
        }
        o = at::empty(q.sizes(), q.options());
        lse = at::empty({s.B, s.Hq, 1}, q.options().dtype(at::kFloat));
        rc = lib.tk_attn_decode(q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(), (float*)lse.data_ptr(),
                                s.B, s.Hq, s.Hkv, s.Nk, s.D, scale, workspace.data_ptr(),
                                (size_t)workspace.numel() * workspace.element_size(), stream.raw);
    }
    return rc != TK_OK ? status(rc) : give({&o, &lse});
}

// rotary(x, sin_table, cos_table, out or None, stream)
PyObject* rotary(PyObject* const* a) {
    const at::Tensor& x = bf16(a[0], "x");
    rank(x, "x", 4);
    const int64_t N = x.size(2), D = x.size(3);
    const at::Tensor& sn = bf16(a[1], "sin_table", {N, D / 2});
    const at::Tensor& cs = bf16(a[2], "cos_table", {N, D / 2});
    const int B = narrow(x.size(0), "x"), H = narrow(x.size(1), "x"), n = narrow(N, "x"), d = narrow(D, "x");
    at::Tensor o;
    if (a[3] != Py_None) o = bf16(a[3], "o", {B, H, N, D});
    const Stream stream = stream_of(a[4]);
    int rc;
    {
        Unlocked unlocked;
        if (!o.defined()) {
            at::AutoDispatchBelowADInplaceOrView plain;
            o = at::empty(x.sizes(), x.options());
        }
        rc = lib.tk_rotary(x.data_ptr(), sn.data_ptr(), cs.data_ptr(), o.data_ptr(), B, H, n, d, stream.raw);
    }
    return rc != TK_OK ? status(rc) : THPVariable_Wrap(o);
}

// gemm(a, b, out or None, stream)
PyObject* gemm(PyObject* const* args) {
    const at::Tensor &a = tensor(args[0], "a"), &b = tensor(args[1], "b");
    if (a.scalar_type() != at::kBFloat16 || b.scalar_type() != at::kBFloat16 || a.dim() != 2 || b.dim() != 2)
        value_error("%s must be 2-D bf16 tensors", "a, b");
    if (!(a.is_cuda() && b.is_cuda() && a.is_contiguous() && b.is_contiguous()) || a.size(1) != b.size(0))
        value_error("%s must be contiguous CUDA tensors", "a [M,K], b [K,N]");
    const int M = narrow(a.size(0), "a"), K = narrow(a.size(1), "a"), N = narrow(b.size(1), "b");
    at::Tensor c;
    if (args[2] != Py_None) c = bf16(args[2], "out", {M, N});
    const Stream stream = stream_of(args[3]);
    int rc;
    {
        Unlocked unlocked;
        if (!c.defined()) {
            at::AutoDispatchBelowADInplaceOrView plain;
            c = at::empty({M, N}, a.options());
        }
        rc = lib.tk_gemm(a.data_ptr(), b.data_ptr(), c.data_ptr(), M, N, K, stream.raw);
    }
    return rc != TK_OK ? status(rc) : THPVariable_Wrap(c);
}

template <PyObject* (*F)(PyObject* const*), int N>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t n) {
    if (n != N) {
        PyErr_Format(PyExc_TypeError, "%d arguments expected, %zd given", N, n);
        return nullptr;
    }
    if (!lib.bound) {
        PyErr_SetString(PyExc_RuntimeError, "no library is bound");
        return nullptr;
    }
    try {
        return F(args);
    } catch (const Raised&) {
    } catch (const c10::OutOfMemoryError& e) {
        PyObject* torch = PyImport_ImportModule("torch");
        PyObject* type = torch ? PyObject_GetAttrString(torch, "OutOfMemoryError") : nullptr;
        if (type) PyErr_SetString(type, e.what_without_backtrace());
        Py_XDECREF(type);
        Py_XDECREF(torch);
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
    }
    return nullptr;
}

// bind(handle): the dlopen handle of the library whose functions are called from now on
PyObject* bind(PyObject*, PyObject* handle) {
    void* const h = PyLong_AsVoidPtr(handle);
    if (PyErr_Occurred()) return nullptr;
    Library found;
#define TK_FIND(name) \
    if (!(found.name = (decltype(found.name))dlsym(h, #name))) { \
        PyErr_SetString(PyExc_AttributeError, "the library has no " #name); \
        return nullptr; \
    }
    TK_FUNCTIONS(TK_FIND)
#undef TK_FIND
    found.bound = true;
    lib = found;
    Py_RETURN_NONE;
}

#define TK_ENTRY(name, n) {#name, (PyCFunction)(void (*)(void))entry<name, n>, METH_FASTCALL, nullptr}
PyMethodDef kMethods[] = {
    {"bind", bind, METH_O, nullptr},
    TK_ENTRY(fwd, 9), TK_ENTRY(bwd, 14), TK_ENTRY(decode, 6), TK_ENTRY(rotary, 5), TK_ENTRY(gemm, 4),
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_binding", "tensor checks, output allocation and dispatch to the C ABI", -1, kMethods,
                       nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void) { return PyModule_Create(&kModule); }
