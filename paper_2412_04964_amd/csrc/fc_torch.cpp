// fc_torch.cpp -- the binding's ordinary calls in native code: a CPython extension between torch tensors and the C ABI.
//
// What a decode-sized call spends its time on is the host: the checks of binding.py ask each tensor for its type,
// shape, contiguity and device through the Python interpreter, and ctypes converts ten to fifteen arguments; that is
// 11 us of the 13 us a call takes where the kernel needs 2.  The functions here make the same checks on the tensors
// themselves, allocate missing outputs, take the current stream and call the library: 3 us a call (inputs
// changing from call to call: three steps of a decode rank 39.0 -> 10.7 us, of a 512-token chunk 38.6 -> 14.8 us, a decode
// all-reduce 11.2 -> 3.5 us, which is its kernel).
//
// They take the ordinary call only.  Anything else -- a tensor of another type, shape, layout, device or Python class,
// an integer that is not a Python int, a geometry the library does not have, an active tracing, dispatch or function
// mode or functional transform -- makes them return None before anything has been allocated or launched, and
// binding.py then goes through its own checks, which raise the error or make the call.  So there is one definition of
// what is accepted and of what is raised: binding.py.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <dlfcn.h>

#include <ATen/ATen.h>
#include <ATen/hip/EmptyTensor.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <array>

#include "fc.h"

namespace {

#define FC_ENTRIES(X)                                                                                                \
    X(fc_quantize) X(fc_quantize_sym) X(fc_quantize_fp8) X(fc_quantize_cmeta) X(fc_quantize_rot)                     \
    X(fc_dequant_reduce_requant) X(fc_dequant_reduce_requant_sym) X(fc_dequant_reduce_requant_fp8)                   \
    X(fc_dequant_reduce_requant_cmeta)                                                                               \
    X(fc_dequantize) X(fc_dequantize_sym) X(fc_dequantize_fp8) X(fc_dequantize_cmeta) X(fc_dequantize_rot)           \
    X(fc_allreduce_sim) X(fc_allreduce_sim_sym) X(fc_allreduce_sim_fp8) X(fc_allreduce_sim_cmeta)                    \
    X(fc_allreduce_sim_rot) X(fc_allreduce_sim_workspace_bytes)

struct Library {
#define FC_MEMBER(f) decltype(&::f) f = nullptr;
    FC_ENTRIES(FC_MEMBER)
#undef FC_MEMBER
};

Library lib;                       // filled once by load(), before any of the calls can be reached
PyObject *on_error = nullptr;      // binding._check(code, name): raises FcError

constexpr int kAsym = 0, kSym = 1, kFp8 = 2, kCmeta = 3;          // which of a family's entry points

// Nothing that intercepts tensor operations is active in this thread (dispatch modes, functional transforms and
// tracing add dispatch keys; function modes have a stack of their own).
bool plain_context()
{
    const auto included = c10::impl::tls_local_dispatch_key_set().included_;
    return (included.raw_repr() & ~c10::default_included_set.raw_repr()) == 0 &&
           at::impl::PythonTorchFunctionTLS::stack_len() == 0;
}

// The current device if `o` is a tensor on it, otherwise -1 (HIP is not asked before there is a GPU tensor)
int device_of(PyObject *o)
{
    if (!THPVariable_CheckExact(o)) return -1;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda()) return -1;
    const int device = t.device().index();
    return device == (int)c10::hip::current_device() ? device : -1;
}

// The tensor behind `o` if it is a dense, contiguous one of `dtype` on GPU `device` and of no Python subclass or
// functional wrapper; otherwise null.
const at::Tensor *plain(PyObject *o, at::ScalarType dtype, int device)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined()) return nullptr;
    static const uint64_t ordinary = c10::DispatchKeySet({c10::DispatchKey::CUDA, c10::DispatchKey::AutogradCUDA,
                                                          c10::DispatchKey::AutocastCUDA,
                                                          c10::DispatchKey::ADInplaceOrView}).raw_repr();
    if ((t.key_set().raw_repr() & ~ordinary) != 0) return nullptr;
    if (!t.is_cuda() || t.scalar_type() != dtype || t.device().index() != device || !t.is_contiguous()) return nullptr;
    return &t;
}

bool shape2(const at::Tensor &t, int64_t a, int64_t b) { return t.dim() == 2 && t.size(0) == a && t.size(1) == b; }
bool shape3(const at::Tensor &t, int64_t a, int64_t b, int64_t c)
{
    return t.dim() == 3 && t.size(0) == a && t.size(1) == b && t.size(2) == c;
}

bool integer(PyObject *o, int64_t &v)
{
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    v = PyLong_AsLongLongAndOverflow(o, &overflow);
    return overflow == 0 && v >= -0x7FFFFFFF && v <= 0x7FFFFFFF;
}

bool width(int64_t bits) { return bits == 4 || bits == 8; }
bool geometry(int64_t hidden, int64_t group)
{
    return group >= 32 && group <= 16384 && (group & (group - 1)) == 0 && hidden > 0 && hidden % group == 0;
}

// An uninitialized tensor.  What torch.empty does behind its dispatcher, which no mode, transform or tracing watches here (see
// plain_context): 0.27 us less of 0.9 a tensor (quantize with its three results allocated 5.95 -> 5.15 us, a launch alone takes 2.9).
// Where torch has been asked to fill new memory it is torch.empty itself.
at::Tensor empty(at::IntArrayRef shape, at::ScalarType dtype, const at::Tensor &like)
{
    if (at::globalContext().deterministicAlgorithms() && at::globalContext().deterministicFillUninitializedMemory())
        return at::empty(shape, at::TensorOptions().dtype(dtype).device(like.device()));
    return at::Tensor(at::detail::empty_cuda(shape, dtype, like.device(), std::nullopt));
}

PyObject *fallback() { Py_RETURN_NONE; }

// FC_OK -> true; otherwise binding._check raises
bool done(int rc, const char *name)
{
    if (rc == FC_OK) return true;
    PyObject *r = PyObject_CallFunction(on_error, "is", rc, name);
    Py_XDECREF(r);
    if (r) PyErr_SetString(PyExc_RuntimeError, name);
    return false;
}

void *stream_of(int device) { return c10::hip::getCurrentHIPStream((c10::DeviceIndex)device).stream(); }

// The coded form of a [tokens, hidden] tensor: codes and one or two metadata arrays
struct Coded {
    std::array<const at::Tensor *, 3> t{};
    std::array<at::Tensor, 3> own;
    PyObject *given = nullptr;             // the caller's buffers as a tuple of this call's own, see take()

    Coded() = default;
    Coded(const Coded &) = delete;
    Coded &operator=(const Coded &) = delete;
    ~Coded() { Py_XDECREF(given); }

    // Takes the caller's buffers (`out` is not None), or fails.  A list may be changed by another thread while the
    // library is called without the interpreter lock: checks, launch and result use one tuple taken from it here,
    // which also keeps the tensors alive until the call has been made.
    bool take(PyObject *out, int n, int64_t tokens, int64_t hidden, int64_t group, int64_t bits, at::ScalarType meta,
              int device, bool at_least)
    {
        if (PyTuple_CheckExact(out)) {
            Py_INCREF(out);
            given = out;
        } else if (PyList_CheckExact(out)) {
            given = PyList_AsTuple(out);
            if (!given) throw python_error();
        } else {
            return false;
        }
        const Py_ssize_t len = PyTuple_GET_SIZE(given);
        if (len != n && !(at_least && len > n)) return false;
        for (int i = 0; i < n; ++i) {
            t[i] = plain(PyTuple_GET_ITEM(given, i), i ? meta : at::kByte, device);
            if (!t[i] || !shape2(*t[i], tokens, i ? hidden / group : hidden * bits / 8)) return false;
        }
        return true;
    }
    void allocate(int n, int64_t tokens, int64_t hidden, int64_t group, int64_t bits, at::ScalarType meta,
                  const at::Tensor &like)
    {
        for (int i = 0; i < n; ++i) {
            own[i] = empty({tokens, i ? hidden / group : hidden * bits / 8}, i ? meta : at::kByte, like);
            t[i] = &own[i];
        }
    }
    void *ptr(int i) const { return t[i] ? t[i]->data_ptr() : nullptr; }
    // n tensors followed by `nones` Nones
    PyObject *result(int n, int nones) const
    {
        if (given && nones == 0) {
            Py_INCREF(given);
            return given;
        }
        PyObject *r = PyTuple_New(n + nones);
        if (!r) return nullptr;
        for (int i = 0; i < n + nones; ++i) {
            PyObject *o = Py_None;
            if (i >= n) {
                Py_INCREF(o);
            } else if (given) {
                o = PyTuple_GET_ITEM(given, i);
                Py_INCREF(o);
            } else {
                o = THPVariable_Wrap(own[i]);
                if (!o) {
                    Py_DECREF(r);
                    return nullptr;
                }
            }
            PyTuple_SET_ITEM(r, i, o);
        }
        return r;
    }
};

at::ScalarType meta_type(int kind) { return kind == kCmeta ? at::kInt : at::kFloat; }

// (x, group[, bits][, quantizer], out): `kind` >= 0 fixed, kRot: taken from the arguments
constexpr int kRot = -1;

template <int KIND>
PyObject *quantize(PyObject *, PyObject *const *a, Py_ssize_t n_args)
{
    HANDLE_TH_ERRORS
    constexpr int want = KIND == kFp8 ? 3 : KIND == kRot ? 5 : 4;
    if (n_args != want || !plain_context()) return fallback();
    const int device = device_of(a[0]);
    if (device < 0) return fallback();
    const at::Tensor *x = plain(a[0], at::kHalf, device);
    int64_t group, bits = 8, kind = KIND;
    if (!x || x->dim() != 2 || !integer(a[1], group) || (KIND != kFp8 && !integer(a[2], bits)) ||
        (KIND == kRot && !integer(a[3], kind)))
        return fallback();
    if (KIND == kRot && (kind < kAsym || kind > kFp8)) return fallback();
    const int64_t t = x->size(0), h = x->size(1);
    if (!width(bits) || !geometry(h, group)) return fallback();
    const int n = kind == kAsym ? 3 : 2;
    PyObject *out = a[want - 1];
    Coded c;
    if (out == Py_None)
        c.allocate(n, t, h, group, bits, meta_type((int)kind), *x);
    else if (!c.take(out, n, t, h, group, bits, meta_type((int)kind), device, KIND == kRot && n == 2))
        return fallback();
    const void *px = x->data_ptr();
    void *codes = c.ptr(0), *meta = c.ptr(1), *zeros = c.ptr(2), *stream = stream_of(device);
    const int g = (int)group, b = (int)bits;
    int rc;
    const char *name;
    Py_BEGIN_ALLOW_THREADS
    if constexpr (KIND == kAsym) {
        name = "fc_quantize";
        rc = lib.fc_quantize(px, t, h, g, b, codes, (float *)meta, (float *)zeros, stream);
    } else if constexpr (KIND == kSym) {
        name = "fc_quantize_sym";
        rc = lib.fc_quantize_sym(px, t, h, g, b, codes, (float *)meta, stream);
    } else if constexpr (KIND == kFp8) {
        name = "fc_quantize_fp8";
        rc = lib.fc_quantize_fp8(px, t, h, g, codes, (float *)meta, stream);
    } else if constexpr (KIND == kCmeta) {
        name = "fc_quantize_cmeta";
        rc = lib.fc_quantize_cmeta(px, t, h, g, b, codes, (uint32_t *)meta, stream);
    } else {
        name = "fc_quantize_rot";
        rc = lib.fc_quantize_rot(px, t, h, g, b, (int)kind, codes, (float *)meta, (float *)zeros, stream);
    }
    Py_END_ALLOW_THREADS
    if (!done(rc, name)) return nullptr;
    return c.result(n, KIND == kRot ? 3 - n : 0);
    END_HANDLE_TH_ERRORS
}

// (codes, meta[, zeros], hidden, group[, bits_in, bits_out], out)
template <int KIND>
PyObject *fused(PyObject *, PyObject *const *a, Py_ssize_t n_args)
{
    HANDLE_TH_ERRORS
    constexpr int n = KIND == kAsym ? 3 : 2;
    constexpr int want = n + (KIND == kFp8 ? 3 : 5);
    if (n_args != want || !plain_context()) return fallback();
    const int device = device_of(a[0]);
    if (device < 0) return fallback();
    int64_t hidden, group, bits_in = 8, bits_out = 8;
    if (!integer(a[n], hidden) || !integer(a[n + 1], group)) return fallback();
    if (KIND != kFp8 && (!integer(a[n + 2], bits_in) || !integer(a[n + 3], bits_out))) return fallback();
    if (!width(bits_in) || !width(bits_out) || !geometry(hidden, group)) return fallback();
    std::array<const at::Tensor *, 3> in{};
    for (int i = 0; i < n; ++i) {
        in[i] = plain(a[i], i ? meta_type(KIND) : at::kByte, device);
        if (!in[i] || in[i]->dim() != 3) return fallback();
    }
    const int64_t n_src = in[0]->size(0), t = in[0]->size(1);
    if (n_src < 1 || n_src > FC_MAX_SRC || !shape3(*in[0], n_src, t, hidden * bits_in / 8)) return fallback();
    for (int i = 1; i < n; ++i)
        if (!shape3(*in[i], n_src, t, hidden / group)) return fallback();
    Coded c;
    if (a[want - 1] == Py_None)
        c.allocate(n, t, hidden, group, bits_out, meta_type(KIND), *in[0]);
    else if (!c.take(a[want - 1], n, t, hidden, group, bits_out, meta_type(KIND), device, false))
        return fallback();
    const int64_t cs = n_src > 1 ? in[0]->stride(0) : 0, ms = n_src > 1 ? in[1]->stride(0) : 0;
    const void *ci = in[0]->data_ptr(), *mi = in[1]->data_ptr(), *zi = n == 3 ? in[2]->data_ptr() : nullptr;
    void *co = c.ptr(0), *mo = c.ptr(1), *zo = c.ptr(2), *stream = stream_of(device);
    const int ns = (int)n_src, g = (int)group, bi = (int)bits_in, bo = (int)bits_out;
    int rc;
    const char *name;
    Py_BEGIN_ALLOW_THREADS
    if constexpr (KIND == kAsym) {
        name = "fc_dequant_reduce_requant";
        rc = lib.fc_dequant_reduce_requant(ci, cs, (const float *)mi, (const float *)zi, ms, ns, t, hidden, g, bi, bo,
                                           co, (float *)mo, (float *)zo, stream);
    } else if constexpr (KIND == kSym) {
        name = "fc_dequant_reduce_requant_sym";
        rc = lib.fc_dequant_reduce_requant_sym(ci, cs, (const float *)mi, ms, ns, t, hidden, g, bi, bo, co, (float *)mo,
                                               stream);
    } else if constexpr (KIND == kFp8) {
        name = "fc_dequant_reduce_requant_fp8";
        rc = lib.fc_dequant_reduce_requant_fp8(ci, cs, (const float *)mi, ms, ns, t, hidden, g, co, (float *)mo, stream);
    } else {
        name = "fc_dequant_reduce_requant_cmeta";
        rc = lib.fc_dequant_reduce_requant_cmeta(ci, cs, (const uint32_t *)mi, ms, ns, t, hidden, g, bi, bo, co,
                                                 (uint32_t *)mo, stream);
    }
    Py_END_ALLOW_THREADS
    if (!done(rc, name)) return nullptr;
    return c.result(n, 0);
    END_HANDLE_TH_ERRORS
}

// the float16 [t, h] result: the caller's tensor, or a new one
const at::Tensor *result_tensor(PyObject *out, int64_t t, int64_t h, const at::Tensor &like, int device, at::Tensor &own)
{
    if (out == Py_None) {
        own = empty({t, h}, at::kHalf, like);
        return &own;
    }
    const at::Tensor *y = plain(out, at::kHalf, device);
    return y && shape2(*y, t, h) ? y : nullptr;
}

PyObject *wrapped(PyObject *out, const at::Tensor &own)
{
    if (out == Py_None) return THPVariable_Wrap(own);
    Py_INCREF(out);
    return out;
}

// (codes, meta[, zeros], hidden, group[, bits][, quantizer], out)
template <int KIND>
PyObject *dequantize(PyObject *, PyObject *const *a, Py_ssize_t n_args)
{
    HANDLE_TH_ERRORS
    constexpr int arrays = KIND == kAsym || KIND == kRot ? 3 : 2;
    constexpr int want = arrays + 3 + (KIND == kFp8 ? 0 : 1) + (KIND == kRot ? 1 : 0);
    if (n_args != want || !plain_context()) return fallback();
    const int device = device_of(a[0]);
    if (device < 0) return fallback();
    int64_t hidden, group, bits = 8, kind = KIND;
    if (!integer(a[arrays], hidden) || !integer(a[arrays + 1], group)) return fallback();
    if (KIND != kFp8 && !integer(a[arrays + 2], bits)) return fallback();
    if (KIND == kRot && (!integer(a[arrays + 3], kind) || kind < kAsym || kind > kFp8)) return fallback();
    if (!width(bits) || !geometry(hidden, group)) return fallback();
    const int n = kind == kAsym ? 3 : 2;
    std::array<const at::Tensor *, 3> in{};
    for (int i = 0; i < n; ++i) {
        in[i] = plain(a[i], i ? meta_type((int)kind) : at::kByte, device);
        if (!in[i] || in[i]->dim() != 2) return fallback();
    }
    const int64_t t = in[0]->size(0);
    if (in[0]->size(1) != hidden * bits / 8) return fallback();
    for (int i = 1; i < n; ++i)
        if (!shape2(*in[i], t, hidden / group)) return fallback();
    at::Tensor own;
    PyObject *out = a[want - 1];
    const at::Tensor *y = result_tensor(out, t, hidden, *in[0], device, own);
    if (!y) return fallback();
    const void *codes = in[0]->data_ptr(), *meta = in[1]->data_ptr(), *zeros = n == 3 ? in[2]->data_ptr() : nullptr;
    void *py = y->data_ptr(), *stream = stream_of(device);
    const int g = (int)group, b = (int)bits;
    int rc;
    const char *name;
    Py_BEGIN_ALLOW_THREADS
    if constexpr (KIND == kAsym) {
        name = "fc_dequantize";
        rc = lib.fc_dequantize(codes, (const float *)meta, (const float *)zeros, t, hidden, g, b, py, stream);
    } else if constexpr (KIND == kSym) {
        name = "fc_dequantize_sym";
        rc = lib.fc_dequantize_sym(codes, (const float *)meta, t, hidden, g, b, py, stream);
    } else if constexpr (KIND == kFp8) {
        name = "fc_dequantize_fp8";
        rc = lib.fc_dequantize_fp8(codes, (const float *)meta, t, hidden, g, py, stream);
    } else if constexpr (KIND == kCmeta) {
        name = "fc_dequantize_cmeta";
        rc = lib.fc_dequantize_cmeta(codes, (const uint32_t *)meta, t, hidden, g, b, py, stream);
    } else {
        name = "fc_dequantize_rot";
        rc = lib.fc_dequantize_rot(codes, (const float *)meta, (const float *)zeros, t, hidden, g, b, (int)kind, py, stream);
    }
    Py_END_ALLOW_THREADS
    if (!done(rc, name)) return nullptr;
    return wrapped(out, own);
    END_HANDLE_TH_ERRORS
}

// (x, group[, bits_rs, bits_ag][, quantizer], out, workspace)
template <int KIND>
PyObject *allreduce(PyObject *, PyObject *const *a, Py_ssize_t n_args)
{
    HANDLE_TH_ERRORS
    constexpr int want = KIND == kFp8 ? 4 : KIND == kRot ? 7 : 6;
    if (n_args != want || !plain_context()) return fallback();
    const int device = device_of(a[0]);
    if (device < 0) return fallback();
    const at::Tensor *x = plain(a[0], at::kHalf, device);
    int64_t group, rs = 8, ag = 8, kind = KIND;
    if (!x || x->dim() != 3 || !integer(a[1], group)) return fallback();
    if (KIND != kFp8 && (!integer(a[2], rs) || !integer(a[3], ag))) return fallback();
    if (KIND == kRot && !integer(a[4], kind)) return fallback();
    const int64_t n = x->size(0), t = x->size(1), h = x->size(2);
    if (n < 1 || n > FC_MAX_SRC || !width(rs) || !width(ag) || !geometry(h, group)) return fallback();
    const int64_t need = (int64_t)lib.fc_allreduce_sim_workspace_bytes((int)n, t, h, (int)group, (int)rs, (int)ag);
    PyObject *out = a[want - 2], *space = a[want - 1];
    const at::Tensor *ws = nullptr;
    if (space != Py_None) {
        ws = plain(space, at::kByte, device);
        if (!ws || ws->numel() < need) return fallback();
    }
    at::Tensor own, own_ws;
    const at::Tensor *y = result_tensor(out, t, h, *x, device, own);
    if (!y) return fallback();
    const void *px = x->data_ptr();
    void *py = y->data_ptr(), *stream = stream_of(device);
    // Only the rotated call writes to its workspace.  The others want the address and size of one and leave it alone (fc.h): where
    // the caller gives none, they get the result's address, and nothing is allocated (2 x 16 x 4096, result allocated: 4.5 -> 3.9 us, both
    // builds in one process).
    void *pw = py;
    size_t bytes = (size_t)need;
    if (KIND == kRot && !ws) {
        own_ws = empty({need > 16 ? need : 16}, at::kByte, *x);
        ws = &own_ws;
    }
    if (ws) {
        pw = ws->data_ptr();
        bytes = (size_t)ws->numel();
    }
    const int ns = (int)n, g = (int)group, b1 = (int)rs, b2 = (int)ag;
    int rc;
    const char *name;
    Py_BEGIN_ALLOW_THREADS
    if constexpr (KIND == kAsym) {
        name = "fc_allreduce_sim";
        rc = lib.fc_allreduce_sim(px, ns, t, h, g, b1, b2, py, pw, bytes, stream);
    } else if constexpr (KIND == kSym) {
        name = "fc_allreduce_sim_sym";
        rc = lib.fc_allreduce_sim_sym(px, ns, t, h, g, b1, b2, py, pw, bytes, stream);
    } else if constexpr (KIND == kFp8) {
        name = "fc_allreduce_sim_fp8";
        rc = lib.fc_allreduce_sim_fp8(px, ns, t, h, g, py, pw, bytes, stream);
    } else if constexpr (KIND == kCmeta) {
        name = "fc_allreduce_sim_cmeta";
        rc = lib.fc_allreduce_sim_cmeta(px, ns, t, h, g, b1, b2, py, pw, bytes, stream);
    } else {
        name = "fc_allreduce_sim_rot";
        rc = lib.fc_allreduce_sim_rot(px, ns, t, h, g, b1, b2, (int)kind, py, pw, bytes, stream);
    }
    Py_END_ALLOW_THREADS
    if (!done(rc, name)) return nullptr;
    return wrapped(out, own);
    END_HANDLE_TH_ERRORS
}

// load(path, on_error): the functions of the library that the process already holds under `path`
PyObject *load(PyObject *, PyObject *args)
{
    const char *path;
    PyObject *raise;
    if (!PyArg_ParseTuple(args, "sO", &path, &raise)) return nullptr;
    void *handle = dlopen(path, RTLD_NOW);
    if (!handle) {
        PyErr_SetString(PyExc_ImportError, dlerror());
        return nullptr;
    }
    Library l;
#define FC_RESOLVE(f)                                                                                                \
    l.f = reinterpret_cast<decltype(&::f)>(dlsym(handle, #f));                                                       \
    if (!l.f) {                                                                                                      \
        PyErr_SetString(PyExc_ImportError, #f " not found in the library");                                          \
        return nullptr;                                                                                              \
    }
    FC_ENTRIES(FC_RESOLVE)
#undef FC_RESOLVE
    if (!lib.fc_quantize) lib = l;         // other threads may be in a call
    Py_INCREF(raise);
    Py_XSETREF(on_error, raise);
    Py_RETURN_NONE;
}

#define FC_METHOD(name, fn) {name, (PyCFunction)(void (*)(void))(fn), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"load", load, METH_VARARGS, nullptr},
    FC_METHOD("quantize", quantize<kAsym>), FC_METHOD("quantize_sym", quantize<kSym>),
    FC_METHOD("quantize_fp8", quantize<kFp8>), FC_METHOD("quantize_cmeta", quantize<kCmeta>),
    FC_METHOD("quantize_rot", quantize<kRot>),
    FC_METHOD("dequant_reduce_requant", fused<kAsym>), FC_METHOD("dequant_reduce_requant_sym", fused<kSym>),
    FC_METHOD("dequant_reduce_requant_fp8", fused<kFp8>), FC_METHOD("dequant_reduce_requant_cmeta", fused<kCmeta>),
    FC_METHOD("dequantize", dequantize<kAsym>), FC_METHOD("dequantize_sym", dequantize<kSym>),
    FC_METHOD("dequantize_fp8", dequantize<kFp8>), FC_METHOD("dequantize_cmeta", dequantize<kCmeta>),
    FC_METHOD("dequantize_rot", dequantize<kRot>),
    FC_METHOD("allreduce_sim", allreduce<kAsym>), FC_METHOD("allreduce_sim_sym", allreduce<kSym>),
    FC_METHOD("allreduce_sim_fp8", allreduce<kFp8>), FC_METHOD("allreduce_sim_cmeta", allreduce<kCmeta>),
    FC_METHOD("allreduce_sim_rot", allreduce<kRot>),
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fc_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fc_torch(void)
{
    PyObject *m = PyModule_Create(&module);
    // the torch whose headers this was compiled with: binding.py does not use the module under another one
    if (m && PyModule_AddStringConstant(m, "torch_version", FC_TORCH_VERSION) != 0) Py_CLEAR(m);
    return m;
}
