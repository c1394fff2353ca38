// The Python side of a call, in native code: argument checks on torch tensors, the output or workspace
// tensor where the caller gives none, the current stream, and the C ABI of include/robe.h.
//
// A call through ctypes spent 8 to 10 us of host time on this (about thirty attribute reads, two
// temporary objects for the stream, an argument conversion each), which is longer than the kernels of a
// small batch run, so a program of small calls was bound by it.  Here one METH_FASTCALL function reads
// the tensors' fields directly.  Messages and exception types are those of the Python functions in
// __init__.py, which hand their arguments over as they are.
//
// Nothing of the library is linked: bind() resolves the entry points of the librobe.so it is given.
#include <Python.h>
#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <dlfcn.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/robe.h"

namespace {

PyObject *g_error = nullptr;      // RobeError

struct Entry {
    decltype(&robe_forward) forward;
    decltype(&robe_forward_bf16) forward_bf16;
    decltype(&robe_backward) backward;
    decltype(&robe_backward_noalloc) backward_noalloc;
    decltype(&robe_workspace_bytes) workspace_bytes;
    decltype(&robe_adagrad_update) adagrad_update;
    decltype(&robe_sgd_update) sgd_update;
    decltype(&robe_fused_workspace_bytes) fused_workspace_bytes;
    decltype(&robe_backward_adagrad) backward_adagrad;
    decltype(&robe_backward_sgd) backward_sgd;
    decltype(&robe_forward_mixed) forward_mixed;
    decltype(&robe_mixed_workspace_bytes) mixed_workspace_bytes;
    decltype(&robe_backward_mixed) backward_mixed;
    decltype(&robe_fused_mixed_workspace_bytes) fused_mixed_workspace_bytes;
    decltype(&robe_backward_adagrad_mixed) backward_adagrad_mixed;
    decltype(&robe_last_error) last_error;
} lib = {};

// Thrown once a Python exception is set.
struct Raised {};

[[noreturn]] void raise(PyObject *type, const char *msg)
{
    PyErr_SetString(type, msg);
    throw Raised();
}

// Status of an entry point: a negative one becomes RobeError(code, text).
void check(int rc)
{
    if (rc == ROBE_OK) return;
    PyObject *args = Py_BuildValue("(is)", rc, lib.last_error());
    if (args != nullptr) {
        PyErr_SetObject(g_error, args);
        Py_DECREF(args);
    }
    throw Raised();
}

// Structures come as ctypes instances; a view of their memory lives as long as the call.
template <typename T>
struct View {
    Py_buffer buf;
    const T *ptr = nullptr;
    View(PyObject *o, const char *name)
    {
        if (o == Py_None) return;
        if (PyObject_GetBuffer(o, &buf, PyBUF_SIMPLE) != 0) throw Raised();
        if (buf.len != (Py_ssize_t)sizeof(T)) {
            PyBuffer_Release(&buf);
            PyErr_Format(PyExc_TypeError, "%s: not the structure of robe.h", name);
            throw Raised();
        }
        ptr = static_cast<const T *>(buf.buf);
    }
    ~View() { if (ptr != nullptr) PyBuffer_Release(&buf); }
    View(const View &) = delete;
};

int64_t integer(PyObject *o)
{
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw Raised();
    return v;
}

float real(PyObject *o)
{
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) throw Raised();
    return (float)v;
}

const at::Tensor &tensor(PyObject *o, const char *name)
{
    if (!THPVariable_Check(o)) {
        PyErr_Format(PyExc_TypeError, "%s: need a tensor", name);
        throw Raised();
    }
    return THPVariable_Unpack(o);
}

template <typename T>
T *device(const at::Tensor &t, at::ScalarType type, const char *type_name, const char *name)
{
    if (!t.is_cuda() || t.scalar_type() != type || !t.is_contiguous()) {
        PyErr_Format(PyExc_TypeError, "%s: need a contiguous %s tensor on the GPU", name, type_name);
        throw Raised();
    }
    return static_cast<T *>(t.data_ptr());
}
float *floats(const at::Tensor &t, const char *name) { return device<float>(t, at::kFloat, "torch.float32", name); }
int64_t *longs(const at::Tensor &t, const char *name) { return device<int64_t>(t, at::kLong, "torch.int64", name); }

hipStream_t stream() { return c10::hip::getCurrentHIPStream().stream(); }

// What forward and backward have in common: ids, optional bag bounds, sample and table counts.
struct Tokens {
    const at::Tensor &indices;
    const at::Tensor *offsets;
    int64_t batch, n_features, n_indices;
    Tokens(PyObject *ids, PyObject *off, int64_t b, int64_t f)
        : indices(tensor(ids, "indices")), offsets(off == Py_None ? nullptr : &tensor(off, "offsets")), batch(b), n_features(f),
          n_indices(indices.numel())
    {
        if (offsets != nullptr && offsets->numel() != batch * n_features + 1)
            raise(PyExc_ValueError, "offsets must hold batch*n_features + 1 entries");
    }
    const int64_t *ids() const { return longs(indices, "indices"); }
    const int64_t *bounds() const { return offsets == nullptr ? nullptr : longs(*offsets, "offsets"); }
};

// The caller's workspace, or one of the size the library asks for.
struct Workspace {
    at::Tensor held;
    void *ptr = nullptr;
    size_t bytes = 0;
    template <typename Query>
    Workspace(PyObject *given, const at::Tensor &like, Query need)
    {
        if (given != Py_None) {
            held = tensor(given, "workspace");
        } else {
            size_t n = 0;
            check(need(&n));
            if (n == 0) return;
            held = at::empty({(int64_t)n}, at::TensorOptions().dtype(at::kByte).device(like.device()));
        }
        ptr = held.data_ptr();
        bytes = (size_t)held.numel() * held.element_size();
    }
};

struct Dims {
    std::vector<uint32_t> d;
    int64_t sum = 0;
    explicit Dims(PyObject *o)
    {
        PyObject *seq = PySequence_Fast(o, "dims: need a sequence of integers");
        if (seq == nullptr) throw Raised();
        const Py_ssize_t n = PySequence_Fast_GET_SIZE(seq);
        d.resize((size_t)n);
        for (Py_ssize_t k = 0; k < n; ++k) {
            PyObject *v = PyNumber_Long(PySequence_Fast_GET_ITEM(seq, k));
            const long long x = v == nullptr ? -1 : PyLong_AsLongLong(v);
            Py_XDECREF(v);
            if (PyErr_Occurred()) {
                Py_DECREF(seq);
                throw Raised();
            }
            d[(size_t)k] = (uint32_t)x;
            sum += x;
        }
        Py_DECREF(seq);
    }
};

void same_length(const at::Tensor &t, const robe_hash_t *h, const char *text)
{
    if ((uint64_t)t.numel() != h->m) raise(PyExc_ValueError, text);
}

const robe_hash_t *need(const View<robe_hash_t> &h)
{
    if (h.ptr == nullptr) raise(PyExc_TypeError, "hash: need a RobeHash");
    return h.ptr;
}

// Runs f, which returns a new reference; every C++ exception becomes a Python one.
template <typename F>
PyObject *guarded(Py_ssize_t n, Py_ssize_t want, F f)
{
    HANDLE_TH_ERRORS
    if (n != want) {
        PyErr_Format(PyExc_TypeError, "%zd arguments, %zd wanted", n, want);
        return nullptr;
    }
    if (lib.forward == nullptr) {
        PyErr_SetString(PyExc_RuntimeError, "bind() first");
        return nullptr;
    }
    try {
        return f();
    } catch (const Raised &) {
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}

template <typename F>
int released(F f)
{
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f();
    Py_END_ALLOW_THREADS
    return rc;
}

// The output tensor: the caller's, or a new one of these sizes.
PyObject *output(PyObject *given, const at::Tensor &array, at::IntArrayRef sizes, int64_t numel, at::Tensor *t)
{
    if (given == Py_None) {
        *t = at::empty(sizes, at::TensorOptions().dtype(at::kFloat).device(array.device()));
        return THPVariable_Wrap(*t);
    }
    *t = tensor(given, "out");
    if (t->numel() != numel) raise(PyExc_ValueError, "out has the wrong size");
    Py_INCREF(given);
    return given;
}

struct Ref {      // an owned reference, dropped if the call fails
    PyObject *o;
    explicit Ref(PyObject *p) : o(p) { if (p == nullptr) throw Raised(); }
    ~Ref() { Py_XDECREF(o); }
    PyObject *take() { PyObject *p = o; o = nullptr; return p; }
};

// forward(hash, array, indices, offsets, batch, n_features, out, options, bf16)
PyObject *call_forward(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 9, [&]() -> PyObject * {
        View<robe_hash_t> hv(a[0], "hash");
        const robe_hash_t *h = need(hv);
        const at::Tensor &array = tensor(a[1], "array");
        same_length(array, h, "array length differs from hash.m");
        const Tokens k(a[2], a[3], integer(a[4]), integer(a[5]));
        View<robe_options_t> opt(a[7], "options");
        at::Tensor out;
        Ref result(output(a[6], array, {k.batch, k.n_features, (int64_t)h->d}, k.batch * k.n_features * (int64_t)h->d, &out));
        const bool bf16 = a[8] == Py_True;
        const void *src = bf16 ? static_cast<const void *>(device<uint16_t>(array, at::kShort, "torch.int16", "array"))
                               : static_cast<const void *>(floats(array, "array"));
        const int64_t *ids = k.ids(), *bounds = k.bounds();
        float *dst = floats(out, "out");
        void *s = stream();
        check(released([&] {
            return bf16 ? lib.forward_bf16(h, static_cast<const uint16_t *>(src), ids, bounds, k.n_indices, k.batch, (int32_t)k.n_features, dst, opt.ptr, s)
                        : lib.forward(h, static_cast<const float *>(src), ids, bounds, k.n_indices, k.batch, (int32_t)k.n_features, dst, opt.ptr, s);
        }));
        return result.take();
    });
}

// backward(hash, grad_out, indices, offsets, batch, n_features, grad_array, workspace, options, noalloc) -> grad_array
PyObject *call_backward(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 10, [&]() -> PyObject * {
        View<robe_hash_t> hv(a[0], "hash");
        const robe_hash_t *h = need(hv);
        const at::Tensor &grad = tensor(a[6], "grad_array"), &grad_out = tensor(a[1], "grad_out");
        same_length(grad, h, "grad_array length differs from hash.m");
        const int64_t batch = integer(a[4]), F = integer(a[5]);
        if (grad_out.numel() != batch * F * (int64_t)h->d) raise(PyExc_ValueError, "grad_out has the wrong size");
        const Tokens k(a[2], a[3], batch, F);
        View<robe_options_t> opt(a[8], "options");
        const bool noalloc = a[9] == Py_True;
        const Workspace ws(a[7], grad, [&](size_t *bytes) {
            return noalloc ? ROBE_OK : lib.workspace_bytes(h, k.batch, (int32_t)k.n_features, k.n_indices, opt.ptr, bytes);
        });
        const float *src = floats(grad_out, "grad_out");
        const int64_t *ids = k.ids(), *bounds = k.bounds();
        float *dst = floats(grad, "grad_array");
        void *s = stream();
        check(released([&] {
            return noalloc ? lib.backward_noalloc(h, src, ids, bounds, k.n_indices, k.batch, (int32_t)k.n_features, dst, opt.ptr, s)
                           : lib.backward(h, src, ids, bounds, k.n_indices, k.batch, (int32_t)k.n_features, dst, ws.ptr, ws.bytes, opt.ptr, s);
        }));
        Py_INCREF(a[6]);
        return a[6];
    });
}

// update(hash, array, state or None (SGD), grad_array, lr, eps)
PyObject *call_update(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 6, [&]() -> PyObject * {
        View<robe_hash_t> hv(a[0], "hash");
        const robe_hash_t *h = need(hv);
        const bool sgd = a[2] == Py_None;
        const at::Tensor &array = tensor(a[1], "array"), &grad = tensor(a[3], "grad_array");
        same_length(array, h, "array length differs from hash.m");
        if (!sgd) same_length(tensor(a[2], "state"), h, "state length differs from hash.m");
        same_length(grad, h, "grad_array length differs from hash.m");
        float *w = floats(array, "array"), *st = sgd ? nullptr : floats(tensor(a[2], "state"), "state"), *g = floats(grad, "grad_array");
        const float lr = real(a[4]), eps = sgd ? 0.0f : real(a[5]);
        void *s = stream();
        check(released([&] { return sgd ? lib.sgd_update(h, w, g, lr, s) : lib.adagrad_update(h, w, st, g, lr, eps, s); }));
        Py_RETURN_NONE;
    });
}

// fused(hash, grad_out, indices, offsets, batch, n_features, array, state or None (SGD), lr, eps, workspace, options)
PyObject *call_fused(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 12, [&]() -> PyObject * {
        View<robe_hash_t> hv(a[0], "hash");
        const robe_hash_t *h = need(hv);
        const bool sgd = a[7] == Py_None;
        const at::Tensor &array = tensor(a[6], "array"), &grad_out = tensor(a[1], "grad_out");
        same_length(array, h, "array length differs from hash.m");
        if (!sgd) same_length(tensor(a[7], "state"), h, "state length differs from hash.m");
        const int64_t batch = integer(a[4]), F = integer(a[5]);
        if (grad_out.numel() != batch * F * (int64_t)h->d) raise(PyExc_ValueError, "grad_out has the wrong size");
        const Tokens k(a[2], a[3], batch, F);
        View<robe_options_t> opt(a[11], "options");
        const Workspace ws(a[10], array, [&](size_t *bytes) {
            return lib.fused_workspace_bytes(h, k.batch, (int32_t)k.n_features, k.n_indices, opt.ptr, bytes);
        });
        const float *src = floats(grad_out, "grad_out");
        const int64_t *ids = k.ids(), *bounds = k.bounds();
        float *w = floats(array, "array"), *st = sgd ? nullptr : floats(tensor(a[7], "state"), "state");
        const float lr = real(a[8]), eps = sgd ? 0.0f : real(a[9]);
        void *s = stream();
        check(released([&] {
            return sgd ? lib.backward_sgd(h, src, ids, bounds, k.n_indices, k.batch, (int32_t)k.n_features, w, lr, ws.ptr, ws.bytes, opt.ptr, s)
                       : lib.backward_adagrad(h, src, ids, bounds, k.n_indices, k.batch, (int32_t)k.n_features, w, st, lr, eps, ws.ptr, ws.bytes, opt.ptr, s);
        }));
        Py_RETURN_NONE;
    });
}

// forward_mixed(hash, dims, array, indices, offsets, batch, out, options)
PyObject *call_forward_mixed(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 8, [&]() -> PyObject * {
        View<robe_hash_t> hv(a[0], "hash");
        const robe_hash_t *h = need(hv);
        const Dims dims(a[1]);
        const at::Tensor &array = tensor(a[2], "array");
        same_length(array, h, "array length differs from hash.m");
        const Tokens k(a[3], a[4], integer(a[5]), (int64_t)dims.d.size());
        View<robe_options_t> opt(a[7], "options");
        at::Tensor out;
        Ref result(output(a[6], array, {k.batch, dims.sum}, k.batch * dims.sum, &out));
        const float *src = floats(array, "array");
        const int64_t *ids = k.ids(), *bounds = k.bounds();
        float *dst = floats(out, "out");
        void *s = stream();
        check(released([&] {
            return lib.forward_mixed(h, dims.d.data(), src, ids, bounds, k.n_indices, k.batch, (int32_t)k.n_features, dst, opt.ptr, s);
        }));
        return result.take();
    });
}

// backward_mixed(hash, dims, grad_out, indices, offsets, batch, grad_array, workspace, options)
PyObject *call_backward_mixed(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 9, [&]() -> PyObject * {
        View<robe_hash_t> hv(a[0], "hash");
        const robe_hash_t *h = need(hv);
        const Dims dims(a[1]);
        const at::Tensor &grad = tensor(a[6], "grad_array"), &grad_out = tensor(a[2], "grad_out");
        same_length(grad, h, "grad_array length differs from hash.m");
        const int64_t batch = integer(a[5]);
        if (grad_out.numel() != batch * dims.sum) raise(PyExc_ValueError, "grad_out has the wrong size");
        const Tokens k(a[3], a[4], batch, (int64_t)dims.d.size());
        View<robe_options_t> opt(a[8], "options");
        const Workspace ws(a[7], grad, [&](size_t *bytes) {
            return lib.mixed_workspace_bytes(h, dims.d.data(), k.batch, (int32_t)k.n_features, k.n_indices, opt.ptr, bytes);
        });
        const float *src = floats(grad_out, "grad_out");
        const int64_t *ids = k.ids(), *bounds = k.bounds();
        float *dst = floats(grad, "grad_array");
        void *s = stream();
        check(released([&] {
            return lib.backward_mixed(h, dims.d.data(), src, ids, bounds, k.n_indices, k.batch, (int32_t)k.n_features, dst, ws.ptr, ws.bytes, opt.ptr, s);
        }));
        Py_RETURN_NONE;
    });
}

// fused_mixed(hash, dims, grad_out, indices, offsets, batch, array, state, lr, eps, workspace, options)
PyObject *call_fused_mixed(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 12, [&]() -> PyObject * {
        View<robe_hash_t> hv(a[0], "hash");
        const robe_hash_t *h = need(hv);
        const Dims dims(a[1]);
        const at::Tensor &array = tensor(a[6], "array"), &state = tensor(a[7], "state"), &grad_out = tensor(a[2], "grad_out");
        same_length(array, h, "array / state length differs from hash.m");
        same_length(state, h, "array / state length differs from hash.m");
        const int64_t batch = integer(a[5]);
        if (grad_out.numel() != batch * dims.sum) raise(PyExc_ValueError, "grad_out has the wrong size");
        const Tokens k(a[3], a[4], batch, (int64_t)dims.d.size());
        View<robe_options_t> opt(a[11], "options");
        const Workspace ws(a[10], array, [&](size_t *bytes) {
            return lib.fused_mixed_workspace_bytes(h, dims.d.data(), k.batch, (int32_t)k.n_features, k.n_indices, opt.ptr, bytes);
        });
        const float *src = floats(grad_out, "grad_out");
        const int64_t *ids = k.ids(), *bounds = k.bounds();
        float *w = floats(array, "array"), *st = floats(state, "state");
        const float lr = real(a[8]), eps = real(a[9]);
        void *s = stream();
        check(released([&] {
            return lib.backward_adagrad_mixed(h, dims.d.data(), src, ids, bounds, k.n_indices, k.batch, (int32_t)k.n_features, w, st, lr, eps,
                                              ws.ptr, ws.bytes, opt.ptr, s);
        }));
        Py_RETURN_NONE;
    });
}

// bind(path of librobe.so, RobeError)
PyObject *call_bind(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 2) {
        PyErr_SetString(PyExc_TypeError, "bind(path, error class)");
        return nullptr;
    }
    const char *path = PyUnicode_AsUTF8(a[0]);
    if (path == nullptr) return nullptr;
    void *so = dlopen(path, RTLD_NOW | RTLD_LOCAL);
    if (so == nullptr) return PyErr_Format(PyExc_ImportError, "%s", dlerror());
    Entry e = {};
    const char *missing = nullptr;
#define ROBE_ENTRY(name) if ((e.name = reinterpret_cast<decltype(e.name)>(dlsym(so, "robe_" #name))) == nullptr) missing = #name
    ROBE_ENTRY(forward); ROBE_ENTRY(forward_bf16); ROBE_ENTRY(backward); ROBE_ENTRY(backward_noalloc); ROBE_ENTRY(workspace_bytes);
    ROBE_ENTRY(adagrad_update); ROBE_ENTRY(sgd_update); ROBE_ENTRY(fused_workspace_bytes); ROBE_ENTRY(backward_adagrad); ROBE_ENTRY(backward_sgd);
    ROBE_ENTRY(forward_mixed); ROBE_ENTRY(mixed_workspace_bytes); ROBE_ENTRY(backward_mixed); ROBE_ENTRY(fused_mixed_workspace_bytes);
    ROBE_ENTRY(backward_adagrad_mixed); ROBE_ENTRY(last_error);
#undef ROBE_ENTRY
    if (missing != nullptr) return PyErr_Format(PyExc_ImportError, "%s has no robe_%s", path, missing);
    Py_INCREF(a[1]);
    Py_XSETREF(g_error, a[1]);
    lib = e;
    Py_RETURN_NONE;
}

#define ROBE_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(call_##name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {ROBE_METHOD(bind), ROBE_METHOD(forward), ROBE_METHOD(backward), ROBE_METHOD(update), ROBE_METHOD(fused),
                         ROBE_METHOD(forward_mixed), ROBE_METHOD(backward_mixed), ROBE_METHOD(fused_mixed), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_robe_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__robe_call(void) { return PyModule_Create(&module); }
