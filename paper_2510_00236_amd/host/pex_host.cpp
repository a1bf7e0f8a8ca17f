// pex_host.cpp -- the binding's calls in native code: what Python checks of every tensor before a call of libpex (a dense tensor on the GPU,
// its element type and size) and the call itself, for the calls a training loop repeats.
//
// A function here does a call only if everything is as the call wants it: plain tensors on the GPU, outputs and workspace given, the
// current stream.  It returns True (or the results) once the library has taken the call, False where anything is otherwise -- nothing
// has been launched then, and the Python path makes the checks again one by one and raises what it always raised -- and the status
// of a launch the HIP runtime refused.  Nothing is kept between calls but the looked-up classes and functions.  Addresses are taken under the
// interpreter's lock (taking one can throw), the library's call is made without it.
//
// Small calls are bound by the host, 3.5 us of a launch and the checks in Python beside it (identity and square of a small layer 6.6 us a call).
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <cxxabi.h>

#include "pex.h"

namespace {

PyObject *adam_class, *moment_class, *get_device, *get_stream;      // set once by setup()
PyObject* names[3];                                                 // "identity", "square", "sign"

constexpr auto F32 = at::kFloat, F64 = at::kDouble, U8 = at::kByte;

// a tensor whose address may be passed on as it is, and that address; t == nullptr: it may not
struct Buffer {
    const at::Tensor* t = nullptr;
    void* at = nullptr;
    size_t n = 0;
    explicit operator bool() const { return t != nullptr; }
    const at::Tensor* operator->() const { return t; }
    float* f() const { return (float*)at; }
    double* d() const { return (double*)at; }
};
Buffer plain(PyObject* o)
{
    if (!o || !THPVariable_CheckExact(o)) return {};
    const at::Tensor& t = THPVariable_Unpack(o);
    const at::TensorImpl* i = t.unsafeGetTensorImpl();
    if (!t.defined() || !i->has_storage() || i->is_python_dispatch() || i->has_symbolic_sizes_strides() || !t.is_cuda() ||
        t.layout() != at::kStrided || !t.is_contiguous())
        return {};
    // under a transform of functions a tensor may stand for another one
    constexpr c10::DispatchKeySet wrapped({c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::FuncTorchGradWrapper, c10::DispatchKey::Functionalize,
                                           c10::DispatchKey::ZeroTensor});
    if (i->key_set().has_any(wrapped)) return {};
    return {&t, t.data_ptr(), (size_t)t.numel()};
}
Buffer plain(PyObject* o, at::ScalarType type)
{
    const Buffer b = plain(o);
    return b && b->scalar_type() == type ? b : Buffer{};
}
Buffer sized(PyObject* o, at::ScalarType type, int64_t n)
{
    const Buffer b = plain(o, type);
    return b && b->numel() == n ? b : Buffer{};
}
Buffer matrix(PyObject* o, int64_t rows, int64_t cols)
{
    const Buffer b = plain(o, F32);
    return b && b->dim() == 2 && b->size(0) == rows && b->size(1) == cols ? b : Buffer{};
}

bool modes_active()
{
    return at::impl::torch_function_mode_enabled() || c10::impl::TorchDispatchModeTLS::any_modes_set();
}

// the raw handle of torch's current stream on the current device
bool current_stream(pex_stream_t* stream)
{
    PyObject* device = PyObject_CallNoArgs(get_device);
    PyObject* raw = device ? PyObject_CallOneArg(get_stream, device) : nullptr;
    Py_XDECREF(device);
    if (raw) *stream = (pex_stream_t)PyLong_AsVoidPtr(raw);
    Py_XDECREF(raw);
    if (!PyErr_Occurred()) return true;
    PyErr_Clear();
    return false;
}

struct Layer {
    Buffer X, G;
    int64_t B, T, din, dout;
    pex_dtype dt;
    bool take(PyObject* x, PyObject* g)
    {
        X = plain(x);
        G = plain(g);
        if (!X || !G || X->dim() != 3 || G->dim() != 3 || X->scalar_type() != G->scalar_type()) return false;
        if (X->scalar_type() != F32 && X->scalar_type() != at::kBFloat16) return false;
        dt = X->scalar_type() == F32 ? PEX_F32 : PEX_BF16;
        B = X->size(0);
        T = X->size(1);
        din = X->size(2);
        dout = G->size(2);
        return B == G->size(0) && T == G->size(1);
    }
};

bool integer(PyObject* o, int64_t* v)
{
    if (!PyLong_CheckExact(o)) return false;
    *v = PyLong_AsLongLong(o);
    if (!PyErr_Occurred()) return true;
    PyErr_Clear();
    return false;
}
bool real(PyObject* o, float* v)
{
    if (!PyFloat_CheckExact(o)) return false;
    *v = (float)PyFloat_AS_DOUBLE(o);
    return true;
}
// a parameter structure of the binding
template <typename P>
bool structure(PyObject* o, PyObject* cls, P* out)
{
    if ((PyObject*)Py_TYPE(o) != cls) return false;
    Py_buffer b;
    if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) {
        PyErr_Clear();
        return false;
    }
    const bool ok = b.len == (Py_ssize_t)sizeof(P);
    if (ok) memcpy(out, b.buf, sizeof(P));
    PyBuffer_Release(&b);
    return ok;
}

// The call, without the interpreter's lock; `ok` is what a call returns that was taken.  (An exception out of the library may have left
// part of a call on the stream: it is an error, and not a call for the Python path to make again.)
template <typename F>
PyObject* done(F&& call, PyObject* ok = nullptr)
{
    pex_status st = PEX_OK;
    bool thrown = false;
    PyThreadState* const state = PyEval_SaveThread();
    try {
        st = call();
    } catch (...) {
        thrown = true;
    }
    PyEval_RestoreThread(state);
    if (st == PEX_OK && !thrown) {
        if (!ok) Py_RETURN_TRUE;
        return ok;
    }
    Py_XDECREF(ok);
    if (thrown) {
        PyErr_SetString(PyExc_RuntimeError, "libpex: an exception left a call");
        return nullptr;
    }
    if (st == PEX_ERR_HIP) return PyLong_FromLong(st);
    Py_RETURN_FALSE;
}

#define PEX_NEEDS(COND) do { if (!(COND)) Py_RETURN_FALSE; } while (0)

// stat(X, G, phi, S, workspace)
PyObject* host_stat(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    Layer l;
    int64_t phi;
    pex_stream_t s;
    PEX_NEEDS(n == 5 && !modes_active() && l.take(a[0], a[1]) && integer(a[2], &phi));
    const Buffer S = matrix(a[3], l.din, l.dout), ws = plain(a[4], U8);
    PEX_NEEDS(S && ws && current_stream(&s));
    return done([&] { return pex_stat(l.X.at, l.G.at, l.B, l.T, l.din, l.dout, l.dt, (pex_phi)phi, S.f(), ws.at, ws.n, s); });
}

// token_sq(X, G, S, workspace)
PyObject* host_token_sq(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    Layer l;
    pex_stream_t s;
    PEX_NEEDS(n == 4 && !modes_active() && l.take(a[0], a[1]));
    const Buffer S = matrix(a[2], l.din, l.dout), ws = plain(a[3], U8);
    PEX_NEEDS(S && ws && current_stream(&s));
    return done([&] { return pex_token_sq(l.X.at, l.G.at, l.B, l.T, l.din, l.dout, l.dt, S.f(), ws.at, ws.n, s); });
}

// example_norms(X, G, N, workspace)
PyObject* host_example_norms(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    Layer l;
    pex_stream_t s;
    PEX_NEEDS(n == 4 && !modes_active() && l.take(a[0], a[1]));
    const Buffer N = sized(a[2], F32, l.B), ws = plain(a[3], U8);
    PEX_NEEDS(N && ws && current_stream(&s));
    return done([&] { return pex_example_norms(l.X.at, l.G.at, l.B, l.T, l.din, l.dout, l.dt, N.f(), ws.at, ws.n, s); });
}

// weighted_sum(X, G, w, S, workspace)
PyObject* host_weighted_sum(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    Layer l;
    pex_stream_t s;
    PEX_NEEDS(n == 5 && !modes_active() && l.take(a[0], a[1]));
    const Buffer w = sized(a[2], F32, l.B), S = matrix(a[3], l.din, l.dout), ws = plain(a[4], U8);
    PEX_NEEDS(w && S && ws && current_stream(&s));
    return done([&] {
        return pex_weighted_sum(l.X.at, l.G.at, w.f(), l.B, l.T, l.din, l.dout, l.dt, S.f(), ws.at, ws.n, s);
    });
}

// The addresses of the wanted outputs of `out`, a dict (cols < 0: vectors of `rows`)
bool outputs(PyObject* out, int64_t want, int64_t rows, int64_t cols, float* (&at)[3])
{
    if (!PyDict_CheckExact(out) || want < 1 || want > 7) return false;
    for (int k = 0; k < 3; ++k) {
        at[k] = nullptr;
        if (!(want >> k & 1)) continue;
        PyObject* o = PyDict_GetItem(out, names[k]);
        const Buffer b = cols < 0 ? sized(o, F32, rows) : matrix(o, rows, cols);
        if (!b) return false;
        at[k] = b.f();
    }
    return true;
}
// The wanted outputs of `out` as a new dict in the order of the names, nullptr with an error set
PyObject* results(PyObject* out, int64_t want)
{
    PyObject* res = PyDict_New();
    for (int k = 0; k < 3 && res; ++k) {
        if (!(want >> k & 1)) continue;
        PyObject* o = PyDict_GetItem(out, names[k]);
        if (!o || PyDict_SetItem(res, names[k], o) != 0) Py_CLEAR(res);
    }
    if (!res && !PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, "an output left its dict during the call");
    return res;
}
// The same of the last members of a list's tuples, as a list
PyObject* results_of_all(PyObject* list, Py_ssize_t count, int64_t want)
{
    PyObject* res = PyList_New(count);
    for (Py_ssize_t k = 0; k < count && res; ++k) {
        PyObject* d = results(PyTuple_GET_ITEM(PyList_GET_ITEM(list, k), 2), want);
        if (d) PyList_SET_ITEM(res, k, d);
        else Py_CLEAR(res);
    }
    return res;
}

// stat_multi(X, G, want, out, workspace) -> the dict of the results
PyObject* host_stat_multi(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    Layer l;
    int64_t want;
    pex_stream_t s;
    float* S[3];
    PEX_NEEDS(n == 5 && !modes_active() && l.take(a[0], a[1]) && integer(a[2], &want));
    const Buffer ws = plain(a[4], U8);
    PEX_NEEDS(ws && current_stream(&s) && outputs(a[3], want, l.din, l.dout, S));
    PyObject* res = results(a[3], want);
    if (!res) return nullptr;
    return done([&] {
        return pex_stat_multi(l.X.at, l.G.at, l.B, l.T, l.din, l.dout, l.dt, (uint32_t)want, S[0], S[1], S[2], ws.at, ws.n, s);
    }, res);
}

// embed_stat(ids, G, V, want, out, workspace) -> the dict of the results
PyObject* host_embed_stat(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    int64_t V, want;
    pex_stream_t s;
    float* S[3];
    PEX_NEEDS(n == 6 && !modes_active() && integer(a[2], &V) && integer(a[3], &want));
    const Buffer ids = plain(a[0]), G = plain(a[1]), ws = plain(a[5], U8);
    PEX_NEEDS(ids && G && ws && ids->dim() == 2 && G->dim() == 3 && ids->size(0) == G->size(0) && ids->size(1) == G->size(1));
    PEX_NEEDS((ids->scalar_type() == at::kLong || ids->scalar_type() == at::kInt) && (G->scalar_type() == F32 || G->scalar_type() == at::kBFloat16));
    const int64_t B = G->size(0), T = G->size(1), d = G->size(2);
    const int32_t id_size = (int32_t)ids->element_size();
    const pex_dtype dt = G->scalar_type() == F32 ? PEX_F32 : PEX_BF16;
    PEX_NEEDS(current_stream(&s) && outputs(a[4], want, V, d, S));
    PyObject* res = results(a[4], want);
    if (!res) return nullptr;
    return done([&] {
        return pex_embed_stat(ids.at, id_size, G.at, B, T, V, d, dt, (uint32_t)want, S[0], S[1], S[2], ws.at, ws.n, s);
    }, res);
}

// clip_weights(N, max_norm, w)
PyObject* host_clip_weights(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    float max_norm;
    pex_stream_t s;
    PEX_NEEDS(n == 3 && !modes_active() && real(a[1], &max_norm));
    const Buffer N = plain(a[0], F32);
    PEX_NEEDS(N && (N->dim() == 1 || N->dim() == 2));
    const int64_t layers = N->dim() == 1 ? 1 : N->size(0), B = N->size(N->dim() - 1);
    const Buffer w = sized(a[2], F32, B);
    PEX_NEEDS(w && layers < ((int64_t)1 << 31) && current_stream(&s));
    return done([&] { return pex_clip_weights(N.f(), B, (int32_t)layers, max_norm, w.f(), s); });
}

// adam_update(theta, m, v, S_id, S_sq or None, variant, params)
PyObject* host_adam_update(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    int64_t variant;
    pex_adam_params prm;
    pex_stream_t s;
    PEX_NEEDS(n == 7 && !modes_active() && integer(a[5], &variant) && structure(a[6], adam_class, &prm));
    const Buffer theta = plain(a[0], F32);
    PEX_NEEDS(theta);
    const int64_t count = theta->numel();
    const Buffer m = sized(a[1], F32, count), v = sized(a[2], F32, count), id = sized(a[3], F32, count), sq = a[4] == Py_None ? Buffer{} : sized(a[4], F32, count);
    PEX_NEEDS(m && v && id && (sq || a[4] == Py_None) && current_stream(&s));
    return done([&] {
        return pex_adam_update(theta.f(), m.f(), v.f(), id.f(), sq.f(), count, (pex_adam_variant)variant, &prm, s);
    });
}

// signsgd_update(theta, m, S, lr, beta, weight_decay, B, debias, step)
PyObject* host_signsgd_update(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    float lr, beta, decay;
    int64_t B, step;
    pex_stream_t s;
    PEX_NEEDS(n == 9 && !modes_active() && real(a[3], &lr) && real(a[4], &beta) && real(a[5], &decay) && integer(a[6], &B) && PyBool_Check(a[7]) && integer(a[8], &step));
    const Buffer theta = plain(a[0], F32);
    PEX_NEEDS(theta && B >= INT32_MIN && B <= INT32_MAX);
    const int64_t count = theta->numel();
    const Buffer m = sized(a[1], F32, count), S = sized(a[2], F32, count);
    PEX_NEEDS(m && S && current_stream(&s));
    const int32_t debias = a[7] == Py_True;
    return done([&] { return pex_signsgd_update(theta.f(), m.f(), S.f(), count, lr, beta, decay, (int32_t)B, debias, step, s); });
}

// adam_step([(theta, m, v, S_id, S_sq or None[, ema_adam, ema_micro])], variant, params, sum_sq, max_norm, moments or None, sums or None, workspace)
PyObject* host_adam_step(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    int64_t variant;
    pex_adam_params prm;
    pex_moment_params mom;
    float max_norm;
    pex_stream_t s;
    PEX_NEEDS(n == 8 && !modes_active() && PyList_CheckExact(a[0]) && integer(a[1], &variant) && structure(a[2], adam_class, &prm) && real(a[4], &max_norm));
    const bool track = a[5] != Py_None;
    PEX_NEEDS(!track || structure(a[5], moment_class, &mom));
    const Py_ssize_t count = PyList_GET_SIZE(a[0]);
    const int width = track ? 7 : 5;
    const Buffer sum_sq = sized(a[3], F64, 1), sums = track ? sized(a[6], F64, 2 * count) : Buffer{}, ws = plain(a[7], U8);
    PEX_NEEDS(count > 0 && sum_sq && ws && (sums || !track));
    std::vector<pex_step_tensor> rows(count);
    for (Py_ssize_t k = 0; k < count; ++k) {
        PyObject* tuple = PyList_GET_ITEM(a[0], k);
        PEX_NEEDS(PyTuple_CheckExact(tuple) && PyTuple_GET_SIZE(tuple) >= width);
        const Buffer theta = plain(PyTuple_GET_ITEM(tuple, 0), F32);
        PEX_NEEDS(theta);
        float* p[7] = {};
        for (int i = 0; i < width; ++i) {
            PyObject* o = PyTuple_GET_ITEM(tuple, i);
            if (o == Py_None) continue;
            const Buffer t = sized(o, F32, theta->numel());
            PEX_NEEDS(t);
            p[i] = t.f();
        }
        rows[k] = pex_step_tensor{p[0], p[1], p[2], p[3], p[4], p[5], p[6], theta->numel()};
    }
    PEX_NEEDS(current_stream(&s));
    return done([&] {
        return pex_adam_step(rows.data(), (int32_t)count, (pex_adam_variant)variant, &prm, track ? &mom : nullptr, max_norm, sum_sq.d(),
                             sums.d(), ws.at, ws.n, s);
    });
}

// stat_pair_batch([(X, G, out)], workspace) -> the list of dicts of the results
PyObject* host_stat_pair_batch(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    pex_stream_t s;
    PEX_NEEDS(n == 2 && !modes_active() && PyList_CheckExact(a[0]));
    const Py_ssize_t count = PyList_GET_SIZE(a[0]);
    const Buffer ws = plain(a[1], U8);
    PEX_NEEDS(count > 0 && ws && current_stream(&s));
    std::vector<pex_pair_item> items(count);
    Layer first{}, l;
    for (Py_ssize_t k = 0; k < count; ++k) {
        PyObject* tuple = PyList_GET_ITEM(a[0], k);
        float* S[3];
        PEX_NEEDS(PyTuple_CheckExact(tuple) && PyTuple_GET_SIZE(tuple) == 3 && l.take(PyTuple_GET_ITEM(tuple, 0), PyTuple_GET_ITEM(tuple, 1)));
        if (k == 0) first = l;
        PEX_NEEDS(l.B == first.B && l.T == first.T && l.dt == first.dt);
        PEX_NEEDS(outputs(PyTuple_GET_ITEM(tuple, 2), PEX_WANT_IDENTITY | PEX_WANT_SQUARE, l.din, l.dout, S));
        items[k] = pex_pair_item{l.X.at, l.G.at, S[0], S[1], l.din, l.dout};
    }
    PyObject* res = results_of_all(a[0], count, PEX_WANT_IDENTITY | PEX_WANT_SQUARE);
    if (!res) return nullptr;
    return done([&] { return pex_stat_pair_batch(items.data(), (int32_t)count, first.B, first.T, first.dt, ws.at, ws.n, s); }, res);
}

// vec_stat_batch([(A, C or None, out)], want, workspace) -> the list of dicts of the results
PyObject* host_vec_stat_batch(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    int64_t want;
    pex_stream_t s;
    PEX_NEEDS(n == 3 && !modes_active() && PyList_CheckExact(a[0]) && integer(a[1], &want));
    const Py_ssize_t count = PyList_GET_SIZE(a[0]);
    const Buffer ws = plain(a[2], U8);
    PEX_NEEDS(count > 0 && ws && want >= 1 && want <= 7 && current_stream(&s));
    std::vector<pex_vec_item> items(count);
    int64_t B = 0, T = 0;
    at::ScalarType type = F32;
    for (Py_ssize_t k = 0; k < count; ++k) {
        PyObject* tuple = PyList_GET_ITEM(a[0], k);
        PEX_NEEDS(PyTuple_CheckExact(tuple) && PyTuple_GET_SIZE(tuple) == 3);
        PyObject* c = PyTuple_GET_ITEM(tuple, 1);
        const Buffer A = plain(PyTuple_GET_ITEM(tuple, 0)), C = c == Py_None ? Buffer{} : plain(c);
        PEX_NEEDS(A && A->dim() == 3 && (A->scalar_type() == F32 || A->scalar_type() == at::kBFloat16) && (C || c == Py_None));
        PEX_NEEDS(!C || (C->scalar_type() == A->scalar_type() && C->sizes() == A->sizes()));
        if (k == 0) {
            B = A->size(0);
            T = A->size(1);
            type = A->scalar_type();
        }
        float* S[3];
        PEX_NEEDS(A->size(0) == B && A->size(1) == T && A->scalar_type() == type && outputs(PyTuple_GET_ITEM(tuple, 2), want, A->size(2), -1, S));
        items[k] = pex_vec_item{A.at, C.at, S[0], S[1], S[2], A->size(2)};
    }
    PyObject* res = results_of_all(a[0], count, want);
    if (!res) return nullptr;
    return done([&] {
        return pex_vec_stat_batch(items.data(), (int32_t)count, B, T, type == F32 ? PEX_F32 : PEX_BF16, (uint32_t)want, ws.at, ws.n, s);
    }, res);
}

// setup(AdamParams, MomentParams, function of the current device's index, function of its stream's handle)
PyObject* host_setup(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    if (n != 4) {
        PyErr_SetString(PyExc_TypeError, "setup takes four arguments");
        return nullptr;
    }
    PyObject** slots[4] = {&adam_class, &moment_class, &get_device, &get_stream};
    for (int k = 0; k < 4; ++k) {
        Py_INCREF(a[k]);
        Py_XDECREF(*slots[k]);
        *slots[k] = a[k];
    }
    Py_RETURN_NONE;
}

// No C++ exception leaves a function: the call is the Python path's then.
template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)>
PyObject* guarded(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    try {
        return F(self, a, n);
    } catch (abi::__forced_unwind&) {      // the end of a thread
        throw;
    } catch (...) {
        if (PyErr_Occurred()) PyErr_Clear();
        Py_RETURN_FALSE;
    }
}

#define PEX_METHOD(NAME) {#NAME, (PyCFunction)(void (*)())guarded<host_##NAME>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {PEX_METHOD(setup), PEX_METHOD(stat), PEX_METHOD(token_sq), PEX_METHOD(example_norms), PEX_METHOD(weighted_sum), PEX_METHOD(stat_multi),
                         PEX_METHOD(embed_stat), PEX_METHOD(clip_weights), PEX_METHOD(adam_update), PEX_METHOD(signsgd_update), PEX_METHOD(adam_step),
                         PEX_METHOD(stat_pair_batch), PEX_METHOD(vec_stat_batch), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pex_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

extern "C" __attribute__((visibility("default"))) PyObject* PyInit__pex_host(void)
{
    const char* text[3] = {"identity", "square", "sign"};
    for (int k = 0; k < 3; ++k)
        if (!(names[k] = PyUnicode_InternFromString(text[k]))) return nullptr;
    PyObject* m = PyModule_Create(&module);
    if (m && PyModule_AddIntConstant(m, "PEX_VERSION", PEX_VERSION) != 0) Py_CLEAR(m);
    return m;
}
