// Marshalling of the Python binding's calls in native code: tensors and parameters to the C ABI of
// include/hdqt.h and back (module _host; binding.py calls it).
//
// A small layer's step (64 x 256 x 128) is three launches, 12 us of kernels one by one, of 2.6 us each on the host;
// the interpreter's share of a call (parameter structures, pointers, checks) was 6.4 us on top of them and
// decided how long the call took: 16.3 us among others, now 13.4 with a share of about 1.5.  The library does
// not need this module: without it every call goes through ctypes.
//
// Every function takes the ordinary form of a call only -- plain tensors in device memory, contiguous, in
// the types of the ABI, integers that are integers -- and returns None for any other: binding.py then goes
// through its own checks, which raise what they always raised.  A refusal of the library comes back as its
// code (an int), a result as a tuple.  The interpreter's lock is not held during the library's call.

#include <Python.h>
#include <dlfcn.h>

#include <optional>

#include <ATen/ops/empty.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/hdqt.h"

namespace {

struct Library {
    decltype(&hdqt_codes_pitch) codes_pitch;
    decltype(&hdqt_quantize_workspace_size) quantize_workspace_size;
    decltype(&hdqt_quantize) quantize;
    decltype(&hdqt_workspace_size) workspace_size, workspace_least;
    decltype(&hdqt_gemm_fwd) gemm[3];
    decltype(&hdqt_gemm_bwd_input_bf16) gemm_bf16;
    decltype(&hdqt_gemm_bwd_input_masked) gemm_masked;
    decltype(&hdqt_layer_step_workspace_size) step_workspace_size;
    decltype(&hdqt_layer_step) step;
    decltype(&hdqt_layer_saved_size) saved_size;
    decltype(&hdqt_layer_fwd_workspace_size) fwd_workspace_size;
    decltype(&hdqt_layer_fwd) fwd;
    decltype(&hdqt_conv_fwd) conv_fwd;
    decltype(&hdqt_layer_bwd_workspace_size) bwd_workspace_size;
    decltype(&hdqt_layer_bwd) bwd;
    decltype(&hdqt_layer_bwd_masked) bwd_masked;
    decltype(&hdqt_conv_bwd) conv_bwd;
    decltype(&hdqt_conv_bwd_masked) conv_bwd_masked;
} lib;
PyObject *get_device, *get_stream;           // torch's: the current device, its current stream's handle

struct Names {
    PyObject *had_block, *acc_bits, *s, *seed, *A, *B, *b, *round, *clip, *tensor_id, *cuda_stream;
} names;

// Not the ordinary form of a call.
struct Other {};

const at::Tensor& tensor(PyObject* o, at::ScalarType type, int64_t dim = -1)
{
    if (!THPVariable_CheckExact(o)) throw Other();
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_cuda() || !t.is_contiguous() || t.scalar_type() != type || (dim >= 0 && t.dim() != dim)) throw Other();
    return t;
}

const at::Tensor* maybe(PyObject* o, at::ScalarType type) { return o == Py_None ? nullptr : &tensor(o, type); }

void* address(const at::Tensor& t) { return t.data_ptr(); }
void* address(const at::Tensor* t) { return t ? t->data_ptr() : nullptr; }

int64_t integer(PyObject* o)
{
    if (!PyLong_Check(o)) throw Other();
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw Other();
    return v;
}

struct Member {
    PyObject* o;
    Member(PyObject* of, PyObject* name) : o(PyObject_GetAttr(of, name)) { if (!o) throw Other(); }
    ~Member() { Py_DECREF(o); }
};

// The members of a tuple or a list of n, kept for the call (a list may change while the interpreter's lock is not held).
struct Members {
    PyObject* t;
    Members(PyObject* o, Py_ssize_t n) : t(PyTuple_Check(o) || PyList_CheckExact(o) ? PySequence_Tuple(o) : nullptr)
    {
        if (t && PyTuple_GET_SIZE(t) == n) return;
        Py_XDECREF(t);
        throw Other();
    }
    ~Members() { Py_DECREF(t); }
    PyObject* operator[](Py_ssize_t k) const { return PyTuple_GET_ITEM(t, k); }
};

// (modulo 2^64 and then the field's width, as ctypes stores an integer)
uint64_t bits_of(PyObject* of, PyObject* name)
{
    const Member m(of, name);
    if (!PyLong_Check(m.o)) throw Other();
    const unsigned long long v = PyLong_AsUnsignedLongLongMask(m.o);
    if (PyErr_Occurred()) throw Other();
    return v;
}

hdqt_operand_t operand(PyObject* o)
{
    const Member clip(o, names.clip);
    const double c = PyFloat_AsDouble(clip.o);
    if (PyErr_Occurred()) throw Other();
    return {(int32_t)bits_of(o, names.b), (int32_t)bits_of(o, names.round), (float)c, (uint32_t)bits_of(o, names.tensor_id)};
}

hdqt_params_t params(PyObject* o)
{
    const Member A(o, names.A), B(o, names.B);
    return {(int32_t)bits_of(o, names.had_block), (int32_t)bits_of(o, names.acc_bits), (int64_t)bits_of(o, names.s),
            bits_of(o, names.seed), operand(A.o), operand(B.o)};
}

struct MaybeParams {
    hdqt_params_t value;
    const hdqt_params_t* p = nullptr;
    explicit MaybeParams(PyObject* o) { if (o != Py_None) { value = params(o); p = &value; } }
};

void* handle_of(PyObject* stream)
{
    PyObject* h = nullptr;
    if (stream == Py_None) {
        PyObject* device = PyObject_CallNoArgs(get_device);
        if (device) { h = PyObject_CallOneArg(get_stream, device); Py_DECREF(device); }
    } else {
        h = PyObject_GetAttr(stream, names.cuda_stream);
    }
    if (!h) throw Other();
    void* p = PyLong_AsVoidPtr(h);
    Py_DECREF(h);
    if (PyErr_Occurred()) throw Other();
    return p;
}

at::Tensor fresh(at::IntArrayRef shape, at::ScalarType type, const at::Tensor& beside)
{
    return at::empty(shape, at::TensorOptions().dtype(type).device(beside.device()));
}

at::Tensor bytes(size_t n, const at::Tensor& beside) { return fresh({(int64_t)(n > 256 ? n : 256)}, at::kByte, beside); }

template <typename F>
int unlocked(F call)
{
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = call();
    Py_END_ALLOW_THREADS
    return rc;
}

// an argument that was given comes back as the object it was, a new tensor as a new object
struct Result {
    PyObject* o;
    explicit Result(PyObject* given) : o(Py_NewRef_(given)) {}
    explicit Result(at::Tensor t) : o(t.defined() ? THPVariable_Wrap(std::move(t)) : Py_NewRef_(Py_None)) {}
    static PyObject* Py_NewRef_(PyObject* x) { Py_INCREF(x); return x; }
};

template <typename... R>
PyObject* tuple(R... r)
{
    PyObject* t = PyTuple_New(sizeof...(R));
    Py_ssize_t k = 0;
    (PyTuple_SET_ITEM(t, k++, r.o), ...);
    return t;
}

// quantize(T, axis, had_block, op, seed, stream) -> (codes, scale)
PyObject* quantize(PyObject* const* a)
{
    const at::Tensor& T = tensor(a[0], at::kFloat, 2);
    const int64_t axis = integer(a[1]), had = integer(a[2]), rows = T.size(0), cols = T.size(1);
    const hdqt_operand_t op = operand(a[3]);
    if (!PyLong_Check(a[4])) throw Other();
    const uint64_t seed = PyLong_AsUnsignedLongLongMask(a[4]);
    if (PyErr_Occurred() || (axis != 0 && axis != 1)) throw Other();
    void* stream = handle_of(a[5]);
    const int64_t D = axis ? cols : rows, lines = axis ? rows : cols;
    at::Tensor codes = fresh({lines, lib.codes_pitch(D, op.b)}, at::kByte, T), scale = fresh({1}, at::kFloat, T);
    at::Tensor ws = fresh({(int64_t)lib.quantize_workspace_size()}, at::kByte, T);
    void *pT = address(T), *pc = address(codes), *ps = address(scale), *pw = address(ws);
    const size_t n = (size_t)ws.numel();
    const int rc = unlocked([&] {
        return lib.quantize((const float*)pT, rows, cols, (int)axis, (int)had, &op, seed, pc, (float*)ps, pw, n, stream);
    });
    if (rc) return PyLong_FromLong(rc);
    return tuple(Result(std::move(codes)), Result(std::move(scale)));
}

// gemm(kind, P, Q, M, K, N, params, out, acc, want_acc, workspace, stream, bf16, mask) -> (out, acc | None, workspace)
PyObject* gemm(PyObject* const* a)
{
    const int64_t kind = integer(a[0]), M = integer(a[3]), K = integer(a[4]), N = integer(a[5]);
    if (kind < 0 || kind > 2 || !PyBool_Check(a[9]) || !PyBool_Check(a[12])) throw Other();
    const at::Tensor &P = tensor(a[1], at::kFloat), &Q = tensor(a[2], at::kFloat);
    const bool want_acc = a[9] == Py_True, bf16 = a[12] == Py_True, masked = a[13] != Py_None;
    const at::ScalarType type = bf16 ? at::kBFloat16 : at::kFloat;
    const int64_t rows = kind == HDQT_GEMM_BWD_WEIGHT ? K : M, cols = kind == HDQT_GEMM_BWD_INPUT ? K : N;
    if ((bf16 || masked) && kind != HDQT_GEMM_BWD_INPUT) throw Other();
    if (bf16 && masked) throw Other();
    const at::Tensor* mask = maybe(a[13], at::kFloat);
    if (mask && (mask->dim() != 2 || mask->size(0) != rows || mask->size(1) != cols)) throw Other();
    const hdqt_params_t p = params(a[6]);
    const at::Tensor *given = maybe(a[7], type), *given_acc = maybe(a[8], at::kInt), *given_ws = maybe(a[10], at::kByte);
    void* stream = handle_of(a[11]);
    at::Tensor out, acc, ws;
    if (!given) out = fresh({rows, cols}, type, P);
    if (!given_acc && want_acc) acc = fresh({rows, cols}, at::kInt, P);
    if (!given_ws) ws = bytes((bf16 || masked ? lib.workspace_least : lib.workspace_size)((int)kind, M, K, N, &p), P);
    const float *pP = (const float*)address(P), *pQ = (const float*)address(Q), *pm = (const float*)address(mask);
    void *po = given ? address(given) : address(out), *pw = given_ws ? address(given_ws) : address(ws);
    int32_t* pa = (int32_t*)(given_acc ? address(given_acc) : acc.defined() ? address(acc) : nullptr);
    const size_t n = (size_t)(given_ws ? given_ws->numel() : ws.numel());
    const int rc = unlocked([&] {
        if (bf16) return lib.gemm_bf16(pP, pQ, (uint16_t*)po, M, K, N, &p, pa, pw, n, stream);
        if (masked) return lib.gemm_masked(pP, pQ, pm, (float*)po, M, K, N, &p, pa, pw, n, stream);
        return lib.gemm[kind](pP, pQ, (float*)po, M, K, N, &p, pa, pw, n, stream);
    });
    if (rc) return PyLong_FromLong(rc);
    return tuple(given ? Result(a[7]) : Result(std::move(out)), given_acc ? Result(a[8]) : Result(std::move(acc)),
                 given_ws ? Result(a[10]) : Result(std::move(ws)));
}

// layer_step(X, W, G, fwd, bwd_input | None, bwd_weight, out | None, workspace | None, stream) -> (Z, dX | None, dW, workspace)
PyObject* layer_step(PyObject* const* a)
{
    const at::Tensor &X = tensor(a[0], at::kFloat, 2), &W = tensor(a[1], at::kFloat, 2), &G = tensor(a[2], at::kFloat, 2);
    const int64_t M = X.size(0), K = X.size(1), N = W.size(1);
    if (W.size(0) != K || G.size(0) != M || G.size(1) != N) throw Other();
    const hdqt_params_t fwd = params(a[3]), bww = params(a[5]);
    const MaybeParams bwi(a[4]);
    const at::Tensor* given_ws = maybe(a[7], at::kByte);
    void* stream = handle_of(a[8]);
    std::optional<Members> given;
    at::Tensor made[3], ws;
    float* po[3];
    if (a[6] == Py_None) {
        made[0] = fresh({M, N}, at::kFloat, X);
        if (bwi.p) made[1] = fresh({M, K}, at::kFloat, X);
        made[2] = fresh({K, N}, at::kFloat, X);
        for (int k = 0; k < 3; ++k) po[k] = made[k].defined() ? (float*)address(made[k]) : nullptr;
    } else {
        given.emplace(a[6], 3);
        for (int k = 0; k < 3; ++k) po[k] = (float*)address(maybe((*given)[k], at::kFloat));
    }
    if (!given_ws) ws = bytes(lib.step_workspace_size(M, K, N, &fwd, bwi.p, &bww), X);
    const float *pX = (const float*)address(X), *pW = (const float*)address(W), *pG = (const float*)address(G);
    void* pw = given_ws ? address(given_ws) : address(ws);
    const size_t n = (size_t)(given_ws ? given_ws->numel() : ws.numel());
    const int rc = unlocked([&] { return lib.step(pX, pW, pG, po[0], po[1], po[2], M, K, N, &fwd, bwi.p, &bww, pw, n, stream); });
    if (rc) return PyLong_FromLong(rc);
    auto result = [&](int k) { return given ? Result((*given)[k]) : Result(std::move(made[k])); };
    return tuple(result(0), result(1), result(2), given_ws ? Result(a[7]) : Result(std::move(ws)));
}

// layer_fwd(X, W, fwd, bwd_weight | None, out | None, saved | None, workspace | None, stream) -> (Z, saved | None)
PyObject* layer_fwd(PyObject* const* a)
{
    const at::Tensor &X = tensor(a[0], at::kFloat, 2), &W = tensor(a[1], at::kFloat, 2);
    const int64_t M = X.size(0), K = X.size(1), N = W.size(1);
    if (W.size(0) != K) throw Other();
    const hdqt_params_t fwd = params(a[2]);
    const MaybeParams bww(a[3]);
    const at::Tensor *given = maybe(a[4], at::kFloat), *given_saved = maybe(a[5], at::kByte), *given_ws = maybe(a[6], at::kByte);
    void* stream = handle_of(a[7]);
    at::Tensor out, saved, ws;
    if (!given) out = fresh({M, N}, at::kFloat, X);
    if (!given_saved && bww.p) saved = fresh({(int64_t)lib.saved_size(M, K, bww.p)}, at::kByte, X);
    if (!given_ws) ws = bytes(lib.fwd_workspace_size(M, K, N, &fwd, bww.p), X);
    const float *pX = (const float*)address(X), *pW = (const float*)address(W);
    float* po = (float*)(given ? address(given) : address(out));
    void *ps = given_saved ? address(given_saved) : saved.defined() ? address(saved) : nullptr;
    void* pw = given_ws ? address(given_ws) : address(ws);
    const size_t ns = (size_t)(given_saved ? given_saved->numel() : saved.defined() ? saved.numel() : 0);
    const size_t n = (size_t)(given_ws ? given_ws->numel() : ws.numel());
    const int rc = unlocked([&] { return lib.fwd(pX, pW, po, M, K, N, &fwd, bww.p, ps, ns, pw, n, stream); });
    if (rc) return PyLong_FromLong(rc);
    return tuple(given ? Result(a[4]) : Result(std::move(out)), given_saved ? Result(a[5]) : Result(std::move(saved)));
}

// layer_bwd(G, W, saved, K, bwd_input | None, bwd_weight, out | None, workspace | None, stream, mask | None) -> (dX | None, dW)
PyObject* layer_bwd(PyObject* const* a)
{
    const at::Tensor &G = tensor(a[0], at::kFloat, 2), &W = tensor(a[1], at::kFloat), &saved = tensor(a[2], at::kByte);
    const int64_t M = G.size(0), N = G.size(1), K = integer(a[3]);
    const MaybeParams bwi(a[4]);
    const hdqt_params_t bww = params(a[5]);
    const at::Tensor *given_ws = maybe(a[7], at::kByte), *mask = maybe(a[9], at::kFloat);
    if (K < 0) throw Other();
    if (mask && (!bwi.p || mask->dim() != 2 || mask->size(0) != M || mask->size(1) != K)) throw Other();
    void* stream = handle_of(a[8]);
    std::optional<Members> given;
    at::Tensor made[2], ws;                  // dX, dW
    float* po[2];
    if (a[6] == Py_None) {
        if (bwi.p) made[0] = fresh({M, K}, at::kFloat, G);
        made[1] = fresh({K, N}, at::kFloat, G);
        for (int k = 0; k < 2; ++k) po[k] = made[k].defined() ? (float*)address(made[k]) : nullptr;
    } else {
        given.emplace(a[6], 2);
        for (int k = 0; k < 2; ++k) po[k] = (float*)address(maybe((*given)[k], at::kFloat));
        if (mask && !po[0]) throw Other();
    }
    if (!given_ws) ws = bytes(lib.bwd_workspace_size(M, K, N, bwi.p, &bww), G);
    const float *pG = (const float*)address(G), *pW = (const float*)address(W), *pm = (const float*)address(mask);
    void *ps = address(saved), *pw = given_ws ? address(given_ws) : address(ws);
    const size_t n = (size_t)(given_ws ? given_ws->numel() : ws.numel());
    const int rc = unlocked([&] {
        return pm ? lib.bwd_masked(pG, pW, ps, pm, po[0], po[1], M, K, N, bwi.p, &bww, pw, n, stream)
                  : lib.bwd(pG, pW, ps, po[0], po[1], M, K, N, bwi.p, &bww, pw, n, stream);
    });
    if (rc) return PyLong_FromLong(rc);
    auto result = [&](int k) { return given ? Result((*given)[k]) : Result(std::move(made[k])); };
    return tuple(result(0), result(1));
}

// (window sizes that the geometry's fields hold)
int32_t window(PyObject* o)
{
    const int64_t v = integer(o);
    if (v < 0 || v > INT32_MAX) throw Other();
    return (int32_t)v;
}

// conv_fwd(act, kh, kw, W, fwd, bwd_weight, stream) -> (Z, saved)
PyObject* conv_fwd(PyObject* const* a)
{
    const at::Tensor &act = tensor(a[0], at::kFloat, 4), &W = tensor(a[3], at::kFloat, 2);
    const hdqt_conv_t geo = {act.size(0), (int32_t)act.size(1), (int32_t)act.size(2), (int32_t)act.size(3), window(a[1]), window(a[2])};
    const int64_t M = act.size(0) * act.size(2) * act.size(3), K = act.size(1) * geo.kh * geo.kw, N = W.size(1);
    if (W.size(0) != K) throw Other();
    const hdqt_params_t fwd = params(a[4]), bww = params(a[5]);
    void* stream = handle_of(a[6]);
    at::Tensor out = fresh({M, N}, at::kFloat, act), saved = fresh({(int64_t)lib.saved_size(M, K, &bww)}, at::kByte, act);
    at::Tensor ws = bytes(lib.fwd_workspace_size(M, K, N, &fwd, &bww), act);
    const float *pa = (const float*)address(act), *pW = (const float*)address(W);
    float* po = (float*)address(out);
    void *ps = address(saved), *pw = address(ws);
    const size_t ns = (size_t)saved.numel(), n = (size_t)ws.numel();
    const int rc = unlocked([&] { return lib.conv_fwd(pa, &geo, pW, po, N, &fwd, &bww, ps, ns, pw, n, stream); });
    if (rc) return PyLong_FromLong(rc);
    return tuple(Result(std::move(out)), Result(std::move(saved)));
}

// conv_bwd(G, W, saved, act_shape, kh, kw, bwd_input, bwd_weight, stream, mask | None) -> (dAct, dW)
PyObject* conv_bwd(PyObject* const* a)
{
    const at::Tensor &G = tensor(a[0], at::kFloat, 2), &W = tensor(a[1], at::kFloat, 2), &saved = tensor(a[2], at::kByte);
    const Members shape(a[3], 4);
    int64_t d[4];
    for (int k = 0; k < 4; ++k) {
        d[k] = integer(shape[k]);
        if (d[k] < 0 || d[k] > INT32_MAX) throw Other();
    }
    const hdqt_conv_t geo = {d[0], (int32_t)d[1], (int32_t)d[2], (int32_t)d[3], window(a[4]), window(a[5])};
    const int64_t M = d[0] * d[2] * d[3], K = d[1] * geo.kh * geo.kw, N = G.size(1);
    if (G.size(0) != M || W.size(0) != K || W.size(1) != N) throw Other();
    const hdqt_params_t bwi = params(a[6]), bww = params(a[7]);
    const at::Tensor* mask = maybe(a[9], at::kFloat);
    if (mask && (mask->dim() != 4 || mask->sizes() != at::IntArrayRef(d, 4))) throw Other();
    void* stream = handle_of(a[8]);
    at::Tensor dAct = fresh(at::IntArrayRef(d, 4), at::kFloat, G), dW = fresh({K, N}, at::kFloat, G);
    at::Tensor ws = bytes(lib.bwd_workspace_size(M, K, N, &bwi, &bww), G);
    const float *pG = (const float*)address(G), *pW = (const float*)address(W), *pm = (const float*)address(mask);
    float *px = (float*)address(dAct), *pd = (float*)address(dW);
    void *ps = address(saved), *pw = address(ws);
    const size_t n = (size_t)ws.numel();
    const int rc = unlocked([&] {
        return pm ? lib.conv_bwd_masked(pG, pW, ps, &geo, pm, px, pd, N, &bwi, &bww, pw, n, stream)
                  : lib.conv_bwd(pG, pW, ps, &geo, px, pd, N, &bwi, &bww, pw, n, stream);
    });
    if (rc) return PyLong_FromLong(rc);
    return tuple(Result(std::move(dAct)), Result(std::move(dW)));
}

// What a function may throw (a call of another form; whatever an allocation or a tensor without
// memory of its own raises, which the other way raises again) ends here.  So do the interpreter's errors that
// only say that a member is missing or no number; any other (an interrupt or a time limit's exception out of
// torch's functions, a property's own error) is the caller's.
template <PyObject* (*F)(PyObject* const*), Py_ssize_t ARGS>
PyObject* entry(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    if (lib.step && n == ARGS) {
        try {
            return F(a);
        } catch (...) {
            if (PyErr_Occurred() && !PyErr_ExceptionMatches(PyExc_AttributeError) && !PyErr_ExceptionMatches(PyExc_TypeError) &&
                !PyErr_ExceptionMatches(PyExc_OverflowError))
                return nullptr;
            PyErr_Clear();
        }
    }
    Py_RETURN_NONE;
}

// bind(path of the library, torch's current-device function, torch's current-stream function)
PyObject* bind(PyObject*, PyObject* args)
{
    const char* path;
    PyObject *device, *stream;
    if (!PyArg_ParseTuple(args, "sOO", &path, &device, &stream)) return nullptr;
    void* h = dlopen(path, RTLD_NOW | RTLD_LOCAL);
    if (!h) return PyErr_Format(PyExc_ImportError, "%s", dlerror());
    Library l{};
    bool all = true;
    auto find = [&](auto& f, const char* name) {
        f = reinterpret_cast<std::decay_t<decltype(f)>>(dlsym(h, name));
        all = all && f;
    };
    find(l.codes_pitch, "hdqt_codes_pitch");
    find(l.quantize_workspace_size, "hdqt_quantize_workspace_size");
    find(l.quantize, "hdqt_quantize");
    find(l.workspace_size, "hdqt_workspace_size");
    find(l.workspace_least, "hdqt_workspace_least");
    find(l.gemm[HDQT_GEMM_FWD], "hdqt_gemm_fwd");
    find(l.gemm[HDQT_GEMM_BWD_INPUT], "hdqt_gemm_bwd_input");
    find(l.gemm[HDQT_GEMM_BWD_WEIGHT], "hdqt_gemm_bwd_weight");
    find(l.gemm_bf16, "hdqt_gemm_bwd_input_bf16");
    find(l.gemm_masked, "hdqt_gemm_bwd_input_masked");
    find(l.step_workspace_size, "hdqt_layer_step_workspace_size");
    find(l.step, "hdqt_layer_step");
    find(l.saved_size, "hdqt_layer_saved_size");
    find(l.fwd_workspace_size, "hdqt_layer_fwd_workspace_size");
    find(l.fwd, "hdqt_layer_fwd");
    find(l.conv_fwd, "hdqt_conv_fwd");
    find(l.bwd_workspace_size, "hdqt_layer_bwd_workspace_size");
    find(l.bwd, "hdqt_layer_bwd");
    find(l.bwd_masked, "hdqt_layer_bwd_masked");
    find(l.conv_bwd, "hdqt_conv_bwd");
    find(l.conv_bwd_masked, "hdqt_conv_bwd_masked");
    if (!all) return PyErr_Format(PyExc_ImportError, "%s lacks functions of include/hdqt.h", path);
    Py_INCREF(device);
    Py_INCREF(stream);
    get_device = device;
    get_stream = stream;
    lib = l;
    Py_RETURN_NONE;
}

#define HDQT_ENTRY(F, ARGS) {#F, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&entry<F, ARGS>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"bind", bind, METH_VARARGS, nullptr},
    HDQT_ENTRY(quantize, 6), HDQT_ENTRY(gemm, 14), HDQT_ENTRY(layer_step, 9), HDQT_ENTRY(layer_fwd, 8),
    HDQT_ENTRY(layer_bwd, 10), HDQT_ENTRY(conv_fwd, 7), HDQT_ENTRY(conv_bwd, 10),
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

} // namespace

PyMODINIT_FUNC PyInit__host()
{
#define HDQT_NAME(x) names.x = PyUnicode_InternFromString(#x)
    HDQT_NAME(had_block); HDQT_NAME(acc_bits); HDQT_NAME(s); HDQT_NAME(seed); HDQT_NAME(A); HDQT_NAME(B);
    HDQT_NAME(b); HDQT_NAME(round); HDQT_NAME(clip); HDQT_NAME(tensor_id); HDQT_NAME(cuda_stream);
#undef HDQT_NAME
    return PyModule_Create(&module);
}
