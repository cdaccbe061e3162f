// CPython extension `_native`: argument marshalling of the entry points a training or serving loop calls for every layer
// and token.  Small calls are bound by the host: checking ten tensors and building fifteen ctypes arguments in Python costs
// 10-20 us, more than the kernels of a short pass take; here it is 1-2 us.  No arithmetic of the layer and no torch types
// beyond this file: the library behind it is the plain C ABI.
//
// Every function takes positional arguments only, raises ValueError for a tensor that is not what the descriptor says, and
// returns the library's status code.
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstring>
#include <string>
#include <vector>

#include "race_attn.h"

namespace {

struct BadArgument {};                      // a Python exception has been set

struct Desc {
    race_attn_desc_t d;
    explicit Desc(PyObject *o)
    {
        Py_buffer view;
        if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) throw BadArgument{};
        const bool ok = view.len == static_cast<Py_ssize_t>(sizeof d);
        if (ok) std::memcpy(&d, view.buf, sizeof d);
        PyBuffer_Release(&view);
        if (!ok) {
            PyErr_SetString(PyExc_TypeError, "desc must be a RaceAttnDesc");
            throw BadArgument{};
        }
    }
    at::ScalarType elem() const { return d.dtype == RACE_F32 ? at::kFloat : at::kBFloat16; }
    int32_t heads() const { return d.N == 0 ? 0 : d.H; }       // seeds that a pass over the sequence reads
};

struct Shape { int n; int64_t s[5]; };

void *tensor(PyObject *o, const char *name, const Shape &shape, at::ScalarType type)
{
    if (THPVariable_Check(o)) {
        const at::Tensor &t = THPVariable_Unpack(o);
        bool ok = t.is_cuda() && t.scalar_type() == type && t.dim() == shape.n && t.is_contiguous();
        for (int i = 0; ok && i < shape.n; ++i) ok = t.size(i) == shape.s[i];
        if (ok) return t.data_ptr();
    }
    std::string want;
    for (int i = 0; i < shape.n; ++i) want += (i ? ", " : "") + std::to_string(shape.s[i]);
    PyErr_Format(PyExc_ValueError, "%s must be a contiguous device tensor of shape (%s) and dtype %s", name, want.c_str(),
                 type == at::kFloat ? "torch.float32" : "torch.bfloat16");
    throw BadArgument{};
}
Shape full(const Desc &d) { return Shape{4, {d.d.B, d.d.H, d.d.N, d.d.d}}; }
Shape rows(const Desc &d) { return Shape{3, {d.d.B, d.d.H, d.d.d}}; }
Shape per_token(const Desc &d) { return Shape{3, {d.d.B, d.d.H, d.d.N}}; }
Shape per_head(const Desc &d) { return Shape{2, {d.d.B, d.d.H}}; }
Shape state_shape(const Desc &d)
{
    return Shape{5, {d.d.B, d.d.H, d.d.L, (d.d.P >= 0 && d.d.P < 31) ? int64_t(1) << d.d.P : 0, int64_t(d.d.d) + 1}};
}

struct Workspace {
    void *ptr = nullptr;
    size_t bytes = 0;
    explicit Workspace(PyObject *o)
    {
        if (o == Py_None) return;
        if (!THPVariable_Check(o)) {
            PyErr_SetString(PyExc_ValueError, "workspace must be a device tensor");
            throw BadArgument{};
        }
        const at::Tensor &t = THPVariable_Unpack(o);
        ptr = t.data_ptr();
        bytes = static_cast<size_t>(t.numel()) * t.element_size();
    }
};

// int(s) modulo 2^64 of every element (any number, not integers only).  needed: how many the call reads (an empty sequence
// needs none); None is for the decoding step alone.
struct Seeds {
    std::vector<uint64_t> v;
    const uint64_t *ptr = nullptr;
    Seeds(PyObject *o, int32_t needed, bool optional = false)
    {
        if (optional && o == Py_None) return;
        PyObject *fast = PySequence_Fast(o, "proj_seeds must be a sequence of integers");
        if (!fast) throw BadArgument{};
        const Py_ssize_t n = PySequence_Fast_GET_SIZE(fast);
        v.resize(n);
        for (Py_ssize_t i = 0; i < n; ++i) {
            PyObject *num = PyNumber_Long(PySequence_Fast_GET_ITEM(fast, i));
            if (num) {
                v[i] = PyLong_AsUnsignedLongLongMask(num);
                Py_DECREF(num);
            }
            if (PyErr_Occurred()) {
                Py_DECREF(fast);
                throw BadArgument{};
            }
        }
        Py_DECREF(fast);
        if (n < needed) {
            PyErr_Format(PyExc_ValueError, "proj_seeds must have one seed per head (%d)", static_cast<int>(needed));
            throw BadArgument{};
        }
        ptr = v.data();
    }
};

race_stream_t stream_of(PyObject *o)
{
    if (o == Py_None) return reinterpret_cast<race_stream_t>(c10::hip::getCurrentHIPStream().stream());
    PyObject *raw = PyObject_HasAttrString(o, "cuda_stream") ? PyObject_GetAttrString(o, "cuda_stream") : (Py_INCREF(o), o);
    if (!raw) throw BadArgument{};
    PyObject *num = PyNumber_Long(raw);
    Py_DECREF(raw);
    if (!num) throw BadArgument{};
    void *p = PyLong_AsVoidPtr(num);
    Py_DECREF(num);
    if (PyErr_Occurred()) throw BadArgument{};
    return reinterpret_cast<race_stream_t>(p);
}

// Other Python threads run while the library works (the first call with new seeds expands W; a full queue makes a launch wait).
struct ReleaseGil {
    PyThreadState *saved = PyEval_SaveThread();
    ~ReleaseGil() { PyEval_RestoreThread(saved); }
};

template <int N, typename F>
PyObject *call(PyObject *const *args, Py_ssize_t nargs, F f)
{
    if (nargs != N) {
        PyErr_Format(PyExc_TypeError, "%d arguments expected, got %zd", N, nargs);
        return nullptr;
    }
    try {
        return PyLong_FromLong(f(args));
    } catch (const BadArgument &) {
        return nullptr;
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

// (desc, Q, K, V, seeds, O, den, workspace, stream); workspace None: the library's built-in scratch
PyObject *fwd(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return call<9>(args, n, [](PyObject *const *a) {
        const Desc d(a[0]);
        const Shape t = full(d);
        const at::ScalarType e = d.elem();
        void *Q = tensor(a[1], "Q", t, e), *K = tensor(a[2], "K", t, e), *V = tensor(a[3], "V", t, e);
        const Seeds s(a[4], d.heads());
        void *O = tensor(a[5], "O", t, e);
        float *den = static_cast<float *>(tensor(a[6], "den", per_token(d), at::kFloat));
        const race_stream_t st = stream_of(a[8]);
        const bool built_in = a[7] == Py_None;
        const Workspace ws(a[7]);
        const ReleaseGil released;
        if (built_in) return race_attn_fwd_static(&d.d, Q, K, V, s.ptr, O, den, st);
        return race_attn_fwd(&d.d, Q, K, V, s.ptr, O, den, ws.ptr, ws.bytes, st);
    });
}

// (desc, Q, K, V, O, den, dO, seeds, dQ, dK, dV, dbeta or None, workspace, stream, saved)
PyObject *bwd(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return call<15>(args, n, [](PyObject *const *a) {
        const Desc d(a[0]);
        const Shape t = full(d);
        const at::ScalarType e = d.elem();
        void *Q = tensor(a[1], "Q", t, e), *K = tensor(a[2], "K", t, e), *V = tensor(a[3], "V", t, e), *O = tensor(a[4], "O", t, e);
        const float *den = static_cast<float *>(tensor(a[5], "den", per_token(d), at::kFloat));
        void *dO = tensor(a[6], "dO", t, e);
        const Seeds s(a[7], d.heads());
        void *dQ = tensor(a[8], "dQ", t, e), *dK = tensor(a[9], "dK", t, e), *dV = tensor(a[10], "dV", t, e);
        float *dbeta = a[11] == Py_None ? nullptr : static_cast<float *>(tensor(a[11], "dbeta", per_head(d), at::kFloat));
        const Workspace ws(a[12]);
        const race_stream_t st = stream_of(a[13]);
        const auto entry = a[14] == Py_True ? race_attn_bwd_saved : race_attn_bwd_beta;
        const ReleaseGil released;
        return entry(&d.d, Q, K, V, O, den, dO, s.ptr, dQ, dK, dV, dbeta, ws.ptr, ws.bytes, st);
    });
}

// (desc, K or None, V or None, seeds, state, workspace or None, stream)
PyObject *state_init(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return call<7>(args, n, [](PyObject *const *a) {
        const Desc d(a[0]);
        float *state = static_cast<float *>(tensor(a[4], "state", state_shape(d), at::kFloat));
        void *K = nullptr, *V = nullptr;
        if (d.d.N > 0) {
            K = tensor(a[1], "K", full(d), d.elem());
            V = tensor(a[2], "V", full(d), d.elem());
        }
        const Seeds s(a[3], d.heads());
        const Workspace ws(a[5]);
        const race_stream_t st = stream_of(a[6]);
        const ReleaseGil released;
        return race_attn_state_init(&d.d, K, V, s.ptr, state, ws.ptr, ws.bytes, st);
    });
}

// (desc, q, k, v, seeds or None, state, o, den, workspace, stream)
PyObject *step(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return call<10>(args, n, [](PyObject *const *a) {
        const Desc d(a[0]);
        const Shape r = rows(d);
        const at::ScalarType e = d.elem();
        void *q = tensor(a[1], "q", r, e), *k = tensor(a[2], "k", r, e), *v = tensor(a[3], "v", r, e);
        const Seeds s(a[4], d.d.H, true);
        float *state = static_cast<float *>(tensor(a[5], "state", state_shape(d), at::kFloat));
        void *o = tensor(a[6], "o", r, e);
        float *den = static_cast<float *>(tensor(a[7], "den", per_head(d), at::kFloat));
        const Workspace ws(a[8]);
        const race_stream_t st = stream_of(a[9]);
        const ReleaseGil released;
        return race_attn_step(&d.d, q, k, v, s.ptr, state, o, den, ws.ptr, ws.bytes, st);
    });
}

#define ENTRY(name, doc) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(name)), METH_FASTCALL, doc}
PyMethodDef kMethods[] = {
    ENTRY(fwd, "race_attn_fwd, or race_attn_fwd_static without a workspace"),
    ENTRY(bwd, "race_attn_bwd_beta or race_attn_bwd_saved"),
    ENTRY(state_init, "race_attn_state_init"),
    ENTRY(step, "race_attn_step"),
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_native", "argument marshalling of the RACE Attention entry points", -1, kMethods,
                       nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() { return PyModule_Create(&kModule); }
