// The calls of the C interface that a decoding loop makes, for Python: torch tensors in, status checked, on the current
// stream.  Through ctypes a call spent 6 to 9 us here (a Stream object, a pointer object and three attribute look-ups per
// tensor), about what its kernels take at small sizes; here it is under one, of the 3 to 4 us that a call of one or two
// launches takes on the host.  What is checked, and what is raised, is what binding.py does for the other calls.
#include <torch/csrc/autograd/python_variable.h>
#include <c10/hip/HIPStream.h>

#include "bastion_tv.h"

namespace {

PyObject *g_error;                                      // BtvError

struct Raised {};                                       // a Python exception is set

[[noreturn]] void raise(PyObject *type, const char *text)
{
    PyErr_SetString(type, text);
    throw Raised();
}

[[noreturn]] void raise_btv(int rc, const char *text)
{
    PyObject *e = PyObject_CallFunction(g_error, "is", rc, text);
    if (e) {
        PyErr_SetObject(g_error, e);
        Py_DECREF(e);
    }
    throw Raised();
}

void require(bool ok, const char *text)
{
    if (!ok) raise(PyExc_AssertionError, text);
}

// The arguments of one call, in order.
struct Args {
    PyObject *const *a;
    Py_ssize_t n, at = 0;

    PyObject *next()
    {
        if (at >= n) raise(PyExc_TypeError, "too few arguments");
        return a[at++];
    }
    const at::Tensor &tensor()
    {
        PyObject *o = next();
        if (!THPVariable_Check(o)) raise(PyExc_TypeError, "expected a torch tensor");
        return THPVariable_Unpack(o);
    }
    const at::Tensor *tensor_or_none()
    {
        if (at < n && a[at] == Py_None) { ++at; return nullptr; }
        return &tensor();
    }
    long long integer()
    {
        const long long v = PyLong_AsLongLong(next());
        if (v == -1 && PyErr_Occurred()) throw Raised();
        return v;
    }
    int int32() { return narrow(integer()); }
    int converted_int32()                               // what int(x) makes of the argument
    {
        PyObject *o = PyNumber_Long(next());
        if (!o) throw Raised();
        const long long v = PyLong_AsLongLong(o);
        Py_DECREF(o);
        if (v == -1 && PyErr_Occurred()) throw Raised();
        return narrow(v);
    }
    static int narrow(long long v)
    {
        if (v != (int)v) raise(PyExc_OverflowError, "integer argument out of range");
        return (int)v;
    }
    double real()
    {
        const double v = PyFloat_AsDouble(next());
        if (v == -1.0 && PyErr_Occurred()) throw Raised();
        return v;
    }
};

template <typename T = void>
T *pointer(const at::Tensor &t)
{
    require(t.is_cuda() && t.is_contiguous(), "device tensors must be contiguous CUDA tensors");
    return static_cast<T *>(t.data_ptr());
}
template <typename T = void>
T *pointer(const at::Tensor *t) { return t ? pointer<T>(*t) : nullptr; }

template <typename T = void>
T *next_pointer(Args &a) { return pointer<T>(a.tensor_or_none()); }

int size(const at::Tensor &t, int dim) { return (int)t.size(dim); }

void dims(const at::Tensor &t, int n)
{
    if (t.dim() != n) raise(PyExc_ValueError, "a tensor has the wrong number of dimensions");
}

int dtype_code(const at::Tensor &t)
{
    if (t.scalar_type() == at::kFloat) return BTV_F32;
    if (t.scalar_type() == at::kBFloat16) return BTV_BF16;
    raise_btv(BTV_EINVAL, "unsupported dtype");
}

struct Workspace { void *ptr; size_t bytes; };
Workspace next_workspace(Args &a)
{
    const at::Tensor *t = a.tensor_or_none();
    return { pointer(t), t ? (size_t)t->numel() : 0 };
}

void *stream() { return c10::hip::getCurrentHIPStream().stream(); }

template <typename F>
PyObject *call(PyObject *const *args, Py_ssize_t n, F f)
{
    try {
        Args a{ args, n };
        int rc = BTV_OK;
        // f reads the arguments and returns the launch itself, which runs without the interpreter's lock
        auto launch = f(a);
        if (a.at != n) raise(PyExc_TypeError, "too many arguments");
        void *st = stream();
        Py_BEGIN_ALLOW_THREADS
        rc = launch(st);
        Py_END_ALLOW_THREADS
        if (rc != BTV_OK) raise_btv(rc, btv_last_error());
        Py_RETURN_NONE;
    } catch (const Raised &) {
        return nullptr;
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

#define FACE(name) PyObject *name(PyObject *, PyObject *const *args, Py_ssize_t n)

FACE(tree_build)
{
    return call(args, n, [](Args &a) {
        const at::Tensor &m = a.tensor();
        dims(m, 2);
        require(m.scalar_type() == at::kFloat, "marginals must be float32");
        const float *marg = pointer<float>(m);
        const int B = size(m, 0), V = size(m, 1), N = a.int32();
        auto *parent = next_pointer<int32_t>(a), *token = next_pointer<int32_t>(a), *depth = next_pointer<int32_t>(a);
        auto *rho = next_pointer<float>(a);
        auto *n_out = next_pointer<int32_t>(a);
        auto *ahat = next_pointer<float>(a);
        const Workspace ws = next_workspace(a);
        return [=](void *st) { return btv_tree_build(marg, B, V, N, parent, token, depth, rho, n_out, ahat, ws.ptr, ws.bytes, st); };
    });
}

FACE(tree_build_adaptive)
{
    return call(args, n, [](Args &a) {
        const at::Tensor &m = a.tensor();
        dims(m, 2);
        const int N = a.int32();
        const at::Tensor &c = a.tensor();
        require(m.scalar_type() == at::kFloat && c.scalar_type() == at::kDouble && c.numel() >= N, "marginals must be float32, cost N_max float64");
        const float *marg = pointer<float>(m);
        const double *cost = pointer<double>(c);
        const int B = size(m, 0), V = size(m, 1);
        const double L_AR = a.real();
        auto *parent = next_pointer<int32_t>(a), *token = next_pointer<int32_t>(a), *depth = next_pointer<int32_t>(a);
        auto *rho = next_pointer<float>(a);
        auto *n_out = next_pointer<int32_t>(a);
        auto *ahat = next_pointer<float>(a);
        auto *s_best = next_pointer<double>(a);
        const Workspace ws = next_workspace(a);
        return [=](void *st) {
            return btv_tree_build_adaptive(marg, B, V, N, cost, L_AR, parent, token, depth, rho, n_out, ahat, s_best, ws.ptr, ws.bytes, st);
        };
    });
}

FACE(tree_build_batch)
{
    return call(args, n, [](Args &a) {
        const at::Tensor &m = a.tensor();
        dims(m, 3);
        const float *marg = pointer<float>(m);
        const int batch = size(m, 0), B = size(m, 1), V = size(m, 2);
        const int32_t *n_nodes = next_pointer<int32_t>(a), *q_offset = next_pointer<int32_t>(a);
        const int N = a.converted_int32();
        auto *parent = next_pointer<int32_t>(a), *token = next_pointer<int32_t>(a), *depth = next_pointer<int32_t>(a);
        auto *rho = next_pointer<float>(a);
        auto *n_out = next_pointer<int32_t>(a);
        auto *ahat = next_pointer<float>(a);
        const Workspace ws = next_workspace(a);
        return [=](void *st) {
            return btv_tree_build_batch(marg, batch, B, V, n_nodes, q_offset, N, parent, token, depth, rho, n_out, ahat, ws.ptr, ws.bytes, st);
        };
    });
}

FACE(tree_verify_attn)
{
    return call(args, n, [](Args &a) {
        const at::Tensor &q = a.tensor(), &k = a.tensor(), &v = a.tensor();
        const int32_t *parent = next_pointer<int32_t>(a);
        const int L = a.int32();
        const at::Tensor &o = a.tensor();
        const Workspace ws = next_workspace(a);
        const float scale = (float)a.real();
        dims(q, 3);
        const int M = size(q, 0), Hq = size(q, 1), D = size(q, 2), Hkv = size(k, 1), dtype = dtype_code(q);
        require(k.size(0) >= (int64_t)L + M && v.sizes() == k.sizes() && o.sizes() == q.sizes(), "shapes of Q, K, V and O do not match");
        const void *Q = pointer(q), *K = pointer(k), *V = pointer(v);
        void *O = pointer(o);
        return [=](void *st) { return btv_tree_verify_attn(Q, K, V, parent, M, L, Hq, Hkv, D, dtype, scale, O, ws.ptr, ws.bytes, st); };
    });
}

FACE(tree_verify_attn_fp8kv)
{
    return call(args, n, [](Args &a) {
        const at::Tensor &q = a.tensor(), &k = a.tensor(), &v = a.tensor();
        const float k_scale = (float)a.real(), v_scale = (float)a.real();
        const int32_t *parent = next_pointer<int32_t>(a);
        const int L = a.int32();
        const at::Tensor &o = a.tensor();
        const Workspace ws = next_workspace(a);
        const float scale = (float)a.real();
        dims(q, 3);
        const int M = size(q, 0), Hq = size(q, 1), D = size(q, 2), Hkv = size(k, 1);
        require(k.size(0) >= (int64_t)L + M && v.sizes() == k.sizes() && o.sizes() == q.sizes(), "shapes of Q, K, V and O do not match");
        require(q.scalar_type() == at::kBFloat16 && k.element_size() == 1 && v.element_size() == 1, "Q must be bfloat16, K and V one byte");
        const void *Q = pointer(q), *K = pointer(k), *V = pointer(v);
        void *O = pointer(o);
        return [=](void *st) {
            return btv_tree_verify_attn_fp8kv(Q, K, V, k_scale, v_scale, parent, M, L, Hq, Hkv, D, scale, O, ws.ptr, ws.bytes, st);
        };
    });
}

PyObject *verify_attn_paged(PyObject *const *args, Py_ssize_t n, bool fp8)
{
    return call(args, n, [fp8](Args &a) {
        const at::Tensor &q = a.tensor(), &k = a.tensor(), &v = a.tensor();
        const float k_scale = fp8 ? (float)a.real() : 1.f, v_scale = fp8 ? (float)a.real() : 1.f;
        const at::Tensor &bt = a.tensor();
        const int32_t *q_offset = next_pointer<int32_t>(a), *prefix_len = next_pointer<int32_t>(a), *parent = next_pointer<int32_t>(a);
        const int M_max = a.int32(), L_max = a.int32();
        void *O = next_pointer(a);
        const Workspace ws = next_workspace(a);
        const float scale = (float)a.real();
        dims(q, 3); dims(k, 4); dims(bt, 2);
        const int total_M = size(q, 0), Hq = size(q, 1), D = size(q, 2), blocks = size(k, 0), Hkv = size(k, 2);
        const int batch = size(bt, 0), max_blocks = size(bt, 1);
        require(k.size(1) == BTV_PAGE && q.scalar_type() == at::kBFloat16, "pages of BTV_PAGE tokens, Q bfloat16");
        if (fp8) require(k.element_size() == 1 && v.element_size() == 1, "K and V must be one byte");
        const void *Q = pointer(q), *K = pointer(k), *V = pointer(v);
        const int32_t *table = pointer<int32_t>(bt);
        return [=](void *st) {
            return fp8 ? btv_tree_verify_attn_paged_fp8kv(Q, K, V, k_scale, v_scale, blocks, table, max_blocks, q_offset, prefix_len, parent,
                                                          batch, total_M, M_max, L_max, Hq, Hkv, D, scale, O, ws.ptr, ws.bytes, st)
                       : btv_tree_verify_attn_paged(Q, K, V, blocks, table, max_blocks, q_offset, prefix_len, parent, batch, total_M, M_max,
                                                    L_max, Hq, Hkv, D, scale, O, ws.ptr, ws.bytes, st);
        };
    });
}
FACE(tree_verify_attn_paged) { return verify_attn_paged(args, n, false); }
FACE(tree_verify_attn_paged_fp8kv) { return verify_attn_paged(args, n, true); }

FACE(tree_accept_greedy)
{
    return call(args, n, [](Args &a) {
        const at::Tensor &l = a.tensor();
        dims(l, 2);
        const void *logits = pointer(l);
        const int dtype = dtype_code(l), M = size(l, 0) - 1, V = size(l, 1);
        const int32_t *parent = next_pointer<int32_t>(a), *token = next_pointer<int32_t>(a);
        auto *path = next_pointer<int32_t>(a), *n_acc = next_pointer<int32_t>(a), *bonus = next_pointer<int32_t>(a);
        auto *argmax_out = next_pointer<int32_t>(a);
        const Workspace ws = next_workspace(a);
        return [=](void *st) {
            return btv_tree_accept_greedy(logits, dtype, parent, token, M, V, path, n_acc, bonus, argmax_out, ws.ptr, ws.bytes, st);
        };
    });
}

FACE(tree_accept_greedy_batch)
{
    return call(args, n, [](Args &a) {
        const at::Tensor &l = a.tensor();
        dims(l, 2);
        const void *logits = pointer(l);
        const int dtype = dtype_code(l), V = size(l, 1);
        const int32_t *parent = next_pointer<int32_t>(a), *token = next_pointer<int32_t>(a);
        const at::Tensor &qo = a.tensor();
        const int32_t *q_offset = pointer<int32_t>(qo);
        const int batch = (int)qo.numel() - 1, total_M = size(l, 0) - batch, M_max = a.converted_int32();
        auto *path = next_pointer<int32_t>(a), *n_acc = next_pointer<int32_t>(a), *bonus = next_pointer<int32_t>(a);
        auto *argmax_out = next_pointer<int32_t>(a);
        const Workspace ws = next_workspace(a);
        return [=](void *st) {
            return btv_tree_accept_greedy_batch(logits, dtype, parent, token, q_offset, batch, total_M, M_max, V, path, n_acc, bonus, argmax_out,
                                                ws.ptr, ws.bytes, st);
        };
    });
}

FACE(tree_accept_greedy_lm_head)
{
    return call(args, n, [](Args &a) {
        const at::Tensor &x = a.tensor(), &w = a.tensor();
        dims(x, 2);
        const int M = size(x, 0) - 1, h = size(x, 1), V = size(w, 0);
        require(w.size(1) == h && dtype_code(x) == BTV_BF16 && dtype_code(w) == BTV_BF16, "hidden [rows, h] and W [V, h] must be bfloat16");
        const void *X = pointer(x), *W = pointer(w);
        const int32_t *parent = next_pointer<int32_t>(a), *token = next_pointer<int32_t>(a);
        auto *path = next_pointer<int32_t>(a), *n_acc = next_pointer<int32_t>(a), *bonus = next_pointer<int32_t>(a);
        auto *argmax_out = next_pointer<int32_t>(a);
        const Workspace ws = next_workspace(a);
        return [=](void *st) {
            return btv_tree_accept_greedy_lm_head(X, W, h, parent, token, M, V, path, n_acc, bonus, argmax_out, ws.ptr, ws.bytes, st);
        };
    });
}

FACE(tree_accept_stochastic)
{
    return call(args, n, [](Args &a) {
        const at::Tensor &l = a.tensor(), &m = a.tensor();
        dims(l, 2);
        const int M = size(l, 0) - 1, V = size(l, 1), B = size(m, 0), dtype = dtype_code(l);
        const void *logits = pointer(l);
        const float *marg = pointer<float>(m);
        const int32_t *parent = next_pointer<int32_t>(a), *token = next_pointer<int32_t>(a);
        const at::Tensor &u = a.tensor();
        require(m.size(1) == V && u.numel() >= l.size(0), "marginals [B, V] and a uniform per row");
        const float *uniforms = pointer<float>(u);
        auto *path = next_pointer<int32_t>(a), *n_acc = next_pointer<int32_t>(a), *bonus = next_pointer<int32_t>(a);
        const Workspace ws = next_workspace(a);
        return [=](void *st) {
            return btv_tree_accept_stochastic(logits, dtype, marg, B, parent, token, M, V, uniforms, path, n_acc, bonus, ws.ptr, ws.bytes, st);
        };
    });
}

int row_bytes(const at::Tensor &t, int first)           // bytes of what lies below the first dimensions
{
    int64_t e = t.element_size();
    for (int d = first; d < t.dim(); ++d) e *= t.size(d);
    return (int)e;
}

FACE(kv_commit)
{
    return call(args, n, [](Args &a) {
        const at::Tensor &k = a.tensor(), &v = a.tensor();
        require(k.sizes() == v.sizes() && k.is_contiguous() && v.is_contiguous() && k.dim() >= 3, "K and V must be contiguous, [layers, rows, ...]");
        void *K = pointer(k), *V = pointer(v);
        const int layers = size(k, 0), bytes = row_bytes(k, 2), L = a.int32(), M = a.int32();
        const long long stride = k.stride(0) * k.element_size();
        const int32_t *path = next_pointer<int32_t>(a), *n_acc = next_pointer<int32_t>(a);
        auto *new_len = next_pointer<int32_t>(a);
        return [=](void *st) { return btv_kv_commit(K, V, layers, stride, L, M, bytes, path, n_acc, new_len, st); };
    });
}

FACE(kv_commit_paged)
{
    return call(args, n, [](Args &a) {
        const at::Tensor &k = a.tensor(), &v = a.tensor();
        require(k.sizes() == v.sizes() && k.is_contiguous() && v.is_contiguous() && k.dim() >= 4, "the pools must be contiguous, [layers, blocks, page, ...]");
        void *K = pointer(k), *V = pointer(v);
        const at::Tensor &bt = a.tensor();
        dims(bt, 2);
        const int32_t *table = pointer<int32_t>(bt), *prefix_len = next_pointer<int32_t>(a);
        const at::Tensor &p = a.tensor();
        const int32_t *path = pointer<int32_t>(p), *n_acc = next_pointer<int32_t>(a);
        auto *new_len = next_pointer<int32_t>(a);
        void *ws = next_pointer(a);
        const int32_t *q_offset = next_pointer<int32_t>(a);
        int M_max = 0, total_M = 0;
        if (q_offset) {
            M_max = a.converted_int32();
            total_M = (int)p.numel();
            require(M_max >= 1, "M_max must be given with q_offset");
        } else {
            a.next();
            M_max = size(p, 1);
        }
        const int layers = size(k, 0), blocks = size(k, 1), bytes = row_bytes(k, 3), batch = size(bt, 0), max_blocks = size(bt, 1);
        const long long stride = k.stride(0) * k.element_size();
        return [=](void *st) {
            return btv_kv_commit_paged(K, V, layers, stride, blocks, table, max_blocks, prefix_len, path, q_offset, total_M, n_acc, batch, M_max, bytes,
                                       new_len, ws, st);
        };
    });
}

PyObject *set_error(PyObject *, PyObject *type)
{
    Py_INCREF(type);
    Py_XSETREF(g_error, type);
    Py_RETURN_NONE;
}

#define ENTRY(name) { #name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr }
PyMethodDef methods[] = {
    ENTRY(tree_build), ENTRY(tree_build_adaptive), ENTRY(tree_build_batch), ENTRY(tree_verify_attn), ENTRY(tree_verify_attn_fp8kv),
    ENTRY(tree_verify_attn_paged), ENTRY(tree_verify_attn_paged_fp8kv), ENTRY(tree_accept_greedy), ENTRY(tree_accept_greedy_batch),
    ENTRY(tree_accept_greedy_lm_head), ENTRY(tree_accept_stochastic), ENTRY(kv_commit), ENTRY(kv_commit_paged),
    { "set_error", set_error, METH_O, nullptr }, { nullptr, nullptr, 0, nullptr },
};
PyModuleDef module = { PyModuleDef_HEAD_INIT, "_face", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr };

}  // namespace

PyMODINIT_FUNC PyInit__face() { return PyModule_Create(&module); }
