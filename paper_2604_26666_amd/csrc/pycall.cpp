// Argument marshalling of the Python binding's launching calls, in C: each function takes the arguments of the binding function of
// its name, positionally, and calls the library through the address that init() was given.  Where an argument is of a type that
// this file does not know (or out of its C type's range), the function returns None and the binding goes its general way through
// ctypes, which converts, or raises as it always did.  A 512 x 512 x 512 call from Python: 5.5 us to issue through
// ctypes, 3.9 this way, 3.2 of them in the plan and the HIP runtime (small calls are bound by this: their kernels take 3-4 us).
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <stdint.h>
#include <string.h>
#include <unistd.h>

#include "../../include/fact.h"

namespace {

PyObject *g_epilogue, *g_block;                             // the binding's classes
PyObject *g_is_initialized, *g_get_device, *g_raw_stream;   // torch's (nullptr: streams go the general way)
PyObject *n_data_ptr, *n_bias, *n_residual, *n_ldr, *n_stride_r, *n_act, *n_out_f32, *n_f16, *n_cuda_stream;
PyObject *n_dims, *n_norm_rms, *n_rope, *n_eps, *n_rope_base, *n_weights;
PyObject *n_block_ptrs[13];

decltype(&fact_gemm) p_gemm;
decltype(&fact_gemm_batched) p_gemm_batched;
decltype(&fact_gemm_splitk) p_gemm_splitk;
decltype(&fact_block_mlp) p_block_mlp, p_block_mlp_f16;
decltype(&fact_attention) p_attention;
decltype(&fact_block_forward) p_block_forward;

// Readers: false where the argument has to go the general way, which meets the same error again; false with a Python error set only
// for what is no error of the argument (an interrupt while an object's own code ran), and that ends the call.
void forget() { if (PyErr_Occurred() && PyErr_ExceptionMatches(PyExc_Exception)) PyErr_Clear(); }
PyObject *general() { if (PyErr_Occurred()) return nullptr; Py_RETURN_NONE; }

bool read(PyObject *o, int64_t *v)
{
    if (!PyLong_Check(o)) return false;
    int over = 0;
    *v = PyLong_AsLongLongAndOverflow(o, &over);
    return !over;
}
bool read(PyObject *o, int *v)
{
    int64_t w;
    if (!read(o, &w) || w < INT32_MIN || w > INT32_MAX) return false;
    *v = (int)w;
    return true;
}
bool read(PyObject *o, size_t *v)
{
    int64_t w;
    if (!read(o, &w) || w < 0) return false;
    *v = (size_t)w;
    return true;
}
bool read(PyObject *o, float *v)
{
    if (!PyFloat_CheckExact(o)) return false;
    *v = (float)PyFloat_AS_DOUBLE(o);
    return true;
}
bool address(PyObject *o, const void **v)                   // None, an address, or something with data_ptr()
{
    if (o == Py_None) { *v = nullptr; return true; }
    PyObject *r = nullptr;
    if (!PyLong_Check(o)) {
        r = o = PyObject_CallMethodNoArgs(o, n_data_ptr);
        if (!r) { forget(); return false; }
        if (!PyLong_CheckExact(r)) { Py_DECREF(r); return false; }
    }
    const unsigned long long w = PyLong_AsUnsignedLongLong(o);
    const bool ok = !(w == (unsigned long long)-1 && PyErr_Occurred());
    if (!ok) forget();
    *v = (const void *)(uintptr_t)w;
    Py_XDECREF(r);
    return ok;
}
bool read(PyObject *o, const void **v) { return address(o, v); }
bool read(PyObject *o, void **v) { return address(o, (const void **)v); }

// an attribute read by `reader`
template <class T> bool attr(PyObject *o, PyObject *name, T *v)
{
    PyObject *a = PyObject_GetAttr(o, name);
    if (!a) { forget(); return false; }
    const bool ok = read(a, v);
    Py_DECREF(a);
    return ok;
}

struct Epilogue { fact_epilogue e; const fact_epilogue *p; };
bool read(PyObject *o, Epilogue *v)
{
    if (o == Py_None) { v->p = nullptr; return true; }
    if ((PyObject *)Py_TYPE(o) != g_epilogue) return false;
    memset(&v->e, 0, sizeof v->e);
    int act, out_f32, f16;
    if (!attr(o, n_bias, &v->e.bias) || !attr(o, n_residual, &v->e.residual) || !attr(o, n_ldr, &v->e.ldr) || !attr(o, n_stride_r, &v->e.stride_r) ||
        !attr(o, n_act, &act) || !attr(o, n_out_f32, &out_f32) || !attr(o, n_f16, &f16)) return false;
    v->e.act = act; v->e.out_f32 = out_f32; v->e.f16 = f16;
    v->p = &v->e;
    return true;
}

struct Stream { void *s; };
bool read(PyObject *o, Stream *v)
{
    if (o != Py_None) {
        if (PyLong_Check(o)) return address(o, (const void **)&v->s);
        PyObject *a = PyObject_GetAttr(o, n_cuda_stream);
        if (!a) forget();
        const bool ok = a && PyLong_Check(a) && address(a, (const void **)&v->s);
        Py_XDECREF(a);
        return ok;
    }
    if (!g_raw_stream) return false;
    static pid_t ready = 0;                                 // process in which torch has been seen initialised (a forked child has not)
    const pid_t me = getpid();
    if (ready != me) {
        PyObject *r = PyObject_CallNoArgs(g_is_initialized);
        const bool ok = r == Py_True;
        if (!r) forget();
        Py_XDECREF(r);
        if (!ok) return false;
        ready = me;
    }
    PyObject *dev = PyObject_CallNoArgs(g_get_device), *r = dev ? PyObject_CallOneArg(g_raw_stream, dev) : nullptr;
    Py_XDECREF(dev);
    if (!r) { forget(); return false; }
    const bool ok = PyLong_Check(r) && address(r, (const void **)&v->s);
    Py_DECREF(r);
    return ok;
}

struct Strides { int64_t s[3]; };
bool read(PyObject *o, Strides *v)
{
    const bool tuple = PyTuple_CheckExact(o);
    if (!tuple && !PyList_CheckExact(o)) return false;
    if ((tuple ? PyTuple_GET_SIZE(o) : PyList_GET_SIZE(o)) != 3) return false;
    for (int i = 0; i < 3; ++i)
        if (!read(tuple ? PyTuple_GET_ITEM(o, i) : PyList_GET_ITEM(o, i), &v->s[i])) return false;
    return true;
}

struct Block { fact_block b; };
bool read(PyObject *o, Block *v)
{
    if ((PyObject *)Py_TYPE(o) != g_block) return false;
    fact_block &b = v->b;
    memset(&b, 0, sizeof b);
    PyObject *dims = PyObject_GetAttr(o, n_dims), *weights = dims ? PyObject_GetAttr(o, n_weights) : nullptr;
    int64_t *const to[7] = {&b.batch, &b.tokens, &b.d_model, &b.n_q_heads, &b.n_kv_heads, &b.head_dim, &b.d_ff};
    const void **const ptr[13] = {&b.norm1_g, &b.norm1_b, &b.Wqkv, &b.bqkv, &b.Wo, &b.bo, &b.norm2_g, &b.norm2_b, &b.W1, &b.W1u, &b.b1, &b.W2, &b.b2};
    int rms = 0, act = 0, rope = 0;
    bool ok = weights && PyTuple_CheckExact(dims) && PyTuple_GET_SIZE(dims) == 7 && PyDict_CheckExact(weights);
    for (int i = 0; ok && i < 7; ++i) ok = read(PyTuple_GET_ITEM(dims, i), to[i]);
    for (int i = 0; ok && i < 13; ++i) {
        PyObject *w = PyDict_GetItemWithError(weights, n_block_ptrs[i]);
        if (w) ok = address(w, ptr[i]);
    }
    ok = ok && attr(o, n_norm_rms, &rms) && attr(o, n_act, &act) && attr(o, n_rope, &rope) && attr(o, n_eps, &b.eps) && attr(o, n_rope_base, &b.rope_base);
    b.norm_rms = rms; b.act = act; b.rope = rope;
    forget();
    Py_XDECREF(dims); Py_XDECREF(weights);
    return ok;
}

// Reads args[i ..] into the rest of the list, one reader each.
bool read_all(PyObject *const *) { return true; }
template <class T, class... Rest> bool read_all(PyObject *const *args, T *v, Rest *...rest) { return read(*args, v) && read_all(args + 1, rest...); }

template <class... T> bool arguments(PyObject *const *args, Py_ssize_t n, T *...v) { return n == (Py_ssize_t)sizeof...(T) && read_all(args, v...); }

#define FACT_CALL(expr) int rc; Py_BEGIN_ALLOW_THREADS rc = (expr); Py_END_ALLOW_THREADS return PyLong_FromLong(rc)

PyObject *gemm(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    int64_t M, N, K, lda, ldb, ldc; const void *A, *B; void *C; int tb; Epilogue ep; Stream s;
    if (!p_gemm || !arguments(args, n, &M, &N, &K, &A, &lda, &B, &ldb, &tb, &C, &ldc, &ep, &s)) return general();
    FACT_CALL(p_gemm(M, N, K, A, lda, B, ldb, tb, C, ldc, ep.p, s.s));
}

PyObject *gemm_batched(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    int64_t b, M, N, K, lda, ldb, ldc, sa, sb, sc; const void *A, *B; void *C; int tb; Epilogue ep; Stream s;
    if (!p_gemm_batched || !arguments(args, n, &b, &M, &N, &K, &A, &lda, &sa, &B, &ldb, &sb, &tb, &C, &ldc, &sc, &ep, &s)) return general();
    FACT_CALL(p_gemm_batched(b, M, N, K, A, lda, sa, B, ldb, sb, tb, C, ldc, sc, ep.p, s.s));
}

PyObject *gemm_splitk(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    int64_t M, N, K, lda, ldb, ldc; const void *A, *B; void *C, *ws; int tb, split; size_t bytes; Epilogue ep; Stream s;
    if (!p_gemm_splitk || !arguments(args, n, &M, &N, &K, &A, &lda, &B, &ldb, &tb, &C, &ldc, &ep, &split, &ws, &bytes, &s)) return general();
    FACT_CALL(p_gemm_splitk(M, N, K, A, lda, B, ldb, tb, C, ldc, ep.p, split, ws, bytes, s.s));
}

PyObject *mlp(decltype(&fact_block_mlp) call, PyObject *const *args, Py_ssize_t n)
{
    int64_t T, d, dff; const void *X, *W1, *W1u, *b1, *W2, *b2, *R; void *H, *Y, *ws; int act; size_t bytes; Stream s;
    if (!call || !arguments(args, n, &T, &d, &dff, &X, &W1, &W1u, &b1, &act, &W2, &b2, &R, &H, &Y, &ws, &bytes, &s)) return general();
    FACT_CALL(call(T, d, dff, X, W1, W1u, b1, act, W2, b2, R, H, Y, ws, bytes, s.s));
}
PyObject *block_mlp(PyObject *, PyObject *const *args, Py_ssize_t n) { return mlp(p_block_mlp, args, n); }
PyObject *block_mlp_f16(PyObject *, PyObject *const *args, Py_ssize_t n) { return mlp(p_block_mlp_f16, args, n); }

PyObject *attention(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    int64_t b, T, hq, hkv, D; const void *Q, *K, *V; void *O; Strides qs, ks, vs, os; int causal; float scale; Stream s;
    if (!p_attention || !arguments(args, n, &b, &T, &hq, &hkv, &D, &Q, &qs, &K, &ks, &V, &vs, &O, &os, &causal, &scale, &s)) return general();
    FACT_CALL(p_attention(b, T, hq, hkv, D, Q, qs.s, K, ks.s, V, vs.s, O, os.s, causal, scale, s.s));
}

PyObject *block_forward(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    Block blk; const void *X; void *Y, *scratch; size_t bytes; Stream s;
    if (!p_block_forward || !arguments(args, n, &blk, &X, &Y, &scratch, &bytes, &s)) return general();
    FACT_CALL(p_block_forward(&blk.b, X, Y, scratch, bytes, s.s));
}

// init({function name: address}, Epilogue, Block, (is_initialized, get_device, raw_stream) or None)
PyObject *init(PyObject *, PyObject *args)
{
    PyObject *table, *ep, *blk, *torch3;
    if (!PyArg_ParseTuple(args, "O!OOO", &PyDict_Type, &table, &ep, &blk, &torch3)) return nullptr;
    struct { const char *name; void **to; } const rows[] = {
        {"fact_gemm", (void **)&p_gemm}, {"fact_gemm_batched", (void **)&p_gemm_batched}, {"fact_gemm_splitk", (void **)&p_gemm_splitk},
        {"fact_block_mlp", (void **)&p_block_mlp}, {"fact_block_mlp_f16", (void **)&p_block_mlp_f16}, {"fact_attention", (void **)&p_attention},
        {"fact_block_forward", (void **)&p_block_forward}};
    for (const auto &r : rows) {
        PyObject *a = PyDict_GetItemString(table, r.name);
        void *p = a ? PyLong_AsVoidPtr(a) : nullptr;
        if (!p) { if (!PyErr_Occurred()) PyErr_Format(PyExc_KeyError, "%s", r.name); return nullptr; }
        *r.to = p;
    }
    Py_INCREF(ep); Py_INCREF(blk);
    g_epilogue = ep; g_block = blk;
    if (torch3 != Py_None) {
        PyObject *a, *b, *c;
        if (!PyArg_ParseTuple(torch3, "OOO", &a, &b, &c)) return nullptr;
        Py_INCREF(a); Py_INCREF(b); Py_INCREF(c);
        g_is_initialized = a; g_get_device = b; g_raw_stream = c;
    }
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"init", init, METH_VARARGS, nullptr},
#define FACT_METHOD(f) {#f, (PyCFunction)(void (*)(void))f, METH_FASTCALL, nullptr}
    FACT_METHOD(gemm), FACT_METHOD(gemm_batched), FACT_METHOD(gemm_splitk), FACT_METHOD(block_mlp), FACT_METHOD(block_mlp_f16),
    FACT_METHOD(attention), FACT_METHOD(block_forward),
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pycall", "argument marshalling of the launching calls", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pycall(void)
{
    struct { PyObject **to; const char *text; } const names[] = {
        {&n_data_ptr, "data_ptr"}, {&n_bias, "bias"}, {&n_residual, "residual"}, {&n_ldr, "ldr"}, {&n_stride_r, "stride_r"}, {&n_act, "act"},
        {&n_out_f32, "out_f32"}, {&n_f16, "f16"}, {&n_cuda_stream, "cuda_stream"}, {&n_dims, "dims"}, {&n_norm_rms, "norm_rms"},
        {&n_rope, "rope"}, {&n_eps, "eps"}, {&n_rope_base, "rope_base"}, {&n_weights, "weights"}};
    for (const auto &s : names)
        if (!(*s.to = PyUnicode_InternFromString(s.text))) return nullptr;
    const char *const ptrs[13] = {"norm1_g", "norm1_b", "Wqkv", "bqkv", "Wo", "bo", "norm2_g", "norm2_b", "W1", "W1u", "b1", "W2", "b2"};
    for (int i = 0; i < 13; ++i)
        if (!(n_block_ptrs[i] = PyUnicode_InternFromString(ptrs[i]))) return nullptr;
    return PyModule_Create(&module);
}
