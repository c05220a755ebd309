// Argument marshalling of the per-step calls in native code (module paper_2511_21862_amd._binding).
//
// A step of a small batch is bound by the host: of the 7.8 us of ooco_plan + ooco_attn_mixed on five short sequences 2.9 us
// are the launch, 0.5 us the plan and the rest was Python -- 1.2 us for the contiguity and the address of eight tensors,
// 1.0 us for three numpy arrays, 0.3 us for the current stream, the rest ctypes' own conversions.  Here those are loads of a
// few fields.  Measured on MI355X in a loop of calls: 7.8 -> 5.0 us, where the kernel itself is the limit; KV append of four rows
// 5.7 -> 3.8; a copy of twelve blocks 5.3 -> 3.5.
//
// Every function takes only the plain form of its arguments (exact torch.Tensor on the GPU and contiguous, exact int32
// C-contiguous numpy.ndarray, exact int, a c_void_p handle) and returns the call's status; for anything else -- None, an
// address, a list, another dtype, a subclass, a tensor that is not contiguous, an active torch function mode -- it calls
// nothing and returns NotImplemented, and binding.py goes its general way, which accepts or refuses it.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#define NPY_NO_DEPRECATED_API NPY_1_7_API_VERSION
#include <numpy/arrayobject.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <climits>

#include "ooco.h"

namespace {

decltype(&ooco_plan) f_plan;
decltype(&ooco_attn_mixed) f_attn;
decltype(&ooco_attn_mixed_static) f_static;
decltype(&ooco_kv_append) f_append;
decltype(&ooco_kv_block_copy) f_copy;
PyTypeObject *handle_type;   // ctypes.c_void_p
PyObject *of_tensor;         // OF_TENSOR, which stands for a size: the length of the tensor's first dimension

// The plain forms; false = not one of them (no Python error is set).
bool get_tensor(PyObject *o, const at::Tensor *&t)
{
    if (!THPVariable_CheckExact(o)) return false;
    t = &THPVariable_Unpack(o);
    return t->defined() && t->is_cuda() && t->layout() == at::kStrided && t->has_storage() && t->is_contiguous();
}
template <class T>
bool get_ptr(PyObject *o, T *&p)
{
    const at::Tensor *t;
    if (!get_tensor(o, t)) return false;
    p = static_cast<T *>(t->data_ptr());
    return true;
}
bool get_int(PyObject *o, int &v)
{
    if (!PyLong_CheckExact(o)) return false;
    int over = 0;
    const long x = PyLong_AsLongAndOverflow(o, &over);
    v = (int)x;
    return !over && x >= INT_MIN && x <= INT_MAX;
}
bool get_size(PyObject *o, PyObject *tensor, int &v)
{
    if (o != of_tensor) return get_int(o, v);
    const at::Tensor *t;
    if (!get_tensor(tensor, t) || t->dim() < 1 || t->size(0) > INT_MAX) return false;
    v = (int)t->size(0);
    return true;
}
bool get_i32(PyObject *o, const int32_t *&p)
{
    if (!PyArray_CheckExact(o)) return false;
    PyArrayObject *const a = reinterpret_cast<PyArrayObject *>(o);
    if (PyArray_TYPE(a) != NPY_INT32 || !PyArray_ISCARRAY_RO(a)) return false;
    p = static_cast<const int32_t *>(PyArray_DATA(a));
    return true;
}
bool get_handle(PyObject *o, ooco_ctx *&h)
{
    if (Py_TYPE(o) != handle_type) return false;
    Py_buffer b;   // (a ctypes object exports its own storage: the pointer)
    if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) {
        PyErr_Clear();
        return false;
    }
    const bool ok = b.len == (Py_ssize_t)sizeof h;
    if (ok) memcpy(&h, b.buf, sizeof h);
    PyBuffer_Release(&b);
    return ok;
}
// None: the current stream of the current device (a tensor on the GPU is in hand, so there is one); an int: its handle.
bool get_stream(PyObject *o, void *&s)
{
    if (o == Py_None) {
        s = reinterpret_cast<void *>(c10::hip::getCurrentHIPStream().stream());
        return true;
    }
    if (!PyLong_CheckExact(o)) return false;
    s = PyLong_AsVoidPtr(o);
    if (!PyErr_Occurred()) return true;
    PyErr_Clear();
    return false;
}
bool plain() { return !at::impl::torch_function_mode_enabled(); }

PyObject *not_plain() { return Py_NewRef(Py_NotImplemented); }

// The call itself, other Python threads running meanwhile as during a ctypes call.  (The library's functions have C linkage
// and report by status: nothing may be thrown out of them.)
template <class F>
int call(F f) noexcept
{
    PyThreadState *const t = PyEval_SaveThread();
    const int st = f();
    PyEval_RestoreThread(t);
    return st;
}

// C++ exceptions of torch's accessors end here: what could not be read in the plain way is left to the general one.
template <class F>
PyObject *guarded(F f) noexcept
{
    try {
        return f();
    } catch (...) {
        return not_plain();
    }
}

PyObject *py_plan(PyObject *, PyObject *const *a, Py_ssize_t n) noexcept
{
    return guarded([&]() -> PyObject * {
        ooco_ctx *ctx;
        int num_seqs;
        const int32_t *seq, *qsl, *cl;
        if (n != 5 || !get_handle(a[0], ctx) || !get_int(a[1], num_seqs) || !get_i32(a[2], seq) || !get_i32(a[3], qsl) || !get_i32(a[4], cl))
            return not_plain();
        const int st = call([&]() { return f_plan(ctx, num_seqs, seq, qsl, cl); });
        return PyLong_FromLong(st);
    });
}

// (ctx, q, k_cache, v_cache, block_tables, seq_lens, query_start_loc, ctx_lens, out, num_seqs, total_q, stream)
PyObject *py_attn(PyObject *, PyObject *const *a, Py_ssize_t n) noexcept
{
    return guarded([&]() -> PyObject * {
        ooco_ctx *ctx;
        void *q, *k, *v, *out, *stream;
        int32_t *bt, *sl, *qsl, *cl;
        int num_seqs, total_q;
        if (n != 12 || !plain() || !get_handle(a[0], ctx) || !get_ptr(a[1], q) || !get_ptr(a[2], k) || !get_ptr(a[3], v) || !get_ptr(a[4], bt) ||
            !get_ptr(a[5], sl) || !get_ptr(a[6], qsl) || !get_ptr(a[7], cl) || !get_ptr(a[8], out) || !get_size(a[9], a[5], num_seqs) ||
            !get_size(a[10], a[1], total_q) || !get_stream(a[11], stream))
            return not_plain();
        const int st = call([&]() { return f_attn(ctx, q, k, v, bt, sl, qsl, cl, out, num_seqs, total_q, stream); });
        return PyLong_FromLong(st);
    });
}

// (num_q_heads, num_kv_heads, head_dim, block_size, max_blocks_per_seq, softmax_scale, h_seq_lens, h_query_start_loc,
// h_ctx_lens, q, k_cache, v_cache, block_tables, seq_lens, query_start_loc, ctx_lens, out, num_seqs, total_q, stream);
// returns the status, or the text of the error with it.
PyObject *py_static(PyObject *, PyObject *const *a, Py_ssize_t n) noexcept
{
    return guarded([&]() -> PyObject * {
        int hq, hkv, hd, bs, mb, num_seqs, total_q;
        const int32_t *hsl, *hqsl, *hcl;
        void *q, *k, *v, *out, *stream;
        int32_t *bt, *sl, *qsl, *cl;
        if (n != 20 || !plain() || !get_int(a[0], hq) || !get_int(a[1], hkv) || !get_int(a[2], hd) || !get_int(a[3], bs) || !get_int(a[4], mb) ||
            !PyFloat_CheckExact(a[5]) || !get_i32(a[6], hsl) || !get_i32(a[7], hqsl) || !get_i32(a[8], hcl) || !get_ptr(a[9], q) ||
            !get_ptr(a[10], k) || !get_ptr(a[11], v) || !get_ptr(a[12], bt) || !get_ptr(a[13], sl) || !get_ptr(a[14], qsl) ||
            !get_ptr(a[15], cl) || !get_ptr(a[16], out) || !get_int(a[17], num_seqs) || !get_int(a[18], total_q) || !get_stream(a[19], stream))
            return not_plain();
        const float scale = (float)PyFloat_AS_DOUBLE(a[5]);
        char msg[512] = "";
        const int st = call([&]() { return f_static(hq, hkv, hd, bs, mb, scale, hsl, hqsl, hcl, q, k, v, bt, sl, qsl, cl, out, num_seqs, total_q, stream, msg, sizeof msg); });
        if (st == 0) return PyLong_FromLong(0);
        return Py_BuildValue("(is)", st, msg);
    });
}

// (ctx, k_new, v_new, k_cache, v_cache, block_tables, query_start_loc, ctx_lens, num_seqs, total_q, stream)
PyObject *py_append(PyObject *, PyObject *const *a, Py_ssize_t n) noexcept
{
    return guarded([&]() -> PyObject * {
        ooco_ctx *ctx;
        void *kn, *vn, *k, *v, *stream;
        int32_t *bt, *qsl, *cl;
        int num_seqs, total_q;
        if (n != 11 || !plain() || !get_handle(a[0], ctx) || !get_ptr(a[1], kn) || !get_ptr(a[2], vn) || !get_ptr(a[3], k) || !get_ptr(a[4], v) ||
            !get_ptr(a[5], bt) || !get_ptr(a[6], qsl) || !get_ptr(a[7], cl) || !get_size(a[8], a[7], num_seqs) || !get_size(a[9], a[1], total_q) ||
            !get_stream(a[10], stream))
            return not_plain();
        const int st = call([&]() { return f_append(ctx, kn, vn, k, v, bt, qsl, cl, num_seqs, total_q, stream); });
        return PyLong_FromLong(st);
    });
}

// (ctx, k_src, v_src, k_dst, v_dst, src_ids, dst_ids, num_pairs, stream)
PyObject *py_copy(PyObject *, PyObject *const *a, Py_ssize_t n) noexcept
{
    return guarded([&]() -> PyObject * {
        ooco_ctx *ctx;
        void *ks, *vs, *kd, *vd, *stream;
        int64_t *src, *dst;
        int pairs;
        if (n != 9 || !plain() || !get_handle(a[0], ctx) || !get_ptr(a[1], ks) || !get_ptr(a[2], vs) || !get_ptr(a[3], kd) || !get_ptr(a[4], vd) ||
            !get_ptr(a[5], src) || !get_ptr(a[6], dst) || !get_size(a[7], a[5], pairs) || !get_stream(a[8], stream))
            return not_plain();
        const int st = call([&]() { return f_copy(ctx, ks, vs, kd, vd, src, dst, pairs, stream); });
        return PyLong_FromLong(st);
    });
}

// bind(c_void_p, addresses of ooco_plan, ooco_attn_mixed, ooco_attn_mixed_static, ooco_kv_append, ooco_kv_block_copy): the
// functions of the library that binding.py has loaded (this module does not load one of its own).
PyObject *py_bind(PyObject *, PyObject *args)
{
    PyObject *type;
    unsigned long long p[5];
    if (!PyArg_ParseTuple(args, "O!KKKKK", &PyType_Type, &type, &p[0], &p[1], &p[2], &p[3], &p[4])) return nullptr;
    Py_INCREF(type);
    handle_type = reinterpret_cast<PyTypeObject *>(type);
    f_plan = reinterpret_cast<decltype(f_plan)>(p[0]);
    f_attn = reinterpret_cast<decltype(f_attn)>(p[1]);
    f_static = reinterpret_cast<decltype(f_static)>(p[2]);
    f_append = reinterpret_cast<decltype(f_append)>(p[3]);
    f_copy = reinterpret_cast<decltype(f_copy)>(p[4]);
    Py_RETURN_NONE;
}

#define OOCO_FAST(name, fn, doc) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(fn)), METH_FASTCALL, doc}
PyMethodDef methods[] = {
    OOCO_FAST("plan", py_plan, "ooco_plan"),
    OOCO_FAST("attn_mixed", py_attn, "ooco_attn_mixed"),
    OOCO_FAST("attn_mixed_static", py_static, "ooco_attn_mixed_static"),
    OOCO_FAST("kv_append", py_append, "ooco_kv_append"),
    OOCO_FAST("kv_block_copy", py_copy, "ooco_kv_block_copy"),
    {"bind", py_bind, METH_VARARGS, "the library's functions"},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", "Native argument marshalling of the per-step calls.", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void)
{
    import_array();
    PyObject *const m = PyModule_Create(&module);
    if (m && !of_tensor) of_tensor = PyObject_CallNoArgs(reinterpret_cast<PyObject *>(&PyBaseObject_Type));
    if (m && (!of_tensor || PyModule_AddObjectRef(m, "OF_TENSOR", of_tensor) != 0 || PyModule_AddStringConstant(m, "BUILT_FOR", OOCO_BUILT_FOR) != 0)) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
