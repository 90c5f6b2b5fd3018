// Argument marshalling of the single-layer calls for CPython: turns torch
// tensors, Layout objects and ints into the C structs of objectcache.h and
// calls the library.  The same conversions in ctypes took 6-8 us per call,
// more than the smallest kernels run; here they take about 1 us.  No
// arithmetic of the method, nothing kept from one call to the next.
//
// The library's functions arrive as addresses (bind), so that whichever build
// of it the package loaded is the one that is called.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstdint>

#include "objectcache.h"

namespace {

decltype(&oc_kv_layer_ingest) f_layer_ingest;
decltype(&oc_kv_chunks_ingest) f_chunks_ingest;
decltype(&oc_kv_layer_gather) f_layer_gather;
decltype(&oc_kv_chunks_gather) f_chunks_gather;
decltype(&oc_kv_suffix_append) f_append;
decltype(&oc_suffix_prefill_layer) f_attention;
decltype(&oc_suffix_prefill_layer_noalloc) f_attention_noalloc;
decltype(&oc_rest_of_layer) f_rest;

PyObject *s_data_ptr, *s_numel, *s_element_size, *s_cuda_stream, *s_value;
PyObject *s_layout[7];                        // Layout's fields, in the struct's order
PyObject *s_weights[5];                       // LayerWeights' fields
PyObject *t_c_void_p;                         // ctypes.c_void_p
PyObject *g_current_stream;                   // () -> the current stream's handle

// An integer, as ctypes takes one: an int or what has __index__ (NumPy
// integers, integer tensors of one element), else a TypeError; wider values
// wrap.
bool as_i64(PyObject *o, int64_t *out) {
    *out = (int64_t)PyLong_AsUnsignedLongLongMask(o);
    return !PyErr_Occurred();
}
bool as_i32(PyObject *o, int32_t *out) {
    int64_t v;
    if (!as_i64(o, &v)) return false;
    *out = (int32_t)v;
    return true;
}

bool call_int(PyObject *o, PyObject *method, int64_t *out) {
    PyObject *r = PyObject_CallMethodNoArgs(o, method);
    if (!r) return false;
    const bool ok = as_i64(r, out);
    Py_DECREF(r);
    return ok;
}

// An address, as ctypes takes one: an int, None or a c_void_p; an object that
// merely has __index__ is a TypeError.
bool as_address(PyObject *o, void **out) {
    *out = nullptr;
    if (o == Py_None) return true;
    if (PyLong_Check(o)) {
        *out = reinterpret_cast<void *>(PyLong_AsUnsignedLongLongMask(o));
        return !PyErr_Occurred();
    }
    const int is = PyObject_IsInstance(o, t_c_void_p);
    if (is < 0) return false;
    if (!is) {
        PyErr_Format(PyExc_TypeError, "%.100s cannot be converted to pointer", Py_TYPE(o)->tp_name);
        return false;
    }
    PyObject *v = PyObject_GetAttr(o, s_value);      // None or an int
    if (!v) return false;
    if (v != Py_None) *out = reinterpret_cast<void *>(PyLong_AsUnsignedLongLongMask(v));
    Py_DECREF(v);
    return !PyErr_Occurred();
}

template <class T>
bool as_ptr(PyObject *tensor, T **out) {      // None: NULL
    *out = nullptr;
    if (tensor == Py_None) return true;
    PyObject *r = PyObject_CallMethodNoArgs(tensor, s_data_ptr);
    if (!r) return false;
    void *v;
    const bool ok = as_address(r, &v);
    Py_DECREF(r);
    *out = static_cast<T *>(v);
    return ok;
}

bool as_layout(PyObject *o, oc_layout *l) {
    int32_t *const dst[6] = {&l->num_layers, &l->num_q_heads, &l->num_kv_heads,
                             &l->head_dim,   &l->page_size,   &l->chunk_tokens};
    for (int i = 0; i < 7; ++i) {
        PyObject *v = PyObject_GetAttr(o, s_layout[i]);
        if (!v) return false;
        const bool ok = i < 6 ? as_i32(v, dst[i]) : as_i64(v, &l->num_pages);
        Py_DECREF(v);
        if (!ok) return false;
    }
    return true;
}

bool as_pool(PyObject *pool, PyObject *layout, oc_kv_pool *out) {
    return as_ptr(pool, &out->base) && as_layout(layout, &out->layout);
}

bool as_table(PyObject *pages, PyObject *num_tokens, oc_block_table *out) {
    out->pages = nullptr;
    out->num_entries = 0;
    if (pages != Py_None) {
        if (!call_int(pages, s_numel, &out->num_entries)) return false;
        if (out->num_entries && !as_ptr(pages, &out->pages)) return false;
    }
    return as_i64(num_tokens, &out->num_tokens);
}

bool as_stream(PyObject *o, void **out) {     // None: the current torch stream
    PyObject *v;
    if (o == Py_None) v = PyObject_CallNoArgs(g_current_stream);
    else if (PyLong_Check(o)) v = Py_NewRef(o);
    else v = PyObject_GetAttr(o, s_cuda_stream);
    if (!v) return false;
    const bool ok = as_address(v, out);
    Py_DECREF(v);
    return ok;
}

// S of eq. (1): bytes of one chunk's layer slice
int64_t slice_bytes(const oc_layout &l) {
    return (int64_t)(2ULL * (uint64_t)(int64_t)l.chunk_tokens * (uint64_t)(int64_t)l.num_kv_heads *
                     (uint64_t)(int64_t)l.head_dim * 2ULL);
}

bool arity(Py_ssize_t got, Py_ssize_t want) {
    if (got == want) return true;
    PyErr_Format(PyExc_TypeError, "%zd arguments expected, got %zd", want, got);
    return false;
}

template <class F>
PyObject *run(F &&call) {
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = call();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// (staging, num_chunks, pages, num_tokens, pool, layout, layer, stream)
PyObject *kv_layer_ingest(PyObject *, PyObject *const *a, Py_ssize_t n) {
    oc_staging st;
    oc_block_table bt;
    oc_kv_pool kp;
    int32_t layer;
    void *s;
    if (!arity(n, 8) || !as_ptr(a[0], &st.data) || !as_i64(a[1], &st.num_chunks) || !as_table(a[2], a[3], &bt) ||
        !as_pool(a[4], a[5], &kp) || !as_i32(a[6], &layer) || !as_stream(a[7], &s))
        return nullptr;
    st.per_layer_chunk_bytes = slice_bytes(kp.layout);
    return run([&] { return f_layer_ingest(&st, &bt, &kp, layer, s); });
}

// (objects, num_chunks, first_chunk, pages, num_tokens, pool, layout, stream)
PyObject *kv_chunks_ingest(PyObject *, PyObject *const *a, Py_ssize_t n) {
    oc_staging st;
    oc_block_table bt;
    oc_kv_pool kp;
    int64_t first;
    void *s;
    if (!arity(n, 8) || !as_ptr(a[0], &st.data) || !as_i64(a[1], &st.num_chunks) || !as_i64(a[2], &first) ||
        !as_table(a[3], a[4], &bt) || !as_pool(a[5], a[6], &kp) || !as_stream(a[7], &s))
        return nullptr;
    st.per_layer_chunk_bytes = slice_bytes(kp.layout);
    return run([&] { return f_chunks_ingest(&st, first, &bt, &kp, s); });
}

// (pages, num_tokens, pool, layout, layer, staging_out, num_chunks, stream)
PyObject *kv_layer_gather(PyObject *, PyObject *const *a, Py_ssize_t n) {
    oc_block_table bt;
    oc_kv_pool kp;
    int32_t layer;
    void *out, *s;
    int64_t chunks;
    if (!arity(n, 8) || !as_table(a[0], a[1], &bt) || !as_pool(a[2], a[3], &kp) || !as_i32(a[4], &layer) ||
        !as_ptr(a[5], &out) || !as_i64(a[6], &chunks) || !as_stream(a[7], &s))
        return nullptr;
    return run([&] { return f_layer_gather(&bt, &kp, layer, out, chunks, slice_bytes(kp.layout), s); });
}

// (pages, num_tokens, pool, layout, first_chunk, num_chunks, objects_out, stream)
PyObject *kv_chunks_gather(PyObject *, PyObject *const *a, Py_ssize_t n) {
    oc_block_table bt;
    oc_kv_pool kp;
    int64_t first, chunks;
    void *out, *s;
    if (!arity(n, 8) || !as_table(a[0], a[1], &bt) || !as_pool(a[2], a[3], &kp) || !as_i64(a[4], &first) ||
        !as_i64(a[5], &chunks) || !as_ptr(a[6], &out) || !as_stream(a[7], &s))
        return nullptr;
    return run([&] { return f_chunks_gather(&bt, &kp, first, chunks, out, s); });
}

// (k_new, v_new, suffix_tokens, pages, num_tokens, pool, layout, layer, stream)
PyObject *kv_suffix_append(PyObject *, PyObject *const *a, Py_ssize_t n) {
    const void *k, *v;
    int64_t ts;
    oc_block_table bt;
    oc_kv_pool kp;
    int32_t layer;
    void *s;
    if (!arity(n, 9) || !as_ptr(a[0], &k) || !as_ptr(a[1], &v) || !as_i64(a[2], &ts) || !as_table(a[3], a[4], &bt) ||
        !as_pool(a[5], a[6], &kp) || !as_i32(a[7], &layer) || !as_stream(a[8], &s))
        return nullptr;
    return run([&] { return f_append(k, v, ts, &bt, &kp, layer, s); });
}

struct AttentionCall {
    const void *q, *k, *v;
    int64_t ts;
    oc_kv_pool kp;
    oc_block_table bt;
    int32_t layer;
    void *out;
    // (q, k_new, v_new, suffix_tokens, pool, layout, pages, num_tokens, layer, out, ...)
    bool parse(PyObject *const *a) {
        return as_ptr(a[0], &q) && as_ptr(a[1], &k) && as_ptr(a[2], &v) && as_i64(a[3], &ts) &&
               as_pool(a[4], a[5], &kp) && as_table(a[6], a[7], &bt) && as_i32(a[8], &layer) && as_ptr(a[9], &out);
    }
};

// (..., workspace, stream)
PyObject *suffix_prefill_layer(PyObject *, PyObject *const *a, Py_ssize_t n) {
    AttentionCall c;
    void *ws, *s;
    int64_t numel, size;
    if (!arity(n, 12) || !c.parse(a) || !as_ptr(a[10], &ws) || !call_int(a[10], s_numel, &numel) ||
        !call_int(a[10], s_element_size, &size) || !as_stream(a[11], &s))
        return nullptr;
    return run([&] {
        return f_attention(c.q, c.k, c.v, c.ts, &c.kp, &c.bt, c.layer, c.out, ws, (size_t)(numel * size), s);
    });
}

// (..., stream)
PyObject *suffix_prefill_layer_noalloc(PyObject *, PyObject *const *a, Py_ssize_t n) {
    AttentionCall c;
    void *s;
    if (!arity(n, 11) || !c.parse(a) || !as_stream(a[10], &s)) return nullptr;
    return run([&] { return f_attention_noalloc(c.q, c.k, c.v, c.ts, &c.kp, &c.bt, c.layer, c.out, s); });
}

// (attn_out, tokens, layout, weights, layer, o, gate_up, act, h, qkv, stream)
PyObject *rest_of_layer(PyObject *, PyObject *const *a, Py_ssize_t n) {
    const void *x;
    int64_t tokens;
    oc_layout l;
    oc_layer_weights w;
    int32_t layer;
    oc_layer_buffers b;
    void *s;
    if (!arity(n, 11) || !as_ptr(a[0], &x) || !as_i64(a[1], &tokens) || !as_layout(a[2], &l)) return nullptr;
    const void **const dst[4] = {&w.w_o, &w.w_gate_up, &w.w_down, &w.w_qkv};
    for (int i = 0; i < 5; ++i) {
        PyObject *v = PyObject_GetAttr(a[3], s_weights[i]);
        if (!v) return nullptr;
        const bool ok = i == 0 ? as_i32(v, &w.ffn_dim) : as_ptr(v, dst[i - 1]);
        Py_DECREF(v);
        if (!ok) return nullptr;
    }
    if (!as_i32(a[4], &layer) || !as_ptr(a[5], &b.o) || !as_ptr(a[6], &b.gate_up) || !as_ptr(a[7], &b.act) ||
        !as_ptr(a[8], &b.h) || !as_ptr(a[9], &b.qkv) || !as_stream(a[10], &s))
        return nullptr;
    return run([&] { return f_rest(x, tokens, &l, &w, layer, &b, s); });
}

// (current_stream, addresses of the eight functions in the order below)
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n) {
    int64_t p[8];
    if (!arity(n, 9)) return nullptr;
    for (int i = 0; i < 8; ++i)
        if (!as_i64(a[i + 1], &p[i])) return nullptr;
    f_layer_ingest = reinterpret_cast<decltype(f_layer_ingest)>(p[0]);
    f_chunks_ingest = reinterpret_cast<decltype(f_chunks_ingest)>(p[1]);
    f_layer_gather = reinterpret_cast<decltype(f_layer_gather)>(p[2]);
    f_chunks_gather = reinterpret_cast<decltype(f_chunks_gather)>(p[3]);
    f_append = reinterpret_cast<decltype(f_append)>(p[4]);
    f_attention = reinterpret_cast<decltype(f_attention)>(p[5]);
    f_attention_noalloc = reinterpret_cast<decltype(f_attention_noalloc)>(p[6]);
    f_rest = reinterpret_cast<decltype(f_rest)>(p[7]);
    Py_XSETREF(g_current_stream, Py_NewRef(a[0]));
    Py_RETURN_NONE;
}

#define FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST(bind),
                         FAST(kv_layer_ingest),
                         FAST(kv_chunks_ingest),
                         FAST(kv_layer_gather),
                         FAST(kv_chunks_gather),
                         FAST(kv_suffix_append),
                         FAST(suffix_prefill_layer),
                         FAST(suffix_prefill_layer_noalloc),
                         FAST(rest_of_layer),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

bool intern(PyObject **out, const char *name) { return (*out = PyUnicode_InternFromString(name)) != nullptr; }

}  // namespace

PyMODINIT_FUNC PyInit__marshal() {
    static const char *const layout[7] = {"num_layers", "num_q_heads",  "num_kv_heads", "head_dim",
                                          "page_size",  "chunk_tokens", "num_pages"};
    static const char *const weights[5] = {"ffn_dim", "w_o", "w_gate_up", "w_down", "w_qkv"};
    if (!intern(&s_data_ptr, "data_ptr") || !intern(&s_numel, "numel") || !intern(&s_element_size, "element_size") ||
        !intern(&s_cuda_stream, "cuda_stream") || !intern(&s_value, "value"))
        return nullptr;
    PyObject *ctypes = PyImport_ImportModule("ctypes");
    if (!ctypes) return nullptr;
    t_c_void_p = PyObject_GetAttrString(ctypes, "c_void_p");
    Py_DECREF(ctypes);
    if (!t_c_void_p) return nullptr;
    for (int i = 0; i < 7; ++i)
        if (!intern(&s_layout[i], layout[i])) return nullptr;
    for (int i = 0; i < 5; ++i)
        if (!intern(&s_weights[i], weights[i])) return nullptr;
    return PyModule_Create(&module);
}
