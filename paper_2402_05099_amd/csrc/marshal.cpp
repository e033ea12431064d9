// The argument marshalling of the decode-step calls (fused attention, cache update) as a CPython extension: the checks of
// binding.py on the tensors, their device pointers, and the call into libhydragen.so, whose functions it is handed as addresses.
//
// Why native: such a call is one to three kernel launches of a few microseconds each, and checking a dozen tensors
// attribute by attribute in Python took longer than the kernels.  4 sequences x 4 heads, 128 shared keys: 10.0 us a call through
// Python, 5.4 through this (the kernel's own time); a decode step of the same size (copy of the lengths, cache update, attention) 20.2 -> 10.3.
//
// Every function returns the library's return code, or None where anything about the arguments is not plainly as the call
// wants it (another type, a wrong shape, a tensor that is not an ordinary one): binding.py then goes through its own
// checks, which say what is wrong or accept it.  Nothing is kept from one call for the next.
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/version.h>

#include <climits>

#include "hydragen.h"

namespace {

decltype(&hg_hydragen_attn) f_attn;
decltype(&hg_hydragen_attn_fp8) f_attn_fp8;
decltype(&hg_hydragen_attn_paged) f_attn_paged;
decltype(&hg_kv_append) f_append;
decltype(&hg_kv_append_fp8) f_append_fp8;
decltype(&hg_kv_append_paged) f_append_paged;
PyObject *level_type, *paged_type;

PyObject *s_h, *s_value, *s_nq, *s_K, *s_V, *s_n_blocks, *s_kv_off, *s_seq_off, *s_max_rows, *s_max_seqs, *s_page_table, *s_page_size,
    *s_kv_format, *s_k_scale, *s_v_scale;

struct NotPlain {};      // thrown: leave it to binding.py

struct Ref {             // an owned reference
    PyObject* p;
    explicit Ref(PyObject* o) : p(o) {
        if (!o) throw NotPlain();
    }
    ~Ref() { Py_DECREF(p); }
    Ref(const Ref&) = delete;
    Ref& operator=(const Ref&) = delete;
};

void require(bool ok) {
    if (!ok) throw NotPlain();
}

int to_int(PyObject* o) {
    require(PyLong_CheckExact(o));
    int overflow = 0;
    const long v = PyLong_AsLongAndOverflow(o, &overflow);
    require(!overflow && v >= INT_MIN && v <= INT_MAX);
    return (int)v;
}
int int_attr(PyObject* o, PyObject* name) { return to_int(Ref(PyObject_GetAttr(o, name)).p); }
float to_float(PyObject* o) {
    require(PyFloat_CheckExact(o));
    return (float)PyFloat_AS_DOUBLE(o);
}

// An ordinary tensor: no subclass, no wrapper of a transform (those have no storage of their own).
const at::Tensor& tensor(PyObject* o) {
    require(THPVariable_CheckExact(o));
    const at::Tensor& t = THPVariable_Unpack(o);
    require(t.defined() && t.layout() == c10::kStrided && t.has_storage() && !t.unsafeGetTensorImpl()->is_python_dispatch());
    return t;
}
const at::Tensor& device_tensor(PyObject* o, at::ScalarType type) {
    const at::Tensor& t = tensor(o);
    require(t.is_cuda() && t.is_contiguous() && t.scalar_type() == type);
    return t;
}
const void* vector_of(PyObject* o, int64_t n) {      // int32 [n]
    const at::Tensor& t = device_tensor(o, at::kInt);
    require(t.dim() == 1 && t.size(0) == n);
    return t.data_ptr();
}
const void* offsets_of(PyObject* level, PyObject* name) {
    const Ref o(PyObject_GetAttr(level, name));
    return o.p == Py_None ? nullptr : tensor(o.p).data_ptr();
}

hg_ctx* context(PyObject* ctx, int nq) {
    const Ref h(PyObject_GetAttr(ctx, s_h));
    const Ref value(PyObject_GetAttr(h.p, s_value));
    require(PyLong_CheckExact(value.p));
    void* const p = PyLong_AsVoidPtr(value.p);
    require(p != nullptr);
    int have = 1;                        // the context's number of queries per sequence
    PyObject* const n = PyObject_GetAttr(ctx, s_nq);
    if (n) {
        const Ref r(n);
        have = to_int(n);
    } else {
        PyErr_Clear();
    }
    require(have == nq);                 // (binding.py sets it)
    return static_cast<hg_ctx*>(p);
}

// [B, H, D] or [B, nq, H, D], bf16
struct Rows {
    const at::Tensor& t;
    int64_t B, nq, H, D;
    explicit Rows(PyObject* o) : t(device_tensor(o, at::kBFloat16)) {
        const int n = (int)t.dim();
        require(n == 3 || n == 4);
        B = t.size(0);
        nq = n == 4 ? t.size(1) : 1;
        H = t.size(n - 2);
        D = t.size(n - 1);
        require(B <= INT_MAX && nq <= INT_MAX && H <= INT_MAX && D <= INT_MAX);
    }
};

struct Outputs {
    void* O;
    int dtype;
    float* lse;
    Outputs(PyObject* o, PyObject* l, const Rows& q) {
        const at::Tensor& t = tensor(o);
        require(t.scalar_type() == at::kFloat || t.scalar_type() == at::kBFloat16);
        device_tensor(o, t.scalar_type());
        require(t.sizes() == q.t.sizes());
        O = t.data_ptr();
        dtype = t.scalar_type() == at::kFloat ? HG_F32 : HG_BF16;
        lse = nullptr;
        if (l != Py_None) {
            const at::Tensor& s = device_tensor(l, at::kFloat);
            require(s.sizes() == q.t.sizes().slice(0, q.t.dim() - 1));
            lse = static_cast<float*>(s.data_ptr());
        }
    }
};

struct Levels {
    hg_level lv[HG_MAX_LEVELS];
    int n;
    int64_t Hkv;
    explicit Levels(PyObject* list) {
        require(PyList_CheckExact(list) && PyList_GET_SIZE(list) <= HG_MAX_LEVELS);
        n = (int)PyList_GET_SIZE(list);
        Hkv = 0;
        for (int i = 0; i < n; ++i) {
            const Ref l(Py_NewRef(PyList_GET_ITEM(list, i)));
            require((PyObject*)Py_TYPE(l.p) == level_type);
            const Ref k(PyObject_GetAttr(l.p, s_K)), v(PyObject_GetAttr(l.p, s_V));
            const at::Tensor &K = device_tensor(k.p, at::kBFloat16), &V = device_tensor(v.p, at::kBFloat16);
            require(K.sizes() == V.sizes() && K.dim() >= 2);
            if (i == 0) Hkv = K.size(1);
            lv[i].K = K.data_ptr();
            lv[i].V = V.data_ptr();
            lv[i].n_blocks = int_attr(l.p, s_n_blocks);
            lv[i].kv_off = static_cast<const int32_t*>(offsets_of(l.p, s_kv_off));
            lv[i].seq_off = static_cast<const int32_t*>(offsets_of(l.p, s_seq_off));
            lv[i].max_rows = int_attr(l.p, s_max_rows);
            lv[i].max_seqs = int_attr(l.p, s_max_seqs);
        }
    }
};

// K and V rows of a packed cache: two tensors [T, Hkv, D] of one shape
struct Cache {
    const at::Tensor &K, &V;
    Cache(PyObject* k, PyObject* v, at::ScalarType type) : K(device_tensor(k, type)), V(device_tensor(v, type)) {
        require(K.sizes() == V.sizes() && K.dim() == 3);
    }
};

struct Paged {
    hg_paged_kv kv;
    int64_t Hkv;
    Paged(PyObject* o, int64_t B, int64_t D) {
        require((PyObject*)Py_TYPE(o) == paged_type);
        kv.kv_format = int_attr(o, s_kv_format);
        const at::ScalarType type = kv.kv_format == HG_KV_E4M3 ? at::kByte : at::kBFloat16;
        const Ref k(PyObject_GetAttr(o, s_K)), v(PyObject_GetAttr(o, s_V)), t(PyObject_GetAttr(o, s_page_table));
        const Cache rows(k.p, v.p, type);
        const at::Tensor& table = device_tensor(t.p, at::kInt);
        kv.page_size = int_attr(o, s_page_size);
        require(kv.page_size > 0 && table.dim() == 2 && table.size(0) == B && rows.K.size(2) == D && rows.K.size(0) % kv.page_size == 0);
        require(table.size(1) <= INT_MAX && rows.K.size(0) / kv.page_size <= INT_MAX);
        kv.K = rows.K.data_ptr();
        kv.V = rows.V.data_ptr();
        kv.page_table = static_cast<const int32_t*>(table.data_ptr());
        kv.table_stride = (int)table.size(1);
        kv.n_pages = (int)(rows.K.size(0) / kv.page_size);
        kv.k_scale = to_float(Ref(PyObject_GetAttr(o, s_k_scale)).p);
        kv.v_scale = to_float(Ref(PyObject_GetAttr(o, s_v_scale)).p);
        Hkv = rows.K.size(1);
    }
};

// Runs `body`, which returns a code of the library; None where it throws.
template <class F>
PyObject* guarded(Py_ssize_t have, Py_ssize_t want, F body) {
    int rc;
    try {
        require(have == want);
        rc = body();
    } catch (...) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    return PyLong_FromLong(rc);
}
template <class F>
int without_gil(F call) {
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = call();
    Py_END_ALLOW_THREADS
    return rc;
}

// (ctx, Q, levels, Ks, Vs, offsets, lengths, max_len, O, LSE, scale)
PyObject* attn(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 11, [&]() {
        const Rows q(a[1]);
        const Levels lv(a[2]);
        const Cache kv(a[3], a[4], at::kBFloat16);
        const void *off = vector_of(a[5], q.B), *len = vector_of(a[6], q.B);
        const int max_len = to_int(a[7]);
        const Outputs out(a[8], a[9], q);
        const float scale = to_float(a[10]);
        hg_ctx* const c = context(a[0], (int)q.nq);
        const int64_t Hkv = lv.n ? lv.Hkv : kv.K.size(1);
        return without_gil([&]() {
            return f_attn(c, q.t.data_ptr(), lv.n, lv.lv, kv.K.data_ptr(), kv.V.data_ptr(), (const int32_t*)off, (const int32_t*)len, max_len, (int)q.B,
                          (int)q.H, (int)Hkv, (int)q.D, scale, out.O, out.dtype, out.lse);
        });
    });
}
// (ctx, Q, levels, Ks8, Vs8, k_scale, v_scale, offsets, lengths, max_len, O, LSE, scale)
PyObject* attn_fp8(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 13, [&]() {
        const Rows q(a[1]);
        const Levels lv(a[2]);
        const Cache kv(a[3], a[4], at::kByte);
        const float ks = to_float(a[5]), vs = to_float(a[6]);
        const void *off = vector_of(a[7], q.B), *len = vector_of(a[8], q.B);
        const int max_len = to_int(a[9]);
        const Outputs out(a[10], a[11], q);
        const float scale = to_float(a[12]);
        hg_ctx* const c = context(a[0], (int)q.nq);
        return without_gil([&]() {
            return f_attn_fp8(c, q.t.data_ptr(), lv.n, lv.lv, kv.K.data_ptr(), kv.V.data_ptr(), ks, vs, (const int32_t*)off, (const int32_t*)len, max_len,
                              (int)q.B, (int)q.H, (int)kv.K.size(1), (int)q.D, scale, out.O, out.dtype, out.lse);
        });
    });
}
// (ctx, Q, levels, kv, lengths, max_len, O, LSE, scale)
PyObject* attn_paged(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 9, [&]() {
        const Rows q(a[1]);
        const Levels lv(a[2]);
        const Paged kv(a[3], q.B, q.D);
        const void* len = vector_of(a[4], q.B);
        const int max_len = to_int(a[5]);
        const Outputs out(a[6], a[7], q);
        const float scale = to_float(a[8]);
        hg_ctx* const c = context(a[0], (int)q.nq);
        return without_gil([&]() {
            return f_attn_paged(c, q.t.data_ptr(), lv.n, lv.lv, &kv.kv, (const int32_t*)len, max_len, (int)q.B, (int)q.H, (int)kv.Hkv, (int)q.D, scale, out.O,
                                out.dtype, out.lse);
        });
    });
}
const at::Tensor& like(PyObject* o, const Rows& k) {
    const at::Tensor& v = device_tensor(o, at::kBFloat16);
    require(v.sizes() == k.t.sizes());
    return v;
}
// (ctx, Knew, Vnew, Ks, Vs, offsets, lengths, capacity)
PyObject* append(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 8, [&]() {
        const Rows k(a[1]);
        const at::Tensor& v = like(a[2], k);
        const Cache kv(a[3], a[4], at::kBFloat16);
        require(kv.K.size(1) == k.H && kv.K.size(2) == k.D);
        const void *off = vector_of(a[5], k.B), *len = vector_of(a[6], k.B);
        const int capacity = to_int(a[7]);
        hg_ctx* const c = context(a[0], (int)k.nq);
        return without_gil([&]() {
            return f_append(c, k.t.data_ptr(), v.data_ptr(), kv.K.data_ptr(), kv.V.data_ptr(), (const int32_t*)off, (int32_t*)len, capacity, (int)k.B, (int)k.H, (int)k.D);
        });
    });
}
// (ctx, Knew, Vnew, Ks8, Vs8, k_scale, v_scale, offsets, lengths, capacity)
PyObject* append_fp8(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 10, [&]() {
        const Rows k(a[1]);
        const at::Tensor& v = like(a[2], k);
        const Cache kv(a[3], a[4], at::kByte);
        require(kv.K.size(1) == k.H && kv.K.size(2) == k.D);
        const float ks = to_float(a[5]), vs = to_float(a[6]);
        const void *off = vector_of(a[7], k.B), *len = vector_of(a[8], k.B);
        const int capacity = to_int(a[9]);
        hg_ctx* const c = context(a[0], (int)k.nq);
        return without_gil([&]() {
            return f_append_fp8(c, k.t.data_ptr(), v.data_ptr(), kv.K.data_ptr(), kv.V.data_ptr(), ks, vs, (const int32_t*)off, (int32_t*)len, capacity, (int)k.B,
                                (int)k.H, (int)k.D);
        });
    });
}
// (ctx, Knew, Vnew, kv, lengths, capacity)
PyObject* append_paged(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 6, [&]() {
        const Rows k(a[1]);
        const at::Tensor& v = like(a[2], k);
        const Paged kv(a[3], k.B, k.D);
        require(kv.Hkv == k.H);
        const void* len = vector_of(a[4], k.B);
        const int capacity = to_int(a[5]);
        hg_ctx* const c = context(a[0], (int)k.nq);
        return without_gil([&]() { return f_append_paged(c, k.t.data_ptr(), v.data_ptr(), &kv.kv, (int32_t*)len, capacity, (int)k.B, (int)k.H, (int)k.D); });
    });
}

// ([addresses of the six functions, in the order above], Level, PagedKV)
PyObject* setup(PyObject*, PyObject* args) {
    PyObject *list, *lt, *pt;
    if (!PyArg_ParseTuple(args, "O!OO", &PyList_Type, &list, &lt, &pt)) return nullptr;
    void* f[6];
    if (PyList_GET_SIZE(list) != 6) {
        PyErr_SetString(PyExc_ValueError, "six addresses are wanted");
        return nullptr;
    }
    for (int i = 0; i < 6; ++i) {
        f[i] = PyLong_AsVoidPtr(PyList_GET_ITEM(list, i));
        if (PyErr_Occurred()) return nullptr;
    }
    f_attn = (decltype(f_attn))f[0];
    f_attn_fp8 = (decltype(f_attn_fp8))f[1];
    f_attn_paged = (decltype(f_attn_paged))f[2];
    f_append = (decltype(f_append))f[3];
    f_append_fp8 = (decltype(f_append_fp8))f[4];
    f_append_paged = (decltype(f_append_paged))f[5];
    Py_INCREF(lt);
    Py_INCREF(pt);
    level_type = lt;
    paged_type = pt;
    Py_RETURN_NONE;
}

#define HG_FAST(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {HG_FAST(attn), HG_FAST(attn_fp8), HG_FAST(attn_paged), HG_FAST(append), HG_FAST(append_fp8), HG_FAST(append_paged),
                         {"setup", setup, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) {
    struct { PyObject** s; const char* text; } names[] = {
        {&s_h, "h"}, {&s_value, "value"}, {&s_nq, "_nq"}, {&s_K, "K"}, {&s_V, "V"}, {&s_n_blocks, "n_blocks"}, {&s_kv_off, "kv_off"}, {&s_seq_off, "seq_off"},
        {&s_max_rows, "max_rows"}, {&s_max_seqs, "max_seqs"}, {&s_page_table, "page_table"}, {&s_page_size, "page_size"}, {&s_kv_format, "kv_format"},
        {&s_k_scale, "k_scale"}, {&s_v_scale, "v_scale"}};
    for (auto& n : names)
        if (!(*n.s = PyUnicode_InternFromString(n.text))) return nullptr;
    PyObject* const m = PyModule_Create(&module);
    // (binding.py compares it: another version's tensors may be laid out in another way)
    if (m && PyModule_AddStringConstant(m, "torch_version", TORCH_VERSION) < 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
