// The binding's checks and marshalling in native code: what lca.py does for a call whose arguments are a plain Desc (and CacheLayout) and
// plain torch tensors, in one C call.  A function here either makes the library call and returns its status, or touches nothing and
// returns -1: an argument is of another kind (a raw address, a tensor subclass, a field that is no plain number), or does not fit (wrong type, too
// small, not contiguous, not on the device).  Then lca.py takes its own way, which handles the first and words the exception for the second.
// An exception that arises on the way and is not about the arguments ends the call.
//
// Why: a decode step's host time was 11.6 us -- two launches of 3.1 us each, 0.7 us in the library, the rest here -- and the step is not longer
// than that on the GPU at one sequence; a prefill of two calls and three launches took 20 us whatever its size.  With the checks in Python the
// marshalling of a call took 4.3 us.
//
// Nothing is kept between calls but the addresses of the library's entry points, the two Python types and lca.py's function for a stream's address.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstring>

#include <torch/csrc/autograd/python_variable.h>

#include "lca.h"

namespace {

PyTypeObject *desc_type = nullptr, *layout_type = nullptr;
PyObject *stream_of = nullptr;         // lca.py's address of a stream argument

enum Entry { ROWS, CONDENSE, PREFILL, PREFILL_UP, DENSE, DECODE, DECODE_CACHED, DECODE_Q8, UPDATE, QUANTIZE, N_ENTRIES };
const char *const ENTRY_NAMES[N_ENTRIES] = {"lca_condensed_rows", "lca_condense", "lca_prefill_attn", "lca_prefill_attn_up", "dense_mla_attn",
                                            "lca_decode_attn", "lca_decode_attn_cached", "lca_decode_attn_q8", "lca_cache_update", "lca_quantize_cache"};
void *entry[N_ENTRIES] = {};

constexpr int N_INTS = 13, N_FLOATS = 2, N_LAYOUT = 3;
const char *const INT_FIELDS[N_INTS] = {"B", "L", "H", "S", "d_pool", "d_sel", "g", "w", "n_q", "mode", "dtype", "pool_reduce", "sel_reduce"};
const char *const FLOAT_FIELDS[N_FLOATS] = {"scale", "rep_logit_bias"};
const char *const LAYOUT_FIELDS[N_LAYOUT] = {"m_cap", "k_cap", "k_start"};
PyObject *int_names[N_INTS], *float_names[N_FLOATS], *layout_names[N_LAYOUT];

// Something that lca.py will meet again and word itself is cleared here; what is not the call's own (an interrupt, a signal handler's exception) stays set, and
// the call ends with it.
bool missing()
{
    if (PyErr_ExceptionMatches(PyExc_AttributeError)) PyErr_Clear();
    return false;
}

bool read_int(PyObject *o, PyObject *name, int32_t &out)
{
    PyObject *v = PyObject_GetAttr(o, name);
    if (v == nullptr) return missing();
    int overflow = 0;
    const long x = PyLong_CheckExact(v) ? PyLong_AsLongAndOverflow(v, &overflow) : 0;
    const bool ok = PyLong_CheckExact(v) && overflow == 0 && x >= INT32_MIN && x <= INT32_MAX;
    out = (int32_t)x;
    Py_DECREF(v);
    return ok;
}

bool read_float(PyObject *o, PyObject *name, float &out)
{
    PyObject *v = PyObject_GetAttr(o, name);
    if (v == nullptr) return missing();
    const double x = PyFloat_CheckExact(v) ? PyFloat_AS_DOUBLE(v) : 0.0;
    const bool ok = PyFloat_CheckExact(v);
    out = (float)x;
    Py_DECREF(v);
    return ok;
}

// A number of elements; a product past 2^63 - 1 stays there, and no tensor is that large.
struct Count {
    int64_t v;
    Count operator*(int64_t x) const
    {
        int64_t r;
        return Count{__builtin_mul_overflow(v, x, &r) ? INT64_MAX : r};
    }
};

// What a call works with: the C descriptor, the row counts that follow from it, the layout if there is one.
struct Call {
    lca_desc d;
    lca_cache_layout lay;
    bool has_layout = false;
    int32_t m = 0, k = 0;
    int64_t P = 1, dqk = 0, m_cap = 0, k_cap = 0;

    bool read(PyObject *desc, PyObject *layout)
    {
        if (Py_TYPE(desc) != desc_type) return false;
        int32_t f[N_INTS];
        for (int i = 0; i < N_INTS; ++i)
            if (!read_int(desc, int_names[i], f[i])) return false;
        d.B = f[0]; d.L = f[1]; d.H = f[2]; d.S = f[3]; d.d_pool = f[4]; d.d_sel = f[5]; d.g = f[6]; d.w = f[7]; d.n_q = f[8];
        d.mode = f[9]; d.dtype = f[10]; d.pool_reduce = f[11]; d.sel_reduce = f[12];
        if (!read_float(desc, float_names[0], d.scale) || !read_float(desc, float_names[1], d.rep_logit_bias)) return false;
        if (d.mode != LCA_MODE_MLA && d.mode != LCA_MODE_GQA) return false;
        if (d.dtype != LCA_BF16 && d.dtype != LCA_F32 && d.dtype != LCA_F16) return false;
        if (((lca_status(*)(const lca_desc *, int32_t *, int32_t *))entry[ROWS])(&d, &m, &k) != LCA_OK) return false;
        P = d.mode == LCA_MODE_MLA ? 1 : d.S;
        dqk = d.mode == LCA_MODE_MLA ? (int64_t)d.d_pool + d.d_sel : d.d_sel;
        m_cap = m;
        k_cap = k;
        if (layout != nullptr && layout != Py_None) {
            if (Py_TYPE(layout) != layout_type || !read_int(layout, layout_names[0], lay.m_cap) || !read_int(layout, layout_names[1], lay.k_cap) ||
                !read_int(layout, layout_names[2], lay.k_start) || lay.m_cap < 0 || lay.k_cap < 0)
                return false;
            has_layout = true;
            m_cap = lay.m_cap;
            k_cap = lay.k_cap;
        }
        return true;
    }
    Count B() const { return Count{d.B}; }
};

enum Kind { ELT, I32, F32, U8, ANY };

// Address of a tensor of at least `elems` elements of the kind asked for; false if lca.py has to look at it.
bool address(PyObject *o, const Call &c, Kind kind, int64_t elems, bool optional, void *&out)
{
    out = nullptr;
    if (o == Py_None) return optional || elems == 0;
    if (!THPVariable_CheckExact(o)) return false;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || !t.has_storage() || !t.is_contiguous()) return false;
    const at::ScalarType s = t.scalar_type();
    switch (kind) {
    case ELT:
        if (c.d.dtype == LCA_BF16 ? s != at::kBFloat16 && s != at::kShort && s != at::kUInt16 : s != (c.d.dtype == LCA_F32 ? at::kFloat : at::kHalf)) return false;
        break;
    case I32: if (s != at::kInt) return false; break;
    case F32: if (s != at::kFloat) return false; break;
    case U8: if (s != at::kByte) return false; break;
    case ANY: break;
    }
    if (t.numel() < elems) return false;
    out = t.data_ptr();
    return true;
}

// Arguments one by one; `ok` goes false at the first that lca.py has to look at.
struct Args {
    PyObject *const *o;
    const Call &c;
    bool ok = true;
    void *take(Kind kind, Count elems, bool optional = false)
    {
        void *p = nullptr;
        if (ok) ok = address(*o, c, kind, elems.v, optional, p);
        ++o;
        return p;
    }
    void *workspace(size_t &bytes)
    {
        PyObject *w = *o;
        void *p = take(ANY, Count{0});
        if (ok && w != Py_None) bytes = (size_t)THPVariable_Unpack(w).nbytes();
        else ok = false;
        return p;
    }
    void *stream()
    {
        if (!ok) return nullptr;                 // (asked for last: without a device there may be no stream to ask for)
        PyObject *v = PyObject_CallOneArg(stream_of, *o++);
        if (v == nullptr) return ok = missing(), nullptr;
        void *p = PyLong_CheckExact(v) ? PyLong_AsVoidPtr(v) : nullptr;
        ok = PyLong_CheckExact(v);
        if (p == nullptr && PyErr_Occurred()) {             // (a number past any address)
            ok = false;
            PyErr_Clear();
        }
        Py_DECREF(v);
        return p;
    }
};

template <typename F> PyObject *run(F &&f)
{
    lca_status st;
    Py_BEGIN_ALLOW_THREADS
    st = f();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong((long)st);
}
PyObject *pass() { return PyErr_Occurred() ? nullptr : PyLong_FromLong(-1); }

typedef const void *CP;
typedef void *VP;

// A function of n arguments, the first a Desc; with LAYOUT the second a CacheLayout or None.  C++ exceptions (a tensor without data) pass to lca.py.
template <bool LAYOUT, typename F> PyObject *guarded(PyObject *const *args, Py_ssize_t n, Py_ssize_t want, F &&body)
{
    if (n != want || entry[ROWS] == nullptr) return pass();
    try {
        Call c;
        if (!c.read(args[0], LAYOUT ? args[1] : nullptr)) return pass();
        Args a{args + (LAYOUT ? 2 : 1), c};
        return body(c, a);
    } catch (...) {
        return pass();
    }
}

PyObject *condense(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return guarded<false>(args, n, 10, [](Call &c, Args &a) {
        const lca_desc &d = c.d;
        VP Q = a.take(ELT, c.B() * d.L * d.H * c.dqk), pool = a.take(ELT, c.B() * d.L * c.P * d.d_pool), sel = a.take(ELT, c.B() * d.L * c.P * d.d_sel);
        VP pr = a.take(ELT, c.B() * d.S * c.m * d.d_pool), sr = a.take(ELT, c.B() * d.S * c.m * d.d_sel), an = a.take(I32, c.B() * d.S * c.m);
        VP al = a.take(F32, c.B() * d.S * c.m * d.g, true);
        size_t bytes = 0;
        VP ws = a.workspace(bytes), st = a.stream();
        if (!a.ok) return pass();
        return run([&] { return ((lca_status(*)(const lca_desc *, CP, CP, CP, VP, VP, VP, VP, VP, size_t, VP))entry[CONDENSE])(&d, Q, pool, sel, pr, sr, an, al, ws, bytes, st); });
    });
}

PyObject *prefill_attn(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return guarded<false>(args, n, 10, [](Call &c, Args &a) {
        const lca_desc &d = c.d;
        VP Q = a.take(ELT, c.B() * d.L * d.H * c.dqk), pool = a.take(ELT, c.B() * d.L * c.P * d.d_pool), sel = a.take(ELT, c.B() * d.L * c.P * d.d_sel);
        VP pr = a.take(ELT, c.B() * d.S * c.m * d.d_pool), sr = a.take(ELT, c.B() * d.S * c.m * d.d_sel), O = a.take(ELT, c.B() * d.L * d.H * d.d_pool);
        VP lse = a.take(F32, c.B() * d.L * d.H, true);
        size_t bytes = 0;
        VP ws = a.workspace(bytes), st = a.stream();
        if (!a.ok) return pass();
        return run([&] { return ((lca_status(*)(const lca_desc *, CP, CP, CP, CP, CP, VP, VP, VP, size_t, VP))entry[PREFILL])(&d, Q, pool, sel, pr, sr, O, lse, ws, bytes, st); });
    });
}

PyObject *prefill_attn_up(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return guarded<false>(args, n, 11, [](Call &c, Args &a) {
        const lca_desc &d = c.d;
        VP Q = a.take(ELT, c.B() * d.L * d.H * c.dqk), pool = a.take(ELT, c.B() * d.L * c.P * d.d_pool), sel = a.take(ELT, c.B() * d.L * c.P * d.d_sel);
        VP pr = a.take(ELT, c.B() * d.S * c.m * d.d_pool), sr = a.take(ELT, c.B() * d.S * c.m * d.d_sel), W = a.take(ELT, Count{d.H} * 128 * d.d_pool);
        VP O = a.take(ELT, c.B() * d.L * d.H * 128), lse = a.take(F32, c.B() * d.L * d.H, true);
        size_t bytes = 0;
        VP ws = a.workspace(bytes), st = a.stream();
        if (!a.ok) return pass();
        return run([&] { return ((lca_status(*)(const lca_desc *, CP, CP, CP, CP, CP, CP, VP, VP, VP, size_t, VP))entry[PREFILL_UP])(&d, Q, pool, sel, pr, sr, W, O, lse, ws, bytes, st); });
    });
}

PyObject *dense_attn(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return guarded<false>(args, n, 8, [](Call &c, Args &a) {
        const lca_desc &d = c.d;
        VP Q = a.take(ELT, c.B() * d.L * d.H * c.dqk), pool = a.take(ELT, c.B() * d.L * c.P * d.d_pool), sel = a.take(ELT, c.B() * d.L * c.P * d.d_sel);
        VP O = a.take(ELT, c.B() * d.L * d.H * d.d_pool), lse = a.take(F32, c.B() * d.L * d.H, true);
        size_t bytes = 0;
        VP ws = a.workspace(bytes), st = a.stream();
        if (!a.ok) return pass();
        return run([&] { return ((lca_status(*)(const lca_desc *, CP, CP, CP, VP, VP, VP, size_t, VP))entry[DENSE])(&d, Q, pool, sel, O, lse, ws, bytes, st); });
    });
}

PyObject *decode_attn(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return guarded<false>(args, n, 9, [](Call &c, Args &a) {
        const lca_desc &d = c.d;
        VP q = a.take(ELT, c.B() * d.H * c.dqk), pr = a.take(ELT, c.B() * d.S * c.m * d.d_pool), sr = a.take(ELT, c.B() * d.S * c.m * d.d_sel);
        VP pt = a.take(ELT, c.B() * c.P * c.k * d.d_pool), st_ = a.take(ELT, c.B() * c.P * c.k * d.d_sel), O = a.take(ELT, c.B() * d.H * d.d_pool);
        size_t bytes = 0;
        VP ws = a.workspace(bytes), st = a.stream();
        if (!a.ok) return pass();
        return run([&] { return ((lca_status(*)(const lca_desc *, CP, CP, CP, CP, CP, VP, VP, size_t, VP))entry[DECODE])(&d, q, pr, sr, pt, st_, O, ws, bytes, st); });
    });
}

PyObject *decode_attn_cached(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return guarded<true>(args, n, 10, [](Call &c, Args &a) {
        if (!c.has_layout) return pass();
        const lca_desc &d = c.d;
        const int64_t rows = c.m > 0 ? c.m_cap : 0;
        VP q = a.take(ELT, c.B() * d.H * c.dqk), pr = a.take(ELT, c.B() * d.S * rows * d.d_pool), sr = a.take(ELT, c.B() * d.S * rows * d.d_sel);
        VP pt = a.take(ELT, c.B() * c.P * c.k_cap * d.d_pool), st_ = a.take(ELT, c.B() * c.P * c.k_cap * d.d_sel), O = a.take(ELT, c.B() * d.H * d.d_pool);
        size_t bytes = 0;
        VP ws = a.workspace(bytes), st = a.stream();
        if (!a.ok) return pass();
        return run([&] { return ((lca_status(*)(const lca_desc *, const lca_cache_layout *, CP, CP, CP, CP, CP, VP, VP, size_t, VP))entry[DECODE_CACHED])(&d, &c.lay, q, pr, sr, pt, st_, O, ws, bytes, st); });
    });
}

PyObject *decode_attn_q8(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return guarded<true>(args, n, 11, [](Call &c, Args &a) {
        const lca_desc &d = c.d;
        const int64_t rows = c.m > 0 ? c.m_cap : 0;
        VP q = a.take(ELT, c.B() * d.H * c.dqk), pr = a.take(U8, c.B() * d.S * rows * d.d_pool), sr = a.take(U8, c.B() * d.S * rows * d.d_sel);
        VP sc = a.take(F32, c.B() * d.S * rows * 2), pt = a.take(ELT, c.B() * c.P * c.k_cap * d.d_pool), st_ = a.take(ELT, c.B() * c.P * c.k_cap * d.d_sel);
        VP O = a.take(ELT, c.B() * d.H * d.d_pool);
        size_t bytes = 0;
        VP ws = a.workspace(bytes), st = a.stream();
        if (!a.ok) return pass();
        return run([&] { return ((lca_status(*)(const lca_desc *, const lca_cache_layout *, CP, CP, CP, CP, CP, CP, VP, VP, size_t, VP))entry[DECODE_Q8])(&d, c.has_layout ? &c.lay : nullptr, q, pr, sr, sc, pt, st_, O, ws, bytes, st); });
    });
}

PyObject *cache_update(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return guarded<true>(args, n, 10, [](Call &c, Args &a) {
        if (!c.has_layout) return pass();
        const lca_desc &d = c.d;
        VP q = a.take(ELT, c.B() * (d.n_q != 0 ? d.n_q : d.g) * d.H * c.dqk);
        VP pt = a.take(ELT, c.B() * c.P * c.k_cap * d.d_pool), st_ = a.take(ELT, c.B() * c.P * c.k_cap * d.d_sel);
        VP pr = a.take(ELT, c.B() * d.S * c.m_cap * d.d_pool), sr = a.take(ELT, c.B() * d.S * c.m_cap * d.d_sel), an = a.take(I32, c.B() * d.S * c.m_cap, true);
        size_t bytes = 0;
        VP ws = a.workspace(bytes), st = a.stream();
        if (!a.ok) return pass();
        return run([&] { return ((lca_status(*)(const lca_desc *, const lca_cache_layout *, CP, CP, CP, VP, VP, VP, VP, size_t, VP))entry[UPDATE])(&d, &c.lay, q, pt, st_, pr, sr, an, ws, bytes, st); });
    });
}

PyObject *quantize_cache(PyObject *, PyObject *const *args, Py_ssize_t n)      // (desc, layout, pool_rep, sel_rep, pool_q8, sel_q8, scales, stream, first_row)
{
    return guarded<true>(args, n, 9, [&](Call &c, Args &a) {
        const lca_desc &d = c.d;
        VP pr = a.take(ELT, c.B() * d.S * c.m_cap * d.d_pool), sr = a.take(ELT, c.B() * d.S * c.m_cap * d.d_sel);
        VP pq = a.take(U8, c.B() * d.S * c.m_cap * d.d_pool), sq = a.take(U8, c.B() * d.S * c.m_cap * d.d_sel), sc = a.take(F32, c.B() * d.S * c.m_cap * 2);
        int overflow = 0;
        const long first = PyLong_CheckExact(args[8]) ? PyLong_AsLongAndOverflow(args[8], &overflow) : -1;
        if (overflow != 0 || first < 0 || first >= c.m) return pass();
        VP st = a.stream();
        if (!a.ok) return pass();
        return run([&] { return ((lca_status(*)(const lca_desc *, const lca_cache_layout *, int32_t, CP, CP, VP, VP, VP, VP))entry[QUANTIZE])(&d, c.has_layout ? &c.lay : nullptr, (int32_t)first, pr, sr, pq, sq, sc, st); });
    });
}

// setup(Desc, CacheLayout, {entry point: address}, stream function, what is imported): torch's accessors are compiled in, so this module reads sizes and
// addresses of tensors of the torch it was built for, and of no other's.
PyObject *setup(PyObject *, PyObject *args)
{
    PyObject *dt, *lt, *addresses, *fn;
    const char *imported;
    if (!PyArg_ParseTuple(args, "OOO!Os", &dt, &lt, &PyDict_Type, &addresses, &fn, &imported)) return nullptr;
    if (!PyType_Check(dt) || !PyType_Check(lt) || !PyCallable_Check(fn)) {
        PyErr_SetString(PyExc_TypeError, "setup(Desc, CacheLayout, addresses, stream function, what is imported)");
        return nullptr;
    }
    if (std::strcmp(imported, LCA_BUILT_FOR) != 0) {
        PyErr_Format(PyExc_ImportError, "built for %s, but %s is imported", LCA_BUILT_FOR, imported);
        return nullptr;
    }
    void *found[N_ENTRIES];
    for (int i = 0; i < N_ENTRIES; ++i) {
        PyObject *v = PyDict_GetItemString(addresses, ENTRY_NAMES[i]);
        if (v == nullptr) {
            PyErr_Format(PyExc_KeyError, "%s", ENTRY_NAMES[i]);
            return nullptr;
        }
        found[i] = PyLong_AsVoidPtr(v);
        if (found[i] == nullptr) {
            if (!PyErr_Occurred()) PyErr_Format(PyExc_ValueError, "%s has no address", ENTRY_NAMES[i]);
            return nullptr;
        }
    }
    Py_INCREF(dt);
    Py_INCREF(lt);
    Py_INCREF(fn);
    stream_of = fn;
    desc_type = (PyTypeObject *)dt;
    layout_type = (PyTypeObject *)lt;
    for (int i = 0; i < N_ENTRIES; ++i) entry[i] = found[i];
    Py_RETURN_NONE;
}

#define LCA_FAST(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {{"setup", setup, METH_VARARGS, nullptr}, LCA_FAST(condense), LCA_FAST(prefill_attn), LCA_FAST(prefill_attn_up), LCA_FAST(dense_attn),
                         LCA_FAST(decode_attn), LCA_FAST(decode_attn_cached), LCA_FAST(decode_attn_q8), LCA_FAST(cache_update), LCA_FAST(quantize_cache),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_lcabind", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__lcabind()
{
    for (int i = 0; i < N_INTS; ++i)
        if ((int_names[i] = PyUnicode_InternFromString(INT_FIELDS[i])) == nullptr) return nullptr;
    for (int i = 0; i < N_FLOATS; ++i)
        if ((float_names[i] = PyUnicode_InternFromString(FLOAT_FIELDS[i])) == nullptr) return nullptr;
    for (int i = 0; i < N_LAYOUT; ++i)
        if ((layout_names[i] = PyUnicode_InternFromString(LAYOUT_FIELDS[i])) == nullptr) return nullptr;
    return PyModule_Create(&module);
}
