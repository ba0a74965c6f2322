// The torch binding's call path in native code: checks the tensors of a call,
// reads their sizes and pointers, sets torch's current stream and calls the
// library (include/xdit.h).  A function returns the library's status, or None
// when an argument is not what its fast path takes (another type, shape,
// layout or device): the caller then goes through the checks in Python, which
// name what is wrong.  A call through Python attribute reads and ctypes took
// 8 to 12 us of host time, more than the shortest kernels run; this path
// takes about 2 us plus the launch.
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/xdit.h"

namespace {

PyObject* g_device = nullptr;      // () -> index of the current device
PyObject* g_raw_stream = nullptr;  // (index) -> raw handle of torch's current stream

// One tensor argument: dense, strided, on the GPU.
struct T {
    void* p = nullptr;
    at::IntArrayRef s;
    at::ScalarType dt = at::kFloat;
    int64_t bytes = 0;
};

bool get(PyObject* o, int64_t dims, T* t) {
    if (!THPVariable_CheckExact(o)) return false;
    const at::Tensor& x = THPVariable_Unpack(o);
    if (x.layout() != at::kStrided || !x.is_cuda() || (dims >= 0 && x.dim() != dims) || !x.is_contiguous()) return false;
    t->s = x.sizes();
    t->dt = x.scalar_type();
    t->p = x.data_ptr();
    t->bytes = x.numel() * (int64_t)x.element_size();
    return true;
}

// a K/V buffer: K's plane, then V's
bool buffer(PyObject* o, T* t) { return get(o, 5, t) && t->s[0] >= 2; }

bool get_or_none(PyObject* o, int64_t dims, T* t) { return o == Py_None || get(o, dims, t); }

bool shape4(const T& t, at::ScalarType dt, int64_t a, int64_t b, int64_t c, int64_t d) {
    return t.dt == dt && t.s[0] == a && t.s[1] == b && t.s[2] == c && t.s[3] == d;
}

// an LSE of B x H x n, or none given
bool is_lse(const T& t, int64_t B, int64_t H, int64_t n) {
    return t.s.empty() || (t.dt == at::kFloat && t.s[0] == B && t.s[1] == H && t.s[2] == n);
}

bool code(at::ScalarType dt, int32_t* c) {
    *c = dt == at::kBFloat16 ? XDIT_BF16 : XDIT_F32;
    return dt == at::kBFloat16 || dt == at::kFloat;
}

bool integer(PyObject* o, int64_t* x) {
    if (!PyLong_CheckExact(o)) return false;
    *x = PyLong_AsLongLong(o);
    if (*x == -1 && PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    return true;
}

// up to XDIT_MAX_RANGES (offset, length) pairs; *F their total length
bool ranges(PyObject* o, int64_t* off, int64_t* len, int32_t* n, int64_t* F) {
    if (!PyList_CheckExact(o) && !PyTuple_CheckExact(o)) return false;
    const Py_ssize_t k = PySequence_Fast_GET_SIZE(o);
    if (k > XDIT_MAX_RANGES) return false;
    *F = 0;
    for (Py_ssize_t i = 0; i < k; ++i) {
        PyObject* r = PySequence_Fast_GET_ITEM(o, i);
        if (!PyTuple_CheckExact(r) || PyTuple_GET_SIZE(r) != 2) return false;
        if (!integer(PyTuple_GET_ITEM(r, 0), off + i) || !integer(PyTuple_GET_ITEM(r, 1), len + i)) return false;
        *F += len[i];
    }
    *n = (int32_t)k;
    return true;
}

// torch's current stream for the calling thread's launches
bool use_current_stream() {
    PyObject* dev = PyObject_CallNoArgs(g_device);
    PyObject* st = dev ? PyObject_CallOneArg(g_raw_stream, dev) : nullptr;
    Py_XDECREF(dev);
    void* h = st ? PyLong_AsVoidPtr(st) : nullptr;
    Py_XDECREF(st);
    if (PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    xdit_set_stream(h);
    return true;
}

// Runs `call` without the interpreter lock, as ctypes does.
template <typename F>
PyObject* run(F&& call) {
    if (!use_current_stream()) Py_RETURN_NONE;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = call();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// A C++ exception (a tensor without storage, symbolic sizes) leaves the call
// to the Python path.
template <PyObject* (*F)(PyObject* const*)>
PyObject* guarded(PyObject* const* a) {
    try {
        return F(a);
    } catch (...) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

template <PyObject* (*F)(PyObject* const*), int N>
PyObject* entry(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != N) {
        PyErr_Format(PyExc_TypeError, "%d arguments expected, got %zd", N, n);
        return nullptr;
    }
    return guarded<F>(a);
}

struct Chunk {
    T q, k, v, out, lse;
    int64_t B, Nq, H, d, Nk;
    int32_t dt;
};

bool chunk_args(PyObject* const* a, bool need_lse, Chunk* c) {
    if (!get(a[0], 4, &c->q) || !get(a[1], 4, &c->k) || !get(a[2], 4, &c->v) || !get(a[3], 4, &c->out) ||
        !get_or_none(a[4], 3, &c->lse) || (need_lse && a[4] == Py_None) || !code(c->q.dt, &c->dt))
        return false;
    c->B = c->q.s[0], c->Nq = c->q.s[1], c->H = c->q.s[2], c->d = c->q.s[3], c->Nk = c->k.s[1];
    return shape4(c->k, c->q.dt, c->B, c->Nk, c->H, c->d) && shape4(c->v, c->q.dt, c->B, c->Nk, c->H, c->d) &&
           shape4(c->out, c->q.dt, c->B, c->Nq, c->H, c->d) && is_lse(c->lse, c->B, c->H, c->Nq);
}

// q, k, v, out, lse, accum
PyObject* chunk(PyObject* const* a) {
    Chunk c;
    const bool accum = a[5] == Py_True;
    if (!chunk_args(a, accum, &c)) Py_RETURN_NONE;
    return run([&] {
        return accum ? xdit_chunk_attn_accum(c.q.p, c.k.p, c.v.p, c.out.p, (float*)c.lse.p, c.B, c.Nq, c.Nk, c.H, c.d, c.dt)
                     : xdit_chunk_attn(c.q.p, c.k.p, c.v.p, c.out.p, (float*)c.lse.p, c.B, c.Nq, c.Nk, c.H, c.d, c.dt);
    });
}

// q, k, v, out, lse, splits, workspace, accum
PyObject* chunk_split(PyObject* const* a) {
    Chunk c;
    T ws;
    int64_t splits;
    const bool accum = a[7] == Py_True;
    if (!chunk_args(a, accum, &c) || !integer(a[5], &splits) || splits != (int32_t)splits || !get_or_none(a[6], -1, &ws))
        Py_RETURN_NONE;
    return run([&] {
        return (accum ? xdit_chunk_attn_accum_split : xdit_chunk_attn_split)(
            c.q.p, c.k.p, c.v.p, c.out.p, (float*)c.lse.p, (int32_t)splits, ws.p, ws.bytes, c.B, c.Nq, c.Nk, c.H, c.d, c.dt);
    });
}

// q, kv_buf, patch_off, patch_len, fresh_k, fresh_v, out
PyObject* patch(PyObject* const* a) {
    T q, kv, fk, fv, out;
    int64_t off, len;
    int32_t dt;
    if (!get(a[0], 4, &q) || !buffer(a[1], &kv) || !integer(a[2], &off) || !integer(a[3], &len) || !get(a[4], 4, &fk) ||
        !get(a[5], 4, &fv) || !get(a[6], 4, &out) || !code(kv.dt, &dt))
        Py_RETURN_NONE;
    const int64_t B = kv.s[1], N = kv.s[2], H = kv.s[3], d = kv.s[4];
    for (const T* t : {&q, &fk, &fv, &out})
        if (!shape4(*t, kv.dt, B, len, H, d)) Py_RETURN_NONE;
    return run([&] { return xdit_patch_attn(q.p, kv.p, off, len, fk.p, fv.p, out.p, B, N, H, d, dt); });
}

// q, kv_buf, ranges, fresh_k, fresh_v, out, lse; SPLIT: then splits, workspace
template <bool SPLIT>
PyObject* general_patch(PyObject* const* a) {
    T q, kv, fk, fv, out, lse, ws;
    int64_t off[XDIT_MAX_RANGES] = {}, len[XDIT_MAX_RANGES] = {}, F, splits = 0;
    int32_t dt, nr;
    if (!get(a[0], 4, &q) || !buffer(a[1], &kv) || !ranges(a[2], off, len, &nr, &F) || !get(a[3], 4, &fk) ||
        !get(a[4], 4, &fv) || !get(a[5], 4, &out) || !get_or_none(a[6], 3, &lse) || !code(kv.dt, &dt) ||
        (SPLIT && (!integer(a[7], &splits) || splits != (int32_t)splits || !get_or_none(a[8], -1, &ws))))
        Py_RETURN_NONE;
    const int64_t Nq = q.s[1], B = kv.s[1], N = kv.s[2], H = kv.s[3], d = kv.s[4];
    if (!shape4(q, kv.dt, B, Nq, H, d) || !shape4(out, kv.dt, B, Nq, H, d) || !shape4(fk, kv.dt, B, F, H, d) ||
        !shape4(fv, kv.dt, B, F, H, d) || !is_lse(lse, B, H, Nq))
        Py_RETURN_NONE;
    return run([&] {
        return SPLIT ? xdit_patch_attn_split(q.p, Nq, kv.p, nr, off, len, fk.p, fv.p, out.p, (float*)lse.p,
                                             (int32_t)splits, ws.p, ws.bytes, B, N, H, d, dt)
                     : xdit_patch_attn_ranges(q.p, Nq, kv.p, nr, off, len, fk.p, fv.p, out.p, (float*)lse.p, B, N, H, d,
                                              dt);
    });
}

constexpr auto patch_ranges = general_patch<false>;
constexpr auto patch_split = general_patch<true>;

// outs, lses, n, out, lse_out
PyObject* merge(PyObject* const* a) {
    T out, lo;
    int64_t n;
    int32_t dt;
    if (!PyList_CheckExact(a[0]) || !PyList_CheckExact(a[1]) || !integer(a[2], &n) || n < 1 || n > XDIT_MAX_PARTIALS ||
        n > PyList_GET_SIZE(a[0]) || n > PyList_GET_SIZE(a[1]) || !get(a[3], 4, &out) || !get_or_none(a[4], 3, &lo) ||
        !code(out.dt, &dt))
        Py_RETURN_NONE;
    const int64_t B = out.s[0], Nq = out.s[1], H = out.s[2], d = out.s[3];
    const void* o[XDIT_MAX_PARTIALS];
    const float* l[XDIT_MAX_PARTIALS];
    for (int64_t r = 0; r < n; ++r) {
        T x, y;
        if (!get(PyList_GET_ITEM(a[0], r), 4, &x) || !get(PyList_GET_ITEM(a[1], r), 3, &y) ||
            !shape4(x, out.dt, B, Nq, H, d) || !is_lse(y, B, H, Nq))
            Py_RETURN_NONE;
        o[r] = x.p;
        l[r] = (const float*)y.p;
    }
    if (!is_lse(lo, B, H, Nq)) Py_RETURN_NONE;
    return run([&] { return xdit_lse_merge(o, l, (int32_t)n, out.p, (float*)lo.p, B, Nq, H, d, dt); });
}

// kv_buf, patch_off, patch_len, fresh_k, fresh_v
PyObject* update(PyObject* const* a) {
    T kv, fk, fv;
    int64_t off, len;
    int32_t dt;
    if (!buffer(a[0], &kv) || !integer(a[1], &off) || !integer(a[2], &len) || !get(a[3], 4, &fk) ||
        !get(a[4], 4, &fv) || !code(kv.dt, &dt))
        Py_RETURN_NONE;
    const int64_t B = kv.s[1], N = kv.s[2], H = kv.s[3], d = kv.s[4];
    if (!shape4(fk, kv.dt, B, len, H, d) || !shape4(fv, kv.dt, B, len, H, d)) Py_RETURN_NONE;
    return run([&] { return xdit_kv_update(kv.p, off, len, fk.p, fv.p, B, N, H, d, dt); });
}

// device, raw_stream: the callables that give torch's current stream
PyObject* init(PyObject* const* a) {
    Py_INCREF(a[0]);
    Py_INCREF(a[1]);
    Py_XSETREF(g_device, a[0]);
    Py_XSETREF(g_raw_stream, a[1]);
    Py_RETURN_NONE;
}

#define ENTRY(name, n) {#name, (PyCFunction)(void (*)(void))&entry<name, n>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {ENTRY(init, 2),         ENTRY(chunk, 6),       ENTRY(chunk_split, 8),
                         ENTRY(patch, 7),        ENTRY(patch_ranges, 7), ENTRY(patch_split, 9),
                         ENTRY(merge, 5),        ENTRY(update, 5),      {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() { return PyModule_Create(&module); }
