// Argument marshalling of the Python binding in native code: the entry points'
// tensors are checked (type, element type, element count, device, contiguity)
// and turned into pointers here, and the C entry point is called with the GIL
// released. It holds no step of the path.
//
// Host time bounds the smallest calls: the kernels of a tiny request take under
// 15 us on the GPU, and checking its 20 tensors through Python attributes and
// calling through ctypes took 13 of 25.4 us of host time; here 13.9 us in all, of
// which the three launches and two pointer queries are 10.
//
// Anything out of the ordinary (a failed check, a host-resident store, an
// argument of another type, a tensor whose size or pointer torch will not give)
// makes a function return None with nothing called; the caller then takes the
// Python path, which handles it or raises.
#include <Python.h>

#include <torch/csrc/autograd/python_variable.h>

#include <exception>

#include "inferscale.h"

namespace {

decltype(&is_retrieve) p_retrieve;
decltype(&is_slot_map) p_slot_map;
decltype(&is_inject_rotary) p_inject_rotary;
decltype(&is_place_inject) p_place_inject;
decltype(&is_paged_scores) p_paged_scores;
decltype(&is_ann_search) p_ann_search;
PyObject* g_resolve_stream;  // Python: stream argument -> raw stream

// One call's arguments, taken in order; ok turns false at the first that this
// path does not handle.
struct Args {
    PyObject* const* v;
    Py_ssize_t n, i = 0;
    bool ok = true;

    PyObject* next() {
        if (i >= n) ok = false;
        return ok ? v[i++] : nullptr;
    }
    int64_t i64() {
        PyObject* o = next();
        if (!o || !PyLong_CheckExact(o)) { ok = false; return 0; }
        const long long x = PyLong_AsLongLong(o);
        if (x == -1 && PyErr_Occurred()) { PyErr_Clear(); ok = false; }
        return x;
    }
    int32_t i32() {
        const int64_t x = i64();
        if (x < INT32_MIN || x > INT32_MAX) ok = false;
        return (int32_t)x;
    }
    float f32() {
        PyObject* o = next();
        if (!o || !PyFloat_CheckExact(o)) { ok = false; return 0.f; }
        return (float)PyFloat_AS_DOUBLE(o);
    }
    // a strided, contiguous device tensor, or null for None where that is allowed
    const at::Tensor* tensor(bool optional) {
        PyObject* o = next();
        if (!o) return nullptr;
        if (optional && o == Py_None) return nullptr;
        if (!THPVariable_CheckExact(o)) { ok = false; return nullptr; }
        const at::Tensor& t = THPVariable_Unpack(o);
        if (t.layout() != at::kStrided || !t.is_cuda() || !t.has_storage() ||
            t.key_set().has(c10::DispatchKey::Python) || !t.is_contiguous()) {
            ok = false;
            return nullptr;
        }
        return &t;
    }
};

// numel * ... with overflow checks (a negative size passes here and is refused
// by the entry point).
struct Count {
    bool ok = true;
    int64_t mul(int64_t a, int64_t b) {
        int64_t r = 0;
        if (__builtin_mul_overflow(a, b, &r)) ok = false;
        return r;
    }
    // entries a per-request table with `stride` between requests spans
    int64_t table(int64_t n, int64_t nq, int64_t stride) {
        if (stride == 0) return n;
        int64_t r = 0;
        if (__builtin_add_overflow(mul(nq - 1, stride), n, &r)) ok = false;
        return r;
    }
};

// Pointer of a checked tensor; *ok turns false when it is not what the entry
// point takes.
template <class T = void>
T* ptr(const at::Tensor* t, at::ScalarType dt, int64_t numel, bool* ok) {
    if (!t) return nullptr;
    if (t->scalar_type() != dt || t->numel() < numel) { *ok = false; return nullptr; }
    return (T*)t->data_ptr();
}

uint32_t* status_ptr(const at::Tensor* t, bool* ok) {
    if (!t) return nullptr;
    if ((t->scalar_type() != at::kInt && t->scalar_type() != at::kUInt32) || t->numel() < 1) {
        *ok = false;
        return nullptr;
    }
    return (uint32_t*)t->data_ptr();
}

bool emb_dtype(const at::Tensor* t, int32_t* dt) {
    if (!t) return false;
    *dt = t->scalar_type() == at::kFloat ? IS_DTYPE_F32 : IS_DTYPE_BF16;
    return t->scalar_type() == at::kFloat || t->scalar_type() == at::kBFloat16;
}

// The last argument of every call: an int, a torch stream or None.
bool stream_of(PyObject* o, void** st) {
    PyObject* r = PyObject_CallOneArg(g_resolve_stream, o);
    if (!r) return false;
    *st = PyLong_AsVoidPtr(r);
    Py_DECREF(r);
    return !PyErr_Occurred();
}

template <class F>
PyObject* finish(Args& a, PyObject* stream, bool ok, F&& call) {
    if (!a.ok || !ok || a.i != a.n) Py_RETURN_NONE;
    void* st = nullptr;
    if (!stream_of(stream, &st)) return nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS rc = call(st);
    Py_END_ALLOW_THREADS return PyLong_FromLong(rc);
}

PyObject* retrieve(PyObject*, PyObject* const* v, Py_ssize_t n_) {
    Args a{v, n_};
    const at::Tensor *q = a.tensor(false), *bank = a.tensor(false);
    const int64_t n = a.i64();
    const int32_t d = a.i32(), k = a.i32();
    const at::Tensor *ids = a.tensor(false), *sc = a.tensor(true);
    const int32_t nq = a.i32();
    const int64_t stride = a.i64();
    const at::Tensor* ws = a.tensor(false);
    PyObject* so = a.next();
    int32_t dt = 0;
    if (!a.ok || !emb_dtype(q, &dt)) Py_RETURN_NONE;
    Count c;
    bool ok = true;
    const auto et = q->scalar_type();
    const int64_t nd = c.mul(n, d), nk = c.mul(nq, k);
    const void* pq = ptr(q, et, c.mul(nq, d), &ok);
    const void* pb = ptr(bank, et, c.table(nd, nq, stride), &ok);
    int32_t* pi = ptr<int32_t>(ids, at::kInt, nk, &ok);
    float* ps = ptr<float>(sc, at::kFloat, nk, &ok);
    void* pw = ws->data_ptr();
    const size_t wb = ws->nbytes();
    return finish(a, so, ok && c.ok, [&](void* st) {
        return p_retrieve(pq, pb, n, d, k, pi, ps, nq, stride, dt, pw, wb, st);
    });
}

PyObject* slot_map(PyObject*, PyObject* const* v, Py_ssize_t n_) {
    Args a{v, n_};
    const at::Tensor *ids = a.tensor(false), *lens = a.tensor(false);
    const int32_t start = a.i32();
    const at::Tensor* bt = a.tensor(false);
    const int32_t page = a.i32();
    const at::Tensor *os = a.tensor(false), *op = a.tensor(false), *om = a.tensor(false);
    const int32_t k = a.i32(), nq = a.i32();
    const int64_t n = a.i64(), stride = a.i64();
    const int32_t mb = a.i32(), mt = a.i32(), rev = a.i32();
    const at::Tensor* status = a.tensor(true);
    PyObject* so = a.next();
    if (!a.ok) Py_RETURN_NONE;
    Count c;
    bool ok = true;
    const int32_t* pi = ptr<int32_t>(ids, at::kInt, c.mul(nq, k), &ok);
    const int32_t* pl = ptr<int32_t>(lens, at::kInt, c.table(n, nq, stride), &ok);
    const int32_t* pb = ptr<int32_t>(bt, at::kInt, c.mul(nq, mb), &ok);
    int64_t* po = ptr<int64_t>(os, at::kLong, c.mul(nq, mt), &ok);
    int32_t* pp = ptr<int32_t>(op, at::kInt, c.mul(nq, mt), &ok);
    int32_t* pm = ptr<int32_t>(om, at::kInt, nq, &ok);
    uint32_t* pst = status_ptr(status, &ok);
    return finish(a, so, ok && c.ok, [&](void* st) {
        return p_slot_map(pi, pl, start, pb, page, po, pp, pm, k, nq, n, stride, mb, mt, rev, pst, st);
    });
}

// What the injections share, in this order: ids, preK, V, slots, positions, m,
// paged_k, paged_v, fact_offsets, fact_lens, rope_theta, inv_freq, pairing, k,
// nq, n, lens_stride, reverse_rank, max_tokens, L, H, D, T_store, num_slots,
// status.
struct Inject {
    const int32_t *ids, *lens;
    const void *preK, *V;
    int64_t* slots;
    int32_t *positions, *m;
    void *pk, *pv;
    const int64_t* offs;
    float theta;
    const double* inv_freq;
    int32_t pairing, k, nq, rev, mt, L, H, D;
    int64_t n, stride, T_store, num_slots;
    uint32_t* status;

    bool take(Args& a) {
        const at::Tensor* t[10];
        for (const at::Tensor*& x : t) x = a.tensor(false);
        theta = a.f32();
        const at::Tensor* f = a.tensor(true);
        pairing = a.i32(); k = a.i32(); nq = a.i32();
        n = a.i64(); stride = a.i64();
        rev = a.i32(); mt = a.i32(); L = a.i32(); H = a.i32(); D = a.i32();
        T_store = a.i64(); num_slots = a.i64();
        const at::Tensor* s = a.tensor(true);
        if (!a.ok) return false;
        Count c;
        bool ok = true;
        const int64_t row = c.mul(L, c.mul(H, D));
        const int64_t store = c.mul(row, T_store), pages = c.mul(row, num_slots);
        const int64_t table = c.table(n, nq, stride), toks = c.mul(nq, mt);
        ids = ptr<int32_t>(t[0], at::kInt, c.mul(nq, k), &ok);
        preK = ptr(t[1], at::kBFloat16, store, &ok);
        V = ptr(t[2], at::kBFloat16, store, &ok);
        slots = ptr<int64_t>(t[3], at::kLong, toks, &ok);
        positions = ptr<int32_t>(t[4], at::kInt, toks, &ok);
        m = ptr<int32_t>(t[5], at::kInt, nq, &ok);
        pk = ptr(t[6], at::kBFloat16, pages, &ok);
        pv = ptr(t[7], at::kBFloat16, pages, &ok);
        offs = ptr<int64_t>(t[8], at::kLong, table, &ok);
        lens = ptr<int32_t>(t[9], at::kInt, table, &ok);
        // (Python's D // 2 rounds down)
        inv_freq = ptr<double>(f, at::kDouble, D >= 0 ? D / 2 : -((1 - (int64_t)D) / 2), &ok);
        status = status_ptr(s, &ok);
        return ok && c.ok;
    }
};

PyObject* inject_rotary(PyObject*, PyObject* const* v, Py_ssize_t n_) {
    Args a{v, n_};
    Inject x;
    if (!x.take(a)) Py_RETURN_NONE;
    PyObject* so = a.next();
    return finish(a, so, true, [&](void* st) {
        return p_inject_rotary(x.ids, x.preK, x.V, x.slots, x.positions, x.theta, x.pk, x.pv, x.offs,
                               x.lens, x.m, x.k, x.nq, x.n, x.stride, x.rev, x.mt, x.L, x.H, x.D,
                               x.T_store, x.num_slots, x.inv_freq, x.pairing, x.status, st);
    });
}

PyObject* place_inject(PyObject*, PyObject* const* v, Py_ssize_t n_) {
    Args a{v, n_};
    Inject x;
    if (!x.take(a)) Py_RETURN_NONE;
    const int32_t start = a.i32();
    const at::Tensor* bt = a.tensor(false);
    const int32_t page = a.i32(), mb = a.i32();
    PyObject* so = a.next();
    if (!a.ok) Py_RETURN_NONE;
    Count c;
    bool ok = true;
    const int32_t* pb = ptr<int32_t>(bt, at::kInt, c.mul(x.nq, mb), &ok);
    return finish(a, so, ok && c.ok, [&](void* st) {
        return p_place_inject(x.ids, x.preK, x.V, x.offs, x.lens, start, pb, page, mb, x.theta,
                              x.inv_freq, x.pairing, x.pk, x.pv, x.slots, x.positions, x.m, x.k,
                              x.nq, x.n, x.stride, x.rev, x.mt, x.L, x.H, x.D, x.T_store,
                              x.num_slots, x.status, st);
    });
}

PyObject* paged_scores(PyObject*, PyObject* const* v, Py_ssize_t n_) {
    Args a{v, n_};
    const at::Tensor *q = a.tensor(false), *qpos = a.tensor(false), *pk = a.tensor(false);
    const int32_t layer = a.i32();
    const at::Tensor* bt = a.tensor(false);
    const int32_t page = a.i32(), start = a.i32();
    const at::Tensor *m = a.tensor(false), *sc = a.tensor(false);
    const int32_t nq = a.i32(), Hq = a.i32(), H = a.i32(), D = a.i32(), L = a.i32();
    const int64_t num_slots = a.i64();
    const int32_t mb = a.i32(), mt = a.i32();
    const float theta = a.f32();
    const at::Tensor* f = a.tensor(true);
    const int32_t pairing = a.i32();
    const at::Tensor* status = a.tensor(true);
    PyObject* so = a.next();
    if (!a.ok) Py_RETURN_NONE;
    Count c;
    bool ok = true;
    const int64_t qh = c.mul(nq, Hq);
    const void* pq = ptr(q, at::kBFloat16, c.mul(qh, D), &ok);
    const int32_t* pp = ptr<int32_t>(qpos, at::kInt, nq, &ok);
    const void* pkk = ptr(pk, at::kBFloat16, c.mul(c.mul(L, num_slots), c.mul(H, D)), &ok);
    const int32_t* pb = ptr<int32_t>(bt, at::kInt, c.mul(nq, mb), &ok);
    const int32_t* pm = ptr<int32_t>(m, at::kInt, nq, &ok);
    float* ps = ptr<float>(sc, at::kFloat, c.mul(qh, mt), &ok);
    const double* pf = ptr<double>(f, at::kDouble, D >= 0 ? D / 2 : -((1 - (int64_t)D) / 2), &ok);
    uint32_t* pst = status_ptr(status, &ok);
    return finish(a, so, ok && c.ok, [&](void* st) {
        return p_paged_scores(pq, pp, pkk, layer, pb, page, start, pm, ps, nq, Hq, H, D, L,
                              num_slots, mb, mt, theta, pf, pairing, pst, st);
    });
}

PyObject* ann_search(PyObject*, PyObject* const* v, Py_ssize_t n_) {
    Args a{v, n_};
    const at::Tensor *q = a.tensor(false), *bank = a.tensor(false);
    const int64_t n = a.i64();
    const int32_t d = a.i32();
    const at::Tensor* graph = a.tensor(false);
    const int32_t R = a.i32();
    const at::Tensor *seeds = a.tensor(false), *sbank = a.tensor(false), *ids = a.tensor(false);
    const int32_t nq = a.i32(), ns = a.i32(), beam = a.i32(), width = a.i32(), k = a.i32();
    const int32_t iters = a.i32();
    const at::Tensor *sc = a.tensor(true), *oi = a.tensor(true), *os = a.tensor(true);
    const at::Tensor *status = a.tensor(true), *ws = a.tensor(false);
    PyObject* so = a.next();
    int32_t dt = 0;
    if (!a.ok || !emb_dtype(q, &dt)) Py_RETURN_NONE;
    Count c;
    bool ok = true;
    const auto et = q->scalar_type();
    const void* pq = ptr(q, et, c.mul(nq, d), &ok);
    const void* pb = ptr(bank, et, c.mul(n, d), &ok);
    const int32_t* pg = ptr<int32_t>(graph, at::kInt, c.mul(n, R), &ok);
    const int32_t* pse = ptr<int32_t>(seeds, at::kInt, ns, &ok);
    const void* psb = ptr(sbank, et, c.mul(ns, d), &ok);
    int32_t* pi = ptr<int32_t>(ids, at::kInt, c.mul(nq, k), &ok);
    float* ps = ptr<float>(sc, at::kFloat, c.mul(nq, k), &ok);
    int32_t* poi = ptr<int32_t>(oi, at::kInt, nq, &ok);
    int32_t* pos = ptr<int32_t>(os, at::kInt, nq, &ok);
    uint32_t* pst = status_ptr(status, &ok);
    void* pw = ws->data_ptr();
    const size_t wb = ws->nbytes();
    return finish(a, so, ok && c.ok, [&](void* st) {
        return p_ann_search(pq, nq, pb, n, d, dt, pg, R, pse, psb, ns, beam, width, k, iters, pi, ps,
                            poi, pos, pst, pw, wb, st);
    });
}

// bind(resolve_stream, {name: address}): the library's entry points.
PyObject* bind(PyObject*, PyObject* args) {
    PyObject *resolve, *addr;
    if (!PyArg_ParseTuple(args, "OO!", &resolve, &PyDict_Type, &addr)) return nullptr;
    auto get = [&](const char* name) -> void* {
        PyObject* o = PyDict_GetItemString(addr, name);
        if (!o) {
            PyErr_Format(PyExc_KeyError, "%s", name);
            return nullptr;
        }
        return PyLong_AsVoidPtr(o);
    };
#define IS_BIND(NAME)                                                    \
    p_##NAME = reinterpret_cast<decltype(p_##NAME)>(get("is_" #NAME));   \
    if (!p_##NAME) return nullptr
    IS_BIND(retrieve);
    IS_BIND(slot_map);
    IS_BIND(inject_rotary);
    IS_BIND(place_inject);
    IS_BIND(paged_scores);
    IS_BIND(ann_search);
#undef IS_BIND
    Py_INCREF(resolve);
    Py_XSETREF(g_resolve_stream, resolve);
    Py_RETURN_NONE;
}

// torch's accessors throw (a tensor without memory of its own, symbolic sizes),
// and no C++ exception may pass through the interpreter. All of them come before
// the entry point is called.
template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)>
PyObject* guarded(PyObject* self, PyObject* const* v, Py_ssize_t n) {
    try {
        return F(self, v, n);
    } catch (const std::exception&) {
        Py_RETURN_NONE;
    }
}

#define IS_FAST(NAME) {#NAME, (PyCFunction)(void (*)(void))guarded<NAME>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {{"bind", bind, METH_VARARGS, nullptr},
                         IS_FAST(retrieve),
                         IS_FAST(slot_map),
                         IS_FAST(inject_rotary),
                         IS_FAST(place_inject),
                         IS_FAST(paged_scores),
                         IS_FAST(ann_search),
                         {nullptr, nullptr, 0, nullptr}};
#undef IS_FAST

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() { return PyModule_Create(&module); }
