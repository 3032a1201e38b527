// Extension module _native: the calls of a decode step, from Python to the library without ctypes.  A step of one row takes 16 us, of
// which marshalling by ctypes and the tensors' attribute checks took 4; here they take a fraction of one.
//   Every function has a plain Python twin in binding.py that it hands the call to whenever something is not the ordinary
// case -- other types, arguments by other names, a check that fails -- so that what the twin does, or raises, stays the definition.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <climits>
#include <cstring>
#include <new>
#include <vector>
#include "zf_py.h"
#include "../../include/zapformat.h"

namespace {

struct {                               // the library's calls (addresses given by binding.py: whichever build of it was loaded)
    int (*state_reset)(zf_state *);
    int (*advance)(zf_state *, int32_t);
    int (*advance_batch)(zf_state *const *, const int32_t *, int32_t, int32_t *);
    int (*compute_mask)(zf_engine *, zf_state *const *, int32_t, uint32_t *, void *);
    int (*compute_mask_noalloc)(zf_engine *, zf_state *const *, int32_t, uint32_t *, void *);
    int (*compute_mask_async)(zf_engine *, zf_state *const *, int32_t, uint32_t *, void *);
    int (*compute_mask_apply_async)(zf_engine *, zf_state *const *, int32_t, uint32_t *, const void *, void *, int32_t, int64_t, void *);
    int (*mask_wait)(zf_engine *, void *);
    int (*apply_mask)(zf_engine *, const void *, void *, int32_t, int32_t, int64_t, const uint32_t *, void *);
} L;
const zfpy::TensorCalls *T = nullptr;  // null until _native_torch has been loaded
PyObject *check_py = nullptr;          // binding._check: raises for a return code
PyObject *twins = nullptr;             // {name: the Python function}

struct EngineBase { PyObject_HEAD zf_engine *h; int32_t device; int64_t V, W; };
struct StateBase { PyObject_HEAD zf_state *h; };
struct BatchBase { PyObject_HEAD std::vector<zf_state *> *rows; std::vector<int32_t> *ids; };
PyTypeObject *EngineType, *StateType, *BatchType;

PyObject *done(int rc) {               // None, or what binding._check raises
    if (rc == ZF_OK) Py_RETURN_NONE;
    PyObject *code = PyLong_FromLong(rc);
    if (!code) return nullptr;
    PyObject *r = PyObject_CallOneArg(check_py, code);
    Py_DECREF(code);
    return r;
}
PyObject *twin(const char *name, PyObject *const *args, Py_ssize_t n, PyObject *kw) {
    PyObject *f = PyDict_GetItemString(twins, name);
    if (!f) { PyErr_Format(PyExc_RuntimeError, "no twin of %s", name); return nullptr; }
    return PyObject_Vectorcall(f, args, (size_t)n, kw);
}
template <class F>
int unlocked(F f) {                    // other Python threads run meanwhile, as they do during a ctypes call
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f();
    Py_END_ALLOW_THREADS
    return rc;
}

// ---- base classes ----
void plain_dealloc(PyObject *o) {
    PyTypeObject *t = Py_TYPE(o);
    t->tp_free(o);
    Py_DECREF(t);
}
PyObject *state_get_h(PyObject *o, void *) { zf_state *h = ((StateBase *)o)->h; if (!h) Py_RETURN_NONE; return PyLong_FromVoidPtr(h); }
int state_set_h(PyObject *o, PyObject *v, void *) {
    if (!v || v == Py_None) { ((StateBase *)o)->h = nullptr; return 0; }
    void *p = PyLong_AsVoidPtr(v);
    if (!p && PyErr_Occurred()) return -1;
    ((StateBase *)o)->h = (zf_state *)p;
    return 0;
}
bool as_token(PyObject *o, int32_t *out) {   // an exact int that fits
    if (!PyLong_CheckExact(o)) return false;
    int over = 0;
    const long v = PyLong_AsLongAndOverflow(o, &over);
    if (over || v < INT32_MIN || v > INT32_MAX) return false;
    *out = (int32_t)v;
    return true;
}
PyObject *state_advance(PyObject *o, PyObject *const *args, Py_ssize_t n, PyObject *kw) {
    zf_state *h = ((StateBase *)o)->h;
    int32_t t;
    if (n != 1 || kw || !h || !as_token(args[0], &t)) {
        std::vector<PyObject *> a(args, args + n + (kw ? PyTuple_GET_SIZE(kw) : 0));
        a.insert(a.begin(), o);
        return twin("State.advance", a.data(), n + 1, kw);
    }
    const int rc = unlocked([&] { return L.advance(h, t); });
    return done(rc);
}
PyObject *state_reset(PyObject *o, PyObject *) {
    zf_state *h = ((StateBase *)o)->h;
    if (!h) return twin("State.reset", &o, 1, nullptr);
    return done(L.state_reset(h));
}
PyObject *engine_bind(PyObject *o, PyObject *args) {   // _bind(handle or None, device, V, W)
    EngineBase *e = (EngineBase *)o;
    PyObject *h;
    int device;
    long long V, W;
    if (!PyArg_ParseTuple(args, "OiLL", &h, &device, &V, &W)) return nullptr;
    void *p = nullptr;
    if (h != Py_None) { p = PyLong_AsVoidPtr(h); if (!p && PyErr_Occurred()) return nullptr; }
    e->h = (zf_engine *)p; e->device = device; e->V = V; e->W = W;
    Py_RETURN_NONE;
}
void batch_dealloc(PyObject *o) {
    delete ((BatchBase *)o)->rows; delete ((BatchBase *)o)->ids;
    ((BatchBase *)o)->rows = nullptr; ((BatchBase *)o)->ids = nullptr;
    plain_dealloc(o);
}
PyObject *batch_bind(PyObject *o, PyObject *list) {    // _bind(states): their handles
    BatchBase *b = (BatchBase *)o;
    if (!PyList_Check(list)) { PyErr_SetString(PyExc_TypeError, "a list of states is wanted"); return nullptr; }
    try {
        if (!b->rows) b->rows = new std::vector<zf_state *>();
        if (!b->ids) b->ids = new std::vector<int32_t>();
        b->rows->clear();
        for (Py_ssize_t k = 0; k < PyList_GET_SIZE(list); k++) {
            PyObject *s = PyList_GET_ITEM(list, k);
            if (!PyObject_TypeCheck(s, StateType)) { PyErr_SetString(PyExc_TypeError, "a list of states is wanted"); return nullptr; }
            b->rows->push_back(((StateBase *)s)->h);
        }
        b->ids->resize(b->rows->size());
    } catch (const std::bad_alloc &) { return PyErr_NoMemory(); }
    Py_RETURN_NONE;
}
PyObject *batch_advance(PyObject *o, PyObject *const *args, Py_ssize_t n, PyObject *kw) {
    BatchBase *b = (BatchBase *)o;
    bool ok = n == 1 && !kw && b->rows && PyList_CheckExact(args[0]) && PyList_GET_SIZE(args[0]) == (Py_ssize_t)b->rows->size();
    if (ok) {
        PyObject *const *item = PySequence_Fast_ITEMS(args[0]);
        int32_t *ids = b->ids->data();
        for (size_t k = 0; k < b->rows->size() && ok; k++) ok = as_token(item[k], &ids[k]);
    }
    if (!ok) {
        std::vector<PyObject *> a(args, args + n + (kw ? PyTuple_GET_SIZE(kw) : 0));
        a.insert(a.begin(), o);
        return twin("StateBatch.advance", a.data(), n + 1, kw);
    }
    const int rc = unlocked([&] { return L.advance_batch(b->rows->data(), b->ids->data(), (int32_t)b->rows->size(), nullptr); });
    return done(rc);
}

// ---- the calls of a step ----
struct Rows {                          // the handles of a StateBatch, or of a list of states
    std::vector<zf_state *> own;
    zf_state *const *p = nullptr;
    int64_t n = 0;
    bool take(PyObject *o) {
        if (PyObject_TypeCheck(o, BatchType)) {
            BatchBase *b = (BatchBase *)o;
            if (!b->rows) return false;
            p = b->rows->data(); n = (int64_t)b->rows->size();
        } else if (PyList_CheckExact(o)) {
            n = PyList_GET_SIZE(o);
            own.resize((size_t)n);
            for (int64_t k = 0; k < n; k++) {
                PyObject *s = PyList_GET_ITEM(o, k);
                if (!PyObject_TypeCheck(s, StateType)) return false;
                own[(size_t)k] = ((StateBase *)s)->h;
            }
            p = own.data();
        } else return false;
        return n > 0 && n <= INT32_MAX;
    }
};
bool engine_of(PyObject *o, EngineBase **e) { *e = (EngineBase *)o; return PyObject_TypeCheck(o, EngineType) && (*e)->h; }
bool mask_of(PyObject *o, const EngineBase *e, int64_t n, zfpy::TensorInfo *m) {
    return T->look(o, m) && m->device >= 0 && m->contiguous && m->dtype == 2 && m->dim == 2 && m->size[0] == n && m->size[1] == e->W;
}
bool logits_of(PyObject *o, const EngineBase *e, zfpy::TensorInfo *x) {
    return T->look(o, x) && x->device >= 0 && x->dim == 2 && x->stride[1] == 1 && x->size[1] == e->V && (x->dtype == 0 || x->dtype == 1);
}
bool same_shape(const zfpy::TensorInfo &a, const zfpy::TensorInfo &b) {
    return a.dim == b.dim && a.dtype == b.dtype && a.size[0] == b.size[0] && a.size[1] == b.size[1] && a.stride[0] == b.stride[0] && a.stride[1] == b.stride[1];
}
PyObject *itself(PyObject *o, int rc) {  // the call's result: its output tensor
    if (rc != ZF_OK) return done(rc);
    Py_INCREF(o);
    return o;
}
// one keyword at most, and that one `out` (the last of `most` arguments): its value, null when there is none
bool only_out(Py_ssize_t n, PyObject *kw, PyObject *const *args, Py_ssize_t most, PyObject **out) {
    *out = n == most ? args[most - 1] : nullptr;
    if (kw && PyTuple_GET_SIZE(kw)) {
        if (PyTuple_GET_SIZE(kw) != 1 || n != most - 1 || PyUnicode_CompareWithASCIIString(PyTuple_GET_ITEM(kw, 0), "out") != 0) return false;
        *out = args[n];
    }
    if (*out == Py_None) *out = nullptr;
    return n == most - 1 || n == most;
}

typedef int (*MaskCall)(zf_engine *, zf_state *const *, int32_t, uint32_t *, void *);
PyObject *mask_call(const char *name, MaskCall call, PyObject *const *args, Py_ssize_t n, PyObject *kw) {
    EngineBase *e;
    Rows rows;
    zfpy::TensorInfo m;
    void *s;
    if (!T || n != 3 || kw || !engine_of(args[0], &e) || !rows.take(args[1]) || !mask_of(args[2], e, rows.n, &m) || !T->stream(e->device, &s)) return twin(name, args, n, kw);
    const int rc = unlocked([&] { return call(e->h, rows.p, (int32_t)rows.n, (uint32_t *)m.data, s); });
    return itself(args[2], rc);
}
PyObject *compute_mask(PyObject *, PyObject *const *args, Py_ssize_t n, PyObject *kw) { return mask_call("compute_mask", L.compute_mask, args, n, kw); }
PyObject *compute_mask_noalloc(PyObject *, PyObject *const *args, Py_ssize_t n, PyObject *kw) { return mask_call("compute_mask_noalloc", L.compute_mask_noalloc, args, n, kw); }
PyObject *compute_mask_async(PyObject *, PyObject *const *args, Py_ssize_t n, PyObject *kw) { return mask_call("compute_mask_async", L.compute_mask_async, args, n, kw); }
PyObject *compute_mask_apply_async(PyObject *, PyObject *const *args, Py_ssize_t n, PyObject *kw) {
    EngineBase *e;
    Rows rows;
    zfpy::TensorInfo m, x, y;
    PyObject *out;
    void *s;
    if (!T || !only_out(n, kw, args, 5, &out) || !engine_of(args[0], &e) || !rows.take(args[1]) || !mask_of(args[2], e, rows.n, &m) ||
        !logits_of(args[3], e, &x) || x.size[0] != rows.n || (out && (!T->look(out, &y) || y.device < 0 || !same_shape(x, y))) || !T->stream(e->device, &s))
        return twin("compute_mask_apply_async", args, n, kw);
    if (!out) { out = args[3]; y = x; }
    const int rc = unlocked([&] { return L.compute_mask_apply_async(e->h, rows.p, (int32_t)rows.n, (uint32_t *)m.data, x.data, y.data, x.dtype, x.stride[0], s); });
    return itself(out, rc);
}
PyObject *apply_mask(PyObject *, PyObject *const *args, Py_ssize_t n, PyObject *kw) {
    EngineBase *e;
    zfpy::TensorInfo m, x, y;
    PyObject *out;
    void *s;
    if (!T || !only_out(n, kw, args, 4, &out) || !engine_of(args[0], &e) || !logits_of(args[1], e, &x) || x.size[0] <= 0 || x.size[0] > INT32_MAX ||
        !T->look(args[2], &m) || m.device < 0 || (out && (!T->look(out, &y) || y.device < 0 || !same_shape(x, y))) || !T->stream(e->device, &s))
        return twin("apply_mask", args, n, kw);
    if (!out) { out = args[1]; y = x; }
    const int rc = unlocked([&] { return L.apply_mask(e->h, x.data, y.data, x.dtype, (int32_t)x.size[0], x.stride[0], (const uint32_t *)m.data, s); });
    return itself(out, rc);
}
PyObject *mask_wait(PyObject *, PyObject *const *args, Py_ssize_t n, PyObject *kw) {
    EngineBase *e;
    void *s;
    if (!T || n != 1 || kw || !engine_of(args[0], &e) || !T->stream(e->device, &s)) return twin("mask_wait", args, n, kw);
    const int rc = unlocked([&] { return L.mask_wait(e->h, s); });
    return done(rc);
}

// pack_vocab(tokens): the byte strings of a list one behind the other, and where each begins (n + 1 64-bit offsets), both as bytearrays; None for anything
// but a list of bytes.  (128,256 tokens: 0.75 ms; numpy over map(len) and a join took 3.)
PyObject *pack_vocab(PyObject *, PyObject *list) {
    if (!PyList_CheckExact(list)) Py_RETURN_NONE;
    const Py_ssize_t n = PyList_GET_SIZE(list);
    PyObject *off = PyByteArray_FromStringAndSize(nullptr, (n + 1) * (Py_ssize_t)sizeof(int64_t));
    if (!off) return nullptr;
    int64_t *at = (int64_t *)PyByteArray_AS_STRING(off);
    at[0] = 0;
    for (Py_ssize_t k = 0; k < n; k++) {
        PyObject *t = PyList_GET_ITEM(list, k);
        if (!PyBytes_CheckExact(t)) { Py_DECREF(off); Py_RETURN_NONE; }
        at[k + 1] = at[k] + PyBytes_GET_SIZE(t);
    }
    PyObject *data = PyByteArray_FromStringAndSize(nullptr, at[n] ? at[n] : 1);
    if (!data) { Py_DECREF(off); return nullptr; }
    char *to = PyByteArray_AS_STRING(data);
    to[0] = 0;
    for (Py_ssize_t k = 0; k < n; k++) memcpy(to + at[k], PyBytes_AS_STRING(PyList_GET_ITEM(list, k)), (size_t)(at[k + 1] - at[k]));
    return Py_BuildValue("(NN)", off, data);
}

// ---- set-up ----
PyObject *bind_library(PyObject *, PyObject *args) {   // ({name: address}, _check, twins)
    PyObject *addr, *chk, *tw;
    if (!PyArg_ParseTuple(args, "O!OO!", &PyDict_Type, &addr, &chk, &PyDict_Type, &tw)) return nullptr;
    auto take = [&](const char *name, void **to) {
        PyObject *v = PyDict_GetItemString(addr, name);
        *to = v ? PyLong_AsVoidPtr(v) : nullptr;
        if (!*to && !PyErr_Occurred()) PyErr_Format(PyExc_RuntimeError, "no address of %s", name);
        return *to != nullptr;
    };
    if (!take("zf_state_reset", (void **)&L.state_reset) || !take("zf_advance", (void **)&L.advance) || !take("zf_advance_batch", (void **)&L.advance_batch) ||
        !take("zf_compute_mask", (void **)&L.compute_mask) || !take("zf_compute_mask_noalloc", (void **)&L.compute_mask_noalloc) ||
        !take("zf_compute_mask_async", (void **)&L.compute_mask_async) || !take("zf_compute_mask_apply_async", (void **)&L.compute_mask_apply_async) ||
        !take("zf_mask_wait", (void **)&L.mask_wait) || !take("zf_apply_mask", (void **)&L.apply_mask)) return nullptr;
    Py_INCREF(chk); Py_XSETREF(check_py, chk);
    Py_INCREF(tw); Py_XSETREF(twins, tw);
    Py_RETURN_NONE;
}
PyObject *bind_torch(PyObject *, PyObject *capsule) {
    void *p = PyCapsule_GetPointer(capsule, zfpy::TENSOR_CALLS_NAME);
    if (!p) return nullptr;
    T = (const zfpy::TensorCalls *)p;
    Py_RETURN_NONE;
}

// Python calls C: no C++ exception goes that way (the vectors of handles and arguments can fail to grow).
typedef PyObject *(*FastCall)(PyObject *, PyObject *const *, Py_ssize_t, PyObject *);
template <FastCall F>
PyObject *guarded(PyObject *self, PyObject *const *args, Py_ssize_t n, PyObject *kw) {
    try { return F(self, args, n, kw); } catch (const std::bad_alloc &) { return PyErr_NoMemory(); }
}
#define FAST(f) (PyCFunction)(void (*)(void))guarded<f>, METH_FASTCALL | METH_KEYWORDS
PyMethodDef state_methods[] = {
    {"advance", FAST(state_advance), "advance($self, token_id)\n--\n\nFeed a token's bytes (raises ZfError when the grammar rejects them)."},
    {"reset", state_reset, METH_NOARGS, "reset($self)\n--\n\nBack to the empty prefix."}, {nullptr, nullptr, 0, nullptr}};
PyGetSetDef state_getset[] = {{"h", state_get_h, state_set_h, "handle of the library's state", nullptr}, {nullptr, nullptr, nullptr, nullptr, nullptr}};
PyMethodDef engine_methods[] = {{"_bind", engine_bind, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyMethodDef batch_methods[] = {
    {"advance", FAST(batch_advance), "advance($self, token_ids)\n--\n\nEvery row by one token; token_ids[b] < 0 resets row b."},
    {"_bind", batch_bind, METH_O, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyType_Slot state_slots[] = {{Py_tp_methods, state_methods}, {Py_tp_getset, state_getset}, {Py_tp_dealloc, (void *)plain_dealloc}, {0, nullptr}};
PyType_Slot engine_slots[] = {{Py_tp_methods, engine_methods}, {Py_tp_dealloc, (void *)plain_dealloc}, {0, nullptr}};
PyType_Slot batch_slots[] = {{Py_tp_methods, batch_methods}, {Py_tp_dealloc, (void *)batch_dealloc}, {0, nullptr}};
PyType_Spec state_spec = {"paper_2506_01151_amd._native.StateBase", sizeof(StateBase), 0, Py_TPFLAGS_DEFAULT | Py_TPFLAGS_BASETYPE, state_slots};
PyType_Spec engine_spec = {"paper_2506_01151_amd._native.EngineBase", sizeof(EngineBase), 0, Py_TPFLAGS_DEFAULT | Py_TPFLAGS_BASETYPE, engine_slots};
PyType_Spec batch_spec = {"paper_2506_01151_amd._native.BatchBase", sizeof(BatchBase), 0, Py_TPFLAGS_DEFAULT | Py_TPFLAGS_BASETYPE, batch_slots};
PyMethodDef methods[] = {
    {"compute_mask", FAST(compute_mask), "compute_mask(engine, states, mask_tensor)\n--\n\nmask_tensor: torch int32 tensor [batch, W] on the engine's device (fully overwritten)."},
    {"compute_mask_noalloc", FAST(compute_mask_noalloc), "compute_mask_noalloc(engine, states, mask_tensor)\n--\n\ncompute_mask through the entry point that allocates no device memory."},
    {"compute_mask_async", FAST(compute_mask_async), "compute_mask_async(engine, states, mask_tensor)\n--\n\nEnqueue only; pair with mask_wait(engine) before reading the mask on the host."},
    {"compute_mask_apply_async", FAST(compute_mask_apply_async), "compute_mask_apply_async(engine, states, mask_tensor, logits, out=None)\n--\n\ncompute_mask and apply_mask of the same rows, enqueued together; pair with mask_wait(engine)."},
    {"mask_wait", FAST(mask_wait), "mask_wait(engine)\n--\n\nWait for the status of the calls in flight."},
    {"apply_mask", FAST(apply_mask), "apply_mask(engine, logits, mask_tensor, out=None)\n--\n\nlogits: torch fp32 or bf16 tensor [batch, V] (last dim contiguous) on the device."},
    {"pack_vocab", pack_vocab, METH_O, nullptr},
    {"bind_library", bind_library, METH_VARARGS, nullptr},
    {"bind_torch", bind_torch, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_native", "The calls of a decode step, from Python to the library.", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) {
    PyObject *m = PyModule_Create(&module_def);
    if (!m) return nullptr;
    EngineType = (PyTypeObject *)PyType_FromSpec(&engine_spec);
    StateType = (PyTypeObject *)PyType_FromSpec(&state_spec);
    BatchType = (PyTypeObject *)PyType_FromSpec(&batch_spec);
    if (!EngineType || !StateType || !BatchType) return nullptr;
    Py_INCREF(EngineType); Py_INCREF(StateType); Py_INCREF(BatchType);
    if (PyModule_AddObject(m, "EngineBase", (PyObject *)EngineType) < 0 || PyModule_AddObject(m, "StateBase", (PyObject *)StateType) < 0 ||
        PyModule_AddObject(m, "BatchBase", (PyObject *)BatchType) < 0) return nullptr;
    return m;
}
