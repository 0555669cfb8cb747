// The layer calls of the Python binding as a CPython extension module.  A decode layer call is a few
// microseconds of GPU work, and marshalling its twenty arguments through ctypes took about 8 us, so
// the calls of a serving loop are converted here: tensors by their data_ptr(), a Segments object by
// its C structure, None as a null pointer, stream None as PyTorch's current stream.  Argument meaning
// and checks are those of include/lora.h; a non-zero status goes back to the Python wrapper, which
// raises.  The library's functions are handed over by address (bind), so that there is one copy of
// the library in the process.  Measured for one call of lora_build_apply_group with one projection and
// one kernel launch: 9.8 us through ctypes, 3.9 us here.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <stdint.h>

#include "../../include/lora.h"

namespace {

struct Library {
    decltype(&lora_build_segments) build_segments;
    decltype(&lora_apply) apply;
    decltype(&lora_apply_group) apply_group;
    decltype(&lora_build_apply_group) build_apply_group;
    decltype(&lora_moe_apply) moe_apply;
    decltype(&lora_moe_build_apply) moe_build_apply;
    decltype(&lora_moe_down_combine) moe_down_combine;
    decltype(&lora_pool_load_adapter_layer) load_adapter_layer;
} lib;

// Python-side helpers, set by bind(): the slow but always right way to a stream's handle, and, once
// torch has initialised the device, the two calls behind torch.cuda.current_stream().
PyObject *slow_stream, *current_device, *raw_stream;
PyObject *s_data_ptr, *s_numel, *s_element_size, *s_handle, *s_value, *s_c, *s_ws;

bool to_u64(PyObject *v, uint64_t &out)            // a Python int: an address or a size
{
    out = PyLong_AsUnsignedLongLongMask(v);
    return !(out == (uint64_t)-1 && PyErr_Occurred());
}

bool call_u64(PyObject *obj, PyObject *method, uint64_t &out)
{
    PyObject *r = PyObject_CallMethodNoArgs(obj, method);
    if (!r) return false;
    const bool ok = to_u64(r, out);
    Py_DECREF(r);
    return ok;
}

// device address of a tensor, an int or None
bool addr(PyObject *v, void *&out)
{
    uint64_t a = 0;
    if (v != Py_None && !(PyLong_Check(v) ? to_u64(v, a) : call_u64(v, s_data_ptr, a))) return false;
    out = reinterpret_cast<void *>(a);
    return true;
}

bool to_int(PyObject *v, int &out)
{
    const long x = PyLong_AsLong(v);
    if (x == -1 && PyErr_Occurred()) return false;
    if (x < INT32_MIN || x > INT32_MAX) {
        PyErr_SetString(PyExc_OverflowError, "argument does not fit a C int");
        return false;
    }
    out = (int)x;
    return true;
}

bool to_i64(PyObject *v, int64_t &out)
{
    out = PyLong_AsLongLong(v);
    return !(out == -1 && PyErr_Occurred());
}

bool pool_of(PyObject *v, lora_pool *&out)         // a Pool, a raw handle (int or ctypes pointer) or None
{
    uint64_t a = 0;
    if (v != Py_None) {
        if (PyLong_Check(v)) {
            if (!to_u64(v, a)) return false;
        } else {
            PyObject *h = PyObject_GetAttr(v, s_handle);
            if (!h && PyErr_ExceptionMatches(PyExc_AttributeError)) {      // a ctypes pointer
                PyErr_Clear();
                h = PyObject_GetAttr(v, s_value);
            }
            if (!h) return false;
            const bool ok = h == Py_None || to_u64(h, a);
            Py_DECREF(h);
            if (!ok) return false;
        }
    }
    out = reinterpret_cast<lora_pool *>(a);
    return true;
}

struct Held {                                       // a reference for as long as a call runs
    PyObject *obj = nullptr;
    ~Held() { Py_XDECREF(obj); }
};

// the lora_segments inside a Segments object (a ctypes structure, reached through the buffer protocol).
// `keep` holds the structure until the call is over: the object may hand out another one meanwhile
bool segments_of(PyObject *v, lora_segments *&out, Held &keep)
{
    keep.obj = PyObject_GetAttr(v, s_c);
    if (!keep.obj) return false;
    Py_buffer view;
    if (PyObject_GetBuffer(keep.obj, &view, PyBUF_WRITABLE) != 0) return false;
    out = static_cast<lora_segments *>(view.buf);
    const bool fits = view.len >= (Py_ssize_t)sizeof(lora_segments);
    PyBuffer_Release(&view);
    if (!fits) PyErr_SetString(PyExc_TypeError, "not a lora_segments structure");
    return fits;
}

bool bytes_of(PyObject *tensor, size_t &out)
{
    uint64_t n, e;
    if (!call_u64(tensor, s_numel, n) || !call_u64(tensor, s_element_size, e)) return false;
    out = (size_t)(n * e);
    return true;
}

// the segment builder's scratch inside a Segments object
bool seg_ws_of(PyObject *v, void *&ws, size_t &bytes)
{
    PyObject *t = PyObject_GetAttr(v, s_ws);
    if (!t) return false;
    uint64_t n;
    const bool ok = addr(t, ws) && call_u64(t, s_numel, n);
    if (ok) bytes = (size_t)n;
    Py_DECREF(t);
    return ok;
}

// workspace and its size; size None: the whole tensor
bool ws_of(PyObject *ws, PyObject *size, void *&p, size_t &bytes)
{
    if (!addr(ws, p)) return false;
    if (size == Py_None) return bytes_of(ws, bytes);
    uint64_t n;
    if (!to_u64(size, n)) return false;
    bytes = (size_t)n;
    return true;
}

bool stream_of(PyObject *v, void *&out)
{
    uint64_t a = 0;
    if (PyLong_Check(v)) {
        if (!to_u64(v, a)) return false;
        out = reinterpret_cast<void *>(a);
        return true;
    }
    PyObject *r;
    if (v == Py_None && raw_stream) {
        PyObject *dev = PyObject_CallNoArgs(current_device);
        if (!dev) return false;
        r = PyObject_CallOneArg(raw_stream, dev);
        Py_DECREF(dev);
    } else {
        r = PyObject_CallOneArg(slow_stream, v);
    }
    if (!r) return false;
    const bool ok = r == Py_None || to_u64(r, a);
    Py_DECREF(r);
    out = reinterpret_cast<void *>(a);
    return ok;
}

struct Outputs {                                    // y and ldy of a group
    void *y[LORA_MAX_PROJ];
    int64_t ld[LORA_MAX_PROJ];
    int n;
};

bool outputs_of(PyObject *ys, PyObject *lds, Outputs &o)
{
    PyObject *a = PySequence_Fast(ys, "outputs: a sequence is needed");
    if (!a) return false;
    PyObject *b = PySequence_Fast(lds, "row strides: a sequence is needed");
    if (!b) {
        Py_DECREF(a);
        return false;
    }
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(a);
    bool ok = true;
    if (PySequence_Fast_GET_SIZE(b) > n) {
        PyErr_SetString(PyExc_IndexError, "more row strides than outputs");
        ok = false;
    }
    o.n = (int)n;                                   // a count the library refuses is passed on as it is
    for (Py_ssize_t j = 0; ok && j < n && j < LORA_MAX_PROJ; ++j) {
        ok = addr(PySequence_Fast_GET_ITEM(a, j), o.y[j]);
        o.ld[j] = 0;                                // a missing stride counts as zero, which the library refuses
        if (ok && j < PySequence_Fast_GET_SIZE(b)) {
            PyObject *ld = PyNumber_Long(PySequence_Fast_GET_ITEM(b, j));
            ok = ld && to_i64(ld, o.ld[j]);
            Py_XDECREF(ld);
        }
    }
    Py_DECREF(a);
    Py_DECREF(b);
    return ok;
}

bool n_args(Py_ssize_t got, Py_ssize_t want)
{
    if (got == want) return true;
    PyErr_Format(PyExc_TypeError, "%zd arguments, %zd expected", got, want);
    return false;
}

#define LORA_PY(name) PyObject *name(PyObject *, PyObject *const *a, Py_ssize_t n)
#define LORA_CALL(expr)                 \
    int rc;                             \
    Py_BEGIN_ALLOW_THREADS              \
    rc = (expr);                        \
    Py_END_ALLOW_THREADS                \
    return PyLong_FromLong(rc)

// pool, adapter_id, expert_id, P, seg, stream
LORA_PY(build_segments)
{
    lora_pool *pool;
    void *aid, *eid, *sws, *st;
    int P;
    size_t sbytes;
    lora_segments *seg;
    Held seg_ref;
    if (!n_args(n, 6) || !pool_of(a[0], pool) || !addr(a[1], aid) || !addr(a[2], eid) || !to_int(a[3], P) ||
        !segments_of(a[4], seg, seg_ref) || !seg_ws_of(a[4], sws, sbytes) || !stream_of(a[5], st))
        return nullptr;
    LORA_CALL(lib.build_segments(pool, (const int32_t *)aid, (const int32_t *)eid, P, seg, sws, sbytes, st));
}

// pool, layer, proj, x, ldx, src_row, seg, y, ldy, v, out_dtype, stream
LORA_PY(apply)
{
    lora_pool *pool;
    int layer, proj, dt;
    void *x, *src, *y, *v, *st;
    int64_t ldx, ldy;
    lora_segments *seg;
    Held seg_ref;
    if (!n_args(n, 12) || !pool_of(a[0], pool) || !to_int(a[1], layer) || !to_int(a[2], proj) || !addr(a[3], x) ||
        !to_i64(a[4], ldx) || !addr(a[5], src) || !segments_of(a[6], seg, seg_ref) || !addr(a[7], y) || !to_i64(a[8], ldy) ||
        !addr(a[9], v) || !to_int(a[10], dt) || !stream_of(a[11], st))
        return nullptr;
    LORA_CALL(lib.apply(pool, layer, proj, x, ldx, (const int32_t *)src, seg, y, ldy, dt, (float *)v, st));
}

// pool, layer, proj0, x, ldx, src_row, seg, ys, ldys, ws, out_dtype, stream
LORA_PY(apply_group)
{
    lora_pool *pool;
    int layer, proj0, dt;
    void *x, *src, *ws, *st;
    int64_t ldx;
    size_t bytes;
    lora_segments *seg;
    Held seg_ref;
    Outputs o;
    if (!n_args(n, 12) || !pool_of(a[0], pool) || !to_int(a[1], layer) || !to_int(a[2], proj0) || !addr(a[3], x) ||
        !to_i64(a[4], ldx) || !addr(a[5], src) || !segments_of(a[6], seg, seg_ref) || !outputs_of(a[7], a[8], o) ||
        !ws_of(a[9], Py_None, ws, bytes) || !to_int(a[10], dt) || !stream_of(a[11], st))
        return nullptr;
    LORA_CALL(lib.apply_group(pool, layer, proj0, o.n, x, ldx, (const int32_t *)src, seg, o.y, o.ld, dt, ws, bytes, st));
}

// pool, layer, proj0, x, ldx, src_row, adapter_id, expert_id, P, seg, ys, ldys, ws, out_dtype, stream
LORA_PY(build_apply_group)
{
    lora_pool *pool;
    int layer, proj0, P, dt;
    void *x, *src, *aid, *eid, *sws, *ws, *st;
    int64_t ldx;
    size_t sbytes, bytes;
    lora_segments *seg;
    Held seg_ref;
    Outputs o;
    if (!n_args(n, 15) || !pool_of(a[0], pool) || !to_int(a[1], layer) || !to_int(a[2], proj0) || !addr(a[3], x) ||
        !to_i64(a[4], ldx) || !addr(a[5], src) || !addr(a[6], aid) || !addr(a[7], eid) || !to_int(a[8], P) ||
        !segments_of(a[9], seg, seg_ref) || !seg_ws_of(a[9], sws, sbytes) || !outputs_of(a[10], a[11], o) ||
        !ws_of(a[12], Py_None, ws, bytes) || !to_int(a[13], dt) || !stream_of(a[14], st))
        return nullptr;
    LORA_CALL(lib.build_apply_group(pool, layer, proj0, o.n, x, ldx, (const int32_t *)src, (const int32_t *)aid,
                                    (const int32_t *)eid, P, seg, sws, sbytes, o.y, o.ld, dt, ws, bytes, st));
}

// pool, layer, which, inp, ld_in, token_of_pair, seg, y0, y1, ldy, ws, ws_bytes, stream
LORA_PY(moe_apply)
{
    lora_pool *pool;
    int layer, which;
    void *in, *tok, *y0, *y1, *ws, *st;
    int64_t ld, ldy;
    size_t bytes;
    lora_segments *seg;
    Held seg_ref;
    if (!n_args(n, 13) || !pool_of(a[0], pool) || !to_int(a[1], layer) || !to_int(a[2], which) || !addr(a[3], in) ||
        !to_i64(a[4], ld) || !addr(a[5], tok) || !segments_of(a[6], seg, seg_ref) || !addr(a[7], y0) || !addr(a[8], y1) ||
        !to_i64(a[9], ldy) || !ws_of(a[10], a[11], ws, bytes) || !stream_of(a[12], st))
        return nullptr;
    LORA_CALL(lib.moe_apply(pool, layer, which, in, ld, (const int32_t *)tok, seg, y0, y1, ldy, ws, bytes, st));
}

// pool, layer, which, inp, ld_in, token_of_pair, adapter_id, expert_id, P, seg, y0, y1, ldy, ws, ws_bytes, stream
LORA_PY(moe_build_apply)
{
    lora_pool *pool;
    int layer, which, P;
    void *in, *tok, *aid, *eid, *sws, *y0, *y1, *ws, *st;
    int64_t ld, ldy;
    size_t sbytes, bytes;
    lora_segments *seg;
    Held seg_ref;
    if (!n_args(n, 16) || !pool_of(a[0], pool) || !to_int(a[1], layer) || !to_int(a[2], which) || !addr(a[3], in) ||
        !to_i64(a[4], ld) || !addr(a[5], tok) || !addr(a[6], aid) || !addr(a[7], eid) || !to_int(a[8], P) ||
        !segments_of(a[9], seg, seg_ref) || !seg_ws_of(a[9], sws, sbytes) || !addr(a[10], y0) || !addr(a[11], y1) ||
        !to_i64(a[12], ldy) || !ws_of(a[13], a[14], ws, bytes) || !stream_of(a[15], st))
        return nullptr;
    LORA_CALL(lib.moe_build_apply(pool, layer, which, in, ld, (const int32_t *)tok, (const int32_t *)aid,
                                  (const int32_t *)eid, P, seg, sws, sbytes, y0, y1, ldy, ws, bytes, st));
}

// pool, layer, hmid, ld_in, adapter_id, expert_id, seg, route_w, top_k, y_tok, ldy, ws, ws_bytes, stream
LORA_PY(moe_down_combine)
{
    lora_pool *pool;
    int layer, top_k;
    void *in, *aid, *eid, *w, *y, *ws, *st;
    int64_t ld, ldy;
    size_t bytes;
    lora_segments *seg;
    Held seg_ref;
    if (!n_args(n, 14) || !pool_of(a[0], pool) || !to_int(a[1], layer) || !addr(a[2], in) || !to_i64(a[3], ld) ||
        !addr(a[4], aid) || !addr(a[5], eid) || !segments_of(a[6], seg, seg_ref) || !addr(a[7], w) || !to_int(a[8], top_k) ||
        !addr(a[9], y) || !to_i64(a[10], ldy) || !ws_of(a[11], a[12], ws, bytes) || !stream_of(a[13], st))
        return nullptr;
    LORA_CALL(lib.moe_down_combine(pool, layer, in, ld, (const int32_t *)aid, (const int32_t *)eid, seg,
                                   (const float *)w, top_k, y, ldy, ws, bytes, st));
}

// pool, adapter, layer, src, stream
LORA_PY(load_adapter_layer)
{
    lora_pool *pool;
    int adapter, layer;
    void *src, *st;
    if (!n_args(n, 5) || !pool_of(a[0], pool) || !to_int(a[1], adapter) || !to_int(a[2], layer) || !addr(a[3], src) ||
        !stream_of(a[4], st))
        return nullptr;
    LORA_CALL(lib.load_adapter_layer(pool, adapter, layer, src, st));
}

// bind(addresses, stream function): the library's functions by name, and the binding's own way from a
// stream argument to its handle
LORA_PY(bind)
{
    if (!n_args(n, 2)) return nullptr;
    struct {
        const char *name;
        void **at;
    } const want[] = {
        {"lora_build_segments", (void **)&lib.build_segments},
        {"lora_apply", (void **)&lib.apply},
        {"lora_apply_group", (void **)&lib.apply_group},
        {"lora_build_apply_group", (void **)&lib.build_apply_group},
        {"lora_moe_apply", (void **)&lib.moe_apply},
        {"lora_moe_build_apply", (void **)&lib.moe_build_apply},
        {"lora_moe_down_combine", (void **)&lib.moe_down_combine},
        {"lora_pool_load_adapter_layer", (void **)&lib.load_adapter_layer},
    };
    for (const auto &w : want) {
        PyObject *v = PyMapping_GetItemString(a[0], w.name);
        if (!v) return nullptr;
        uint64_t p;
        const bool ok = to_u64(v, p) && p;
        Py_DECREF(v);
        if (!ok) {
            if (!PyErr_Occurred()) PyErr_Format(PyExc_ValueError, "no address for %s", w.name);
            return nullptr;
        }
        *w.at = reinterpret_cast<void *>(p);
    }
    Py_INCREF(a[1]);
    Py_XSETREF(slow_stream, a[1]);
    Py_RETURN_NONE;
}

// use_current_stream(current device, raw stream of a device): torch's calls, once it has initialised
// the device
LORA_PY(use_current_stream)
{
    if (!n_args(n, 2)) return nullptr;
    Py_INCREF(a[0]);
    Py_INCREF(a[1]);
    Py_XSETREF(current_device, a[0]);
    Py_XSETREF(raw_stream, a[1]);
    Py_RETURN_NONE;
}

#define LORA_METHOD(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    LORA_METHOD(bind), LORA_METHOD(use_current_stream), LORA_METHOD(build_segments), LORA_METHOD(apply),
    LORA_METHOD(apply_group), LORA_METHOD(build_apply_group), LORA_METHOD(moe_apply), LORA_METHOD(moe_build_apply),
    LORA_METHOD(moe_down_combine), LORA_METHOD(load_adapter_layer), {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pycall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pycall(void)
{
    struct {
        PyObject **at;
        const char *text;
    } const names[] = {{&s_data_ptr, "data_ptr"}, {&s_numel, "numel"}, {&s_element_size, "element_size"},
                       {&s_handle, "handle"}, {&s_value, "value"}, {&s_c, "c"}, {&s_ws, "ws"}};
    for (const auto &v : names)
        if (!(*v.at = PyUnicode_InternFromString(v.text))) return nullptr;
    return PyModule_Create(&module);
}
