// Native half of the Python binding: checks tensors, gathers their device pointers and makes the library call.
//
// Why it exists: a data-parallel worker hands over 2P block pointers per layer and step.  Checking and collecting
// them in Python took 9-15 us per call, several times what the smaller kernels run for, so the GPU waited for the
// host (1024 -> 1000 layer, B = 32, P = 8: 42 us per pass for 19 us of kernels).  Here the same checks cost about
// 20 ns per tensor.  Everything that is not marshalling stays in the library.  A tensor that does not fit is a ValueError, an
// argument of the wrong kind (a structure above all) a TypeError.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/DynamicTypes.h>
#include <torch/csrc/autograd/python_variable.h>
#include "psd.h"

namespace {

// The binding's ctypes classes, handed over by bind() when it loads this module, and kept for good.
struct Classes { PyObject *plan, *ssp_state, *segment, *task, *void_p; } classes;

// A ctypes structure or array, looked at through the buffer protocol for the length of one call.
struct View {
    Py_buffer b{};
    bool held = false;
    template <class T> T* as() const { return static_cast<T*>(b.buf); }
    ~View() { if (held) PyBuffer_Release(&b); }

    bool open(PyObject* o, int flags) { return held = PyObject_GetBuffer(o, &b, flags) == 0; }
    // an instance of a structure class
    bool open_struct(PyObject* o, PyObject* type, size_t bytes, const char* what, int flags = PyBUF_SIMPLE)
    {
        if (!type || !PyObject_TypeCheck(o, reinterpret_cast<PyTypeObject*>(type))) return refuse(o, what);
        return open(o, flags) && (b.len >= static_cast<Py_ssize_t>(bytes) || refuse(o, what));
    }
    // an array of at least `count` elements of a class
    bool open_array(PyObject* o, PyObject* type, int64_t count, size_t bytes, const char* what)
    {
        PyObject* element = PyObject_GetAttrString(reinterpret_cast<PyObject*>(Py_TYPE(o)), "_type_");
        PyErr_Clear();
        Py_XDECREF(element);                       // (borrowed from the type from here on)
        if (!element || element != type) return refuse(o, what);
        return open(o, PyBUF_SIMPLE) && (b.len / static_cast<int64_t>(bytes) >= count || refuse(o, what));
    }
    bool refuse(PyObject* o, const char* what)
    {
        PyErr_Format(PyExc_TypeError, "%s expected, not %s", what, Py_TYPE(o)->tp_name);
        return false;
    }
};

bool plan_of(PyObject* o, View& v) { return v.open_struct(o, classes.plan, sizeof(psd_plan), "a Plan"); }

bool type_ok(c10::ScalarType t, long factor_dtype)
{
    if (factor_dtype == PSD_F32) return t == c10::kFloat;
    if (factor_dtype == PSD_BF16) return t == c10::kBFloat16 || t == c10::kShort || t == c10::kUInt16;
    return false;
}

// Device pointer of a tensor that can hold what the kernel will touch; false with ValueError set if it cannot.
// index >= 0 names an element of a list in the error text.
template <class T>
bool dev_ptr(PyObject* o, long factor_dtype, int64_t min_elems, const char* what, T** out, Py_ssize_t index = -1)
{
    char name[64];
    auto called = [&]() {
        if (index < 0) snprintf(name, sizeof name, "%s", what);
        else snprintf(name, sizeof name, "%s[%zd]", what, index);
        return name;
    };
    if (!THPVariable_Check(o)) {
        PyErr_Format(PyExc_ValueError, "%s must be a contiguous CUDA tensor", called());
        return false;
    }
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_cuda() || !t.is_contiguous()) {
        PyErr_Format(PyExc_ValueError, "%s must be a contiguous CUDA tensor", called());
        return false;
    }
    if (!type_ok(t.scalar_type(), factor_dtype)) {
        PyErr_Format(PyExc_ValueError, "%s has dtype %S", called(), reinterpret_cast<PyObject*>(torch::getTHPDtype(t.scalar_type())));
        return false;
    }
    if (t.numel() < min_elems) {
        PyErr_Format(PyExc_ValueError, "%s holds %lld elements, needs %lld", called(), static_cast<long long>(t.numel()),
                     static_cast<long long>(min_elems));
        return false;
    }
    *out = static_cast<T*>(t.data_ptr());
    return true;
}

// A sequence of tensors, held until the library has been called: a caller's sequence may make its tensors as it is read.
class Tensors {
    PyObject* held = nullptr;

public:
    Tensors() = default;
    Tensors(const Tensors&) = delete;
    ~Tensors() { Py_XDECREF(held); }
    Py_ssize_t count() const { return PyTuple_GET_SIZE(held); }

    // All are checked, the pointers of the first `room` are stored (the library refuses longer lists by their count); false
    // with an exception set if one does not fit.
    bool take(PyObject* seq, long factor_dtype, int64_t min_elems, const char* what, const void** out, Py_ssize_t room)
    {
        if (PyObject_Size(seq) < 0) return false;        // an iterator is no sequence
        held = PySequence_Tuple(seq);
        if (!held) return false;
        for (Py_ssize_t i = 0; i < count(); ++i) {
            const void* p = nullptr;
            if (!dev_ptr(PyTuple_GET_ITEM(held, i), factor_dtype, min_elems, what, &p, i)) return false;
            if (i < room) out[i] = p;
        }
        return true;
    }
};

// None: the current stream of the current device; an int: a raw handle; else an object with .cuda_stream
bool stream_of(PyObject* o, void** out)
{
    if (o == Py_None) {
        *out = c10::hip::getCurrentHIPStream().stream();
        return true;
    }
    if (PyLong_Check(o)) {
        *out = PyLong_AsVoidPtr(o);
        return !PyErr_Occurred();
    }
    PyObject* h = PyObject_GetAttrString(o, "cuda_stream");
    if (!h) return false;
    *out = PyLong_AsVoidPtr(h);
    Py_DECREF(h);
    return !PyErr_Occurred();
}

bool workspace_of(PyObject* o, void** p, size_t* bytes)
{
    *p = nullptr;
    *bytes = 0;
    if (o == Py_None) return true;
    if (!THPVariable_Check(o) || !THPVariable_Unpack(o).is_cuda() || !THPVariable_Unpack(o).is_contiguous()) {
        PyErr_SetString(PyExc_ValueError, "workspace must be a contiguous CUDA tensor");
        return false;
    }
    const at::Tensor& t = THPVariable_Unpack(o);
    *p = t.data_ptr();
    *bytes = t.nbytes();
    return true;
}

int64_t as_i64(PyObject* o) { return PyLong_AsLongLong(o); }
float as_f32(PyObject* o) { return static_cast<float>(PyFloat_AsDouble(o)); }

bool arity(Py_ssize_t got, Py_ssize_t want)
{
    if (got == want) return true;
    PyErr_Format(PyExc_TypeError, "%zd arguments, %zd wanted", got, want);
    return false;
}

template <class F>
PyObject* call(F f)
{
    psd_status r;
    Py_BEGIN_ALLOW_THREADS
    r = f();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(r);
}

bool need_P_blocks()
{
    PyErr_SetString(PyExc_ValueError, "need P per-worker blocks");
    return false;
}

// the P error and P activation blocks of a layer: `eu`, `ev` elements each at least
struct Blocks {
    const void* u[PSD_MAX_WORKERS];
    const void* v[PSD_MAX_WORKERS];
    Tensors tu, tv;

    bool take_u(PyObject* us, const psd_plan& plan, long dtype, int64_t eu, const char* name)
    {
        return tu.take(us, dtype, eu, name, u, PSD_MAX_WORKERS) && (tu.count() == plan.P || need_P_blocks());
    }
    bool take_v(PyObject* vs, const psd_plan& plan, long dtype, int64_t ev, const char* name)
    {
        return tv.take(vs, dtype, ev, name, v, PSD_MAX_WORKERS) && (tv.count() == plan.P || need_P_blocks());
    }
    bool take(PyObject* us, PyObject* vs, const psd_plan& plan, long dtype, int64_t eu, int64_t ev, const char* nu, const char* nv)
    {
        const Py_ssize_t n = PyObject_Size(us), m = n < 0 ? n : PyObject_Size(vs);
        if (n < 0 || m < 0) return false;
        if (n != plan.P || m != plan.P) return need_P_blocks();
        return take_u(us, plan, dtype, eu, nu) && take_v(vs, plan, dtype, ev, nv);
    }
};

const float* const* f32s(const void* const* p) { return reinterpret_cast<const float* const*>(p); }

// plan, delta, act, out_dtype, U, ldu, V, ldv, stream
PyObject* pack_factors(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    View pv;
    Blocks b;
    void* st;
    if (!arity(n, 9) || !plan_of(a[0], pv)) return nullptr;
    const psd_plan& plan = *pv.as<psd_plan>();
    if (!b.take(a[1], a[2], plan, PSD_F32, plan.B * plan.N, plan.B * plan.M, "delta", "act")) return nullptr;
    const long dt = PyLong_AsLong(a[3]);
    const int64_t ldu = as_i64(a[5]), ldv = as_i64(a[7]);
    if (PyErr_Occurred()) return nullptr;
    void *U, *V;
    if (!dev_ptr(a[4], dt, plan.P * plan.B * ldu, "U", &U) || !dev_ptr(a[6], dt, plan.P * plan.B * ldv, "V", &V) ||
        !stream_of(a[8], &st))
        return nullptr;
    return call([&] { return psd_pack_factors(&plan, f32s(b.u), f32s(b.v), dt, U, ldu, V, ldv, st); });
}

// plan, factor_dtype, U, ldu, V, ldv, W, Mom, lr, mu, wd, workspace (None, a tensor, or ... for the static array), stream
PyObject* sync_fc_sfb(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    View pv;
    void *st, *ws = nullptr;
    size_t ws_bytes = 0;
    if (!arity(n, 13) || !plan_of(a[0], pv)) return nullptr;
    const psd_plan& plan = *pv.as<psd_plan>();
    const long dt = PyLong_AsLong(a[1]);
    const int64_t ldu = as_i64(a[3]), ldv = as_i64(a[5]), K = plan.P * plan.B;
    const float lr = as_f32(a[8]), mu = as_f32(a[9]), wd = as_f32(a[10]);
    if (PyErr_Occurred()) return nullptr;
    void *U, *V;
    float *W, *Mom;
    if (!dev_ptr(a[2], dt, K * ldu, "U", &U) || !dev_ptr(a[4], dt, K * ldv, "V", &V) ||
        !dev_ptr(a[6], PSD_F32, plan.N * plan.M, "W", &W) ||
        !dev_ptr(a[7], PSD_F32, plan.N * plan.M, "Mom", &Mom))
        return nullptr;
    const bool use_static = a[11] == Py_Ellipsis;
    if ((!use_static && !workspace_of(a[11], &ws, &ws_bytes)) || !stream_of(a[12], &st)) return nullptr;
    return call([&] {
        return use_static ? psd_sync_fc_sfb_static(&plan, dt, U, ldu, V, ldv, W, Mom, lr, mu, wd, st)
                          : psd_sync_fc_sfb(&plan, dt, U, ldu, V, ldv, W, Mom, lr, mu, wd, ws, ws_bytes, st);
    });
}

// plan, factor_dtype, U_blocks, ldu, V_blocks, ldv, W, Mom, lr, mu, wd, stream
PyObject* sync_fc_sfb_blocks(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    View pv;
    Blocks b;
    void* st;
    if (!arity(n, 12) || !plan_of(a[0], pv)) return nullptr;
    const psd_plan& plan = *pv.as<psd_plan>();
    const long dt = PyLong_AsLong(a[1]);
    const int64_t ldu = as_i64(a[3]), ldv = as_i64(a[5]);
    const float lr = as_f32(a[8]), mu = as_f32(a[9]), wd = as_f32(a[10]);
    if (PyErr_Occurred() || !b.take(a[2], a[4], plan, dt, plan.B * ldu, plan.B * ldv, "U_blocks", "V_blocks")) return nullptr;
    float *W, *Mom;
    if (!dev_ptr(a[6], PSD_F32, plan.N * plan.M, "W", &W) ||
        !dev_ptr(a[7], PSD_F32, plan.N * plan.M, "Mom", &Mom) || !stream_of(a[11], &st))
        return nullptr;
    return call([&] { return psd_sync_fc_sfb_blocks(&plan, dt, b.u, ldu, b.v, ldv, W, Mom, lr, mu, wd, st); });
}

// plan, factor_dtype, U, ldu, bias, mom_bias, lr, mu, wd, stream
PyObject* sync_fc_bias(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    View pv;
    void* st;
    if (!arity(n, 10) || !plan_of(a[0], pv)) return nullptr;
    const psd_plan& plan = *pv.as<psd_plan>();
    const long dt = PyLong_AsLong(a[1]);
    const int64_t ldu = as_i64(a[3]);
    const float lr = as_f32(a[6]), mu = as_f32(a[7]), wd = as_f32(a[8]);
    if (PyErr_Occurred()) return nullptr;
    void* U;
    float *bias, *mom;
    if (!dev_ptr(a[2], dt, plan.P * plan.B * ldu, "U", &U) || !dev_ptr(a[4], PSD_F32, plan.N, "bias", &bias) ||
        !dev_ptr(a[5], PSD_F32, plan.N, "mom_bias", &mom) || !stream_of(a[9], &st))
        return nullptr;
    return call([&] { return psd_sync_fc_bias(&plan, dt, U, ldu, bias, mom, lr, mu, wd, st); });
}

// G, W, Mom, lr, mu, wd, S, stream
PyObject* sync_dense_ps(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    const void* g[PSD_MAX_WORKERS];
    Tensors G;
    void* st;
    if (!arity(n, 8) || PyObject_Size(a[0]) < 0) return nullptr;
    const float lr = as_f32(a[3]), mu = as_f32(a[4]), wd = as_f32(a[5]);
    const long S = PyLong_AsLong(a[6]);
    if (PyErr_Occurred()) return nullptr;
    float* W;
    if (!dev_ptr(a[1], PSD_F32, 0, "W", &W)) return nullptr;
    const int64_t keys = THPVariable_Unpack(a[1]).numel();
    float* Mom;
    if (!G.take(a[0], PSD_F32, keys, "G", g, PSD_MAX_WORKERS) ||
        !dev_ptr(a[2], PSD_F32, keys, "Mom", &Mom) || !stream_of(a[7], &st))
        return nullptr;
    return call([&] { return psd_sync_dense_ps(keys, static_cast<int32_t>(G.count()), f32s(g), W, Mom, lr, mu, wd, static_cast<int32_t>(S), st); });
}

// L, segments, lr, mu, wd, stream
PyObject* sync_dense_ps_multi(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    View sv;
    void* st;
    if (!arity(n, 6)) return nullptr;
    const long L = PyLong_AsLong(a[0]);
    if (PyErr_Occurred() || !sv.open_array(a[1], classes.segment, L, sizeof(psd_dense_segment), "an array of L DenseSegments")) return nullptr;
    const float lr = as_f32(a[2]), mu = as_f32(a[3]), wd = as_f32(a[4]);
    if (PyErr_Occurred() || !stream_of(a[5], &st)) return nullptr;
    return call([&] { return psd_sync_dense_ps_multi(static_cast<int32_t>(L), sv.as<psd_dense_segment>(), lr, mu, wd, st); });
}

// L, tasks, lr, mu, wd, rule
PyObject* sync_iteration(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    View tv;
    if (!arity(n, 6)) return nullptr;
    const long L = PyLong_AsLong(a[0]), rule = PyLong_AsLong(a[5]);
    if (PyErr_Occurred() || !tv.open_array(a[1], classes.task, L, sizeof(psd_layer_task), "an array of L LayerTasks")) return nullptr;
    const float lr = as_f32(a[2]), mu = as_f32(a[3]), wd = as_f32(a[4]);
    if (PyErr_Occurred()) return nullptr;
    return call([&] { return psd_sync_iteration(static_cast<int32_t>(L), tv.as<psd_layer_task>(), lr, mu, wd, static_cast<int32_t>(rule)); });
}

// state, plan, factor_dtype, delta (or None), act (or None), U_ring, ldu, V_ring, ldv, W, Mom, lr, mu, wd, workspace, stream
PyObject* ssp_clock_fc(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    View sv, pv, uv, vv;
    Blocks b;
    void *st, *ws;
    size_t ws_bytes;
    if (!arity(n, 16) || !sv.open_struct(a[0], classes.ssp_state, sizeof(psd_ssp_state), "an SspState", PyBUF_WRITABLE) ||
        !plan_of(a[1], pv))
        return nullptr;
    const psd_plan& plan = *pv.as<psd_plan>();
    const int64_t ring = int64_t(sv.as<psd_ssp_state>()->s) + 1;
    if (!uv.open_array(a[5], classes.void_p, ring, sizeof(void*), "an array of s + 1 pointers") ||
        !vv.open_array(a[7], classes.void_p, ring, sizeof(void*), "an array of s + 1 pointers"))
        return nullptr;
    const long dt = PyLong_AsLong(a[2]);
    const int64_t ldu = as_i64(a[6]), ldv = as_i64(a[8]);
    const float lr = as_f32(a[11]), mu = as_f32(a[12]), wd = as_f32(a[13]);
    if (PyErr_Occurred()) return nullptr;
    const bool du = a[3] != Py_None, dv = a[4] != Py_None;
    if ((du && !b.take_u(a[3], plan, PSD_F32, plan.B * plan.N, "delta")) || (dv && !b.take_v(a[4], plan, PSD_F32, plan.B * plan.M, "act")))
        return nullptr;
    float *W, *Mom;
    if (!dev_ptr(a[9], PSD_F32, plan.N * plan.M, "W", &W) ||
        !dev_ptr(a[10], PSD_F32, plan.N * plan.M, "Mom", &Mom) || !workspace_of(a[14], &ws, &ws_bytes) ||
        !stream_of(a[15], &st))
        return nullptr;
    return call([&] {
        return psd_ssp_clock_fc(sv.as<psd_ssp_state>(), &plan, dt, du ? f32s(b.u) : nullptr, dv ? f32s(b.v) : nullptr, uv.as<void*>(), ldu,
                                vv.as<void*>(), ldv, W, Mom, lr, mu, wd, ws, ws_bytes, st);
    });
}

// table (a ctypes array of pointers), tensors, factor_dtype, min_elems, what: fills the table
PyObject* fill_pointers(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    View tv;
    if (!arity(n, 5) || !tv.open(a[0], PyBUF_WRITABLE)) return nullptr;
    const long dt = PyLong_AsLong(a[2]);
    const int64_t least = as_i64(a[3]);
    const char* what = PyUnicode_AsUTF8(a[4]);
    Tensors t;
    if (PyErr_Occurred() || !what || !t.take(a[1], dt, least, what, tv.as<const void*>(), tv.b.len / static_cast<Py_ssize_t>(sizeof(void*))))
        return nullptr;
    Py_RETURN_NONE;
}

// tensor, factor_dtype, min_elems, what -> address
PyObject* pointer(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    if (!arity(n, 4)) return nullptr;
    const long dt = PyLong_AsLong(a[1]);
    const int64_t least = as_i64(a[2]);
    const char* what = PyUnicode_AsUTF8(a[3]);
    if (PyErr_Occurred() || !what) return nullptr;
    void* p;
    return dev_ptr(a[0], dt, least, what, &p) ? PyLong_FromVoidPtr(p) : nullptr;
}

// Plan, SspState, DenseSegment, LayerTask, c_void_p
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    if (!arity(n, 5)) return nullptr;
    for (Py_ssize_t i = 0; i < n; ++i)
        if (!PyType_Check(a[i])) {
            PyErr_SetString(PyExc_TypeError, "classes expected");
            return nullptr;
        }
    PyObject** to[] = {&classes.plan, &classes.ssp_state, &classes.segment, &classes.task, &classes.void_p};
    for (Py_ssize_t i = 0; i < n; ++i) {
        Py_INCREF(a[i]);
        Py_XSETREF(*to[i], a[i]);
    }
    Py_RETURN_NONE;
}

template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)>
PyObject* guarded(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    try {
        return F(self, a, n);
    } catch (const std::exception& e) {          // torch reports its own errors by throwing
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

#define PSD_METHOD(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(&guarded<f>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {PSD_METHOD(pack_factors), PSD_METHOD(sync_fc_sfb), PSD_METHOD(sync_fc_sfb_blocks), PSD_METHOD(sync_fc_bias),
                         PSD_METHOD(sync_dense_ps), PSD_METHOD(sync_dense_ps_multi), PSD_METHOD(sync_iteration),
                         PSD_METHOD(ssp_clock_fc), PSD_METHOD(fill_pointers), PSD_METHOD(pointer), PSD_METHOD(bind), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_psdpy", "argument marshalling of libpsd.so", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__psdpy(void) { return PyModule_Create(&module); }
