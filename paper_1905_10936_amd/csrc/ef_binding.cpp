// The step calls of libef from Python: tensors to pointers without a dozen Python calls each.
//
// A call whose arguments are what the binding's own checks (__init__.py) accept goes to the C entry point, and its error code
// comes back.  Anything else (another type, device, layout or size, a stream given) is answered with None: the caller
// then takes the path through ctypes, which words the error or knows what to do.
//
// A call of 2 to 5 us on the GPU is enqueued through ctypes in 4.9 us (update), 5.7 (server) and 6.8 (worker), from here in
// 3.3, 3.5 and 3.7, nearly all of it the launch.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <climits>
#include <cstdint>
#include <cstring>

#include "ef.h"

namespace {

// The entry points, as ctypes has loaded them (bind).
struct Entries {
    decltype(&ef_worker_step) worker_step;
    decltype(&ef_worker_step_sgd) worker_step_sgd;
    decltype(&ef_server_step) server_step;
    decltype(&ef_apply) apply;
    decltype(&ef_apply_wd) apply_wd;
    decltype(&ef_worker_step_fused) worker_step_fused;
    decltype(&ef_server_step_fused) server_step_fused;
    decltype(&ef_apply_fused) apply_fused;
    decltype(&ef_worker_step_state) worker_step_state;
    decltype(&ef_server_step_state) server_step_state;
    decltype(&ef_compressor_quality) compressor_quality;
} F;

// What a Plan or a State knows about itself, packed by Python (no bytes: it is closed).
struct PlanKey {
    ef_plan *plan;
    int64_t d, W, B, message;
};
struct StateKey {
    ef_state *state;
    int64_t n;
};

// Arguments one after the other; `ok` is false from the first one on that is not as expected.
class Args {
public:
    Args(PyObject *const *a, Py_ssize_t n, Py_ssize_t expected) : a_(a), ok(n == expected) {}

    template <class Key>
    Key key()
    {
        Key k;
        memset(&k, 0, sizeof k);
        PyObject *o = next();
        ok = ok && PyBytes_CheckExact(o) && PyBytes_GET_SIZE(o) == (Py_ssize_t)sizeof k;
        if (ok) memcpy(&k, PyBytes_AS_STRING(o), sizeof k);
        return k;
    }
    // a contiguous tensor on the GPU
    const at::Tensor *tensor()
    {
        PyObject *o = next();
        ok = ok && THPVariable_CheckExact(o);
        if (!ok) return nullptr;
        const at::Tensor &t = THPVariable_Unpack(o);
        ok = t.defined() && t.is_cuda() && t.is_contiguous();
        return ok ? &t : nullptr;
    }
    const at::Tensor *tensor(at::ScalarType type)
    {
        const at::Tensor *t = tensor();
        ok = ok && t->scalar_type() == type;
        return t;
    }
    const at::Tensor *floats() { return tensor(at::kFloat); }
    float number()
    {
        PyObject *o = next();
        ok = ok && (PyFloat_Check(o) || PyLong_Check(o));
        const double v = ok ? PyFloat_AsDouble(o) : 0.0;
        ok = ok && !PyErr_Occurred();
        return (float)v;
    }
    int count()
    {
        PyObject *o = next();
        ok = ok && PyLong_Check(o);
        const long long v = ok ? PyLong_AsLongLong(o) : 0;
        ok = ok && !PyErr_Occurred() && v >= INT_MIN && v <= INT_MAX;
        return (int)v;
    }
    void *stream()
    {
        ok = ok && next() == Py_None;
        return ok ? (void *)c10::hip::getCurrentHIPStream().stream() : nullptr;
    }
    void need(bool condition) { ok = ok && condition; }

private:
    PyObject *next() { return ok ? a_[i_++] : Py_None; }
    PyObject *const *a_;
    Py_ssize_t i_ = 0;

public:
    bool ok;
};

int64_t rows(const at::Tensor &t) { return t.dim() == 1 ? 1 : t.size(0); }
bool has_rows(const at::Tensor &t) { return (t.dim() == 1 || t.dim() == 2) && rows(t) <= INT_MAX; }
int64_t stride(const at::Tensor &t) { return t.dim() == 1 ? t.numel() : t.stride(0); }
float *f32(const at::Tensor *t) { return static_cast<float *>(t->data_ptr()); }
uint64_t *words(const at::Tensor *t) { return static_cast<uint64_t *>(t->data_ptr()); }

// body(args) makes the call if args.ok, and returns its code.
template <class Body>
PyObject *call(PyObject *const *a, Py_ssize_t n, Py_ssize_t expected, Body body)
{
    int rc = EF_OK;
    bool ok = false;
    try {
        Args x(a, n, expected);
        rc = body(x);
        ok = x.ok;
    } catch (...) {
        ok = false;
    }
    if (!ok) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    return PyLong_FromLong(rc);
}

// The C call itself, without the interpreter's lock, as ctypes makes it.
template <class Call>
int unlocked(Call c)
{
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = c();
    Py_END_ALLOW_THREADS
    return rc;
}

PyObject *worker_step(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return call(a, n, 10, [](Args &x) {
        const PlanKey k = x.key<PlanKey>();
        const at::Tensor *g = x.floats(), *m = x.floats(), *e = x.floats();
        const float mu = x.number(), eta_prev = x.number(), eta = x.number();
        const at::Tensor *signs = x.tensor(), *scales = x.floats();
        void *s = x.stream();
        if (!x.ok) return 0;
        x.need(has_rows(*g) && has_rows(*m) && has_rows(*e));
        if (!x.ok) return 0;
        const int64_t nw = rows(*g);
        x.need(stride(*m) == stride(*e) && m->sizes() == e->sizes() && signs->numel() == nw * k.W && scales->numel() == nw * k.B);
        if (!x.ok) return 0;
        const float *gp = f32(g);
        float *mp = f32(m), *ep = f32(e), *cp = f32(scales);
        uint64_t *wp = words(signs);
        const int64_t gs = stride(*g), ss = stride(*m);
        return unlocked([&] { return F.worker_step(k.plan, (int)nw, gp, gs, mp, ep, ss, mu, eta_prev, eta, wp, cp, s); });
    });
}

PyObject *worker_step_sgd(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return call(a, n, 8, [](Args &x) {
        const PlanKey k = x.key<PlanKey>();
        const at::Tensor *g = x.floats(), *e = x.floats();
        const float eta_prev = x.number(), eta = x.number();
        const at::Tensor *signs = x.tensor(), *scales = x.floats();
        void *s = x.stream();
        if (!x.ok) return 0;
        x.need(has_rows(*g) && has_rows(*e));
        if (!x.ok) return 0;
        const int64_t nw = rows(*g);
        x.need(signs->numel() == nw * k.W && scales->numel() == nw * k.B);
        if (!x.ok) return 0;
        const float *gp = f32(g);
        float *ep = f32(e), *cp = f32(scales);
        uint64_t *wp = words(signs);
        const int64_t gs = stride(*g), ss = stride(*e);
        return unlocked([&] { return F.worker_step_sgd(k.plan, (int)nw, gp, gs, ep, ss, eta_prev, eta, wp, cp, s); });
    });
}

PyObject *worker_step_fused(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return call(a, n, 9, [](Args &x) {
        const PlanKey k = x.key<PlanKey>();
        const at::Tensor *g = x.floats(), *m = x.floats(), *e = x.floats();
        const float mu = x.number(), eta_prev = x.number(), eta = x.number();
        const at::Tensor *messages = x.tensor(at::kByte);
        void *s = x.stream();
        if (!x.ok) return 0;
        x.need(has_rows(*g) && has_rows(*m) && has_rows(*e));
        if (!x.ok) return 0;
        const int64_t nw = rows(*g);
        x.need(stride(*m) == stride(*e) && m->sizes() == e->sizes() && messages->numel() == nw * k.message);
        if (!x.ok) return 0;
        const float *gp = f32(g);
        float *mp = f32(m), *ep = f32(e);
        void *out = messages->data_ptr();
        const int64_t gs = stride(*g), ss = stride(*m);
        return unlocked([&] { return F.worker_step_fused(k.plan, (int)nw, gp, gs, mp, ep, ss, mu, eta_prev, eta, out, s); });
    });
}

PyObject *worker_step_state(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return call(a, n, 9, [](Args &x) {
        const PlanKey k = x.key<PlanKey>();
        const StateKey st = x.key<StateKey>();
        const at::Tensor *g = x.floats();
        const float mu = x.number(), eta_prev = x.number(), eta = x.number();
        const at::Tensor *signs = x.tensor(), *scales = x.floats();
        void *s = x.stream();
        if (!x.ok) return 0;
        x.need(has_rows(*g) && rows(*g) == st.n && signs->numel() == st.n * k.W && scales->numel() == st.n * k.B);
        if (!x.ok) return 0;
        const float *gp = f32(g);
        float *cp = f32(scales);
        uint64_t *wp = words(signs);
        const int64_t gs = stride(*g);
        return unlocked([&] { return F.worker_step_state(k.plan, st.state, gp, gs, mu, eta_prev, eta, wp, cp, s); });
    });
}

PyObject *server_step(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return call(a, n, 10, [](Args &x) {
        const PlanKey k = x.key<PlanKey>();
        const int M = x.count();
        const at::Tensor *signs = x.tensor(), *scales = x.floats(), *err = x.floats();
        const float eta_prev = x.number(), eta = x.number();
        const at::Tensor *out_signs = x.tensor(), *out_scales = x.floats();
        void *s = x.stream();
        if (!x.ok) return 0;
        x.need(signs->numel() == M * k.W && scales->numel() == M * k.B && err->numel() == k.d && out_signs->numel() == k.W &&
               out_scales->numel() == k.B);
        if (!x.ok) return 0;
        const uint64_t *wp = words(signs);
        const float *cp = f32(scales);
        float *ep = f32(err), *oc = f32(out_scales);
        uint64_t *ow = words(out_signs);
        return unlocked([&] { return F.server_step(k.plan, M, wp, cp, ep, eta_prev, eta, ow, oc, s); });
    });
}

PyObject *server_step_state(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return call(a, n, 10, [](Args &x) {
        const PlanKey k = x.key<PlanKey>();
        const StateKey st = x.key<StateKey>();
        const int M = x.count();
        const at::Tensor *signs = x.tensor(), *scales = x.floats();
        const float eta_prev = x.number(), eta = x.number();
        const at::Tensor *out_signs = x.tensor(), *out_scales = x.floats();
        void *s = x.stream();
        if (!x.ok) return 0;
        x.need(signs->numel() == M * k.W && scales->numel() == M * k.B && out_signs->numel() == k.W && out_scales->numel() == k.B);
        if (!x.ok) return 0;
        const uint64_t *wp = words(signs);
        const float *cp = f32(scales);
        float *oc = f32(out_scales);
        uint64_t *ow = words(out_signs);
        return unlocked([&] { return F.server_step_state(k.plan, st.state, M, wp, cp, eta_prev, eta, ow, oc, s); });
    });
}

PyObject *server_step_fused(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return call(a, n, 8, [](Args &x) {
        const PlanKey k = x.key<PlanKey>();
        const int M = x.count();
        const at::Tensor *messages = x.tensor(at::kByte), *err = x.floats();
        const float eta_prev = x.number(), eta = x.number();
        const at::Tensor *out = x.tensor(at::kByte);
        void *s = x.stream();
        if (!x.ok) return 0;
        x.need(messages->numel() >= M * k.message && err->numel() == k.d && out->numel() == k.message);
        if (!x.ok) return 0;
        const void *in = messages->data_ptr();
        float *ep = f32(err);
        void *op = out->data_ptr();
        return unlocked([&] { return F.server_step_fused(k.plan, M, in, ep, eta_prev, eta, op, s); });
    });
}

PyObject *apply(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return call(a, n, 6, [](Args &x) {
        const PlanKey k = x.key<PlanKey>();
        const at::Tensor *params = x.floats(), *signs = x.tensor(), *scales = x.floats();
        const float eta = x.number();
        void *s = x.stream();
        if (!x.ok) return 0;
        x.need(params->numel() == k.d && signs->numel() == k.W && scales->numel() == k.B);
        if (!x.ok) return 0;
        float *xp = f32(params);
        const uint64_t *wp = words(signs);
        const float *cp = f32(scales);
        return unlocked([&] { return F.apply(k.plan, xp, wp, cp, eta, s); });
    });
}

PyObject *apply_wd(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return call(a, n, 9, [](Args &x) {
        const PlanKey k = x.key<PlanKey>();
        const at::Tensor *params = x.floats(), *decay = x.floats(), *signs = x.tensor(), *scales = x.floats();
        const float eta = x.number(), mu = x.number(), lam = x.number();
        void *s = x.stream();
        if (!x.ok) return 0;
        x.need(params->numel() == k.d && decay->numel() == k.d && signs->numel() == k.W && scales->numel() == k.B);
        if (!x.ok) return 0;
        float *xp = f32(params), *mp = f32(decay);
        const uint64_t *wp = words(signs);
        const float *cp = f32(scales);
        return unlocked([&] { return F.apply_wd(k.plan, xp, mp, wp, cp, eta, mu, lam, s); });
    });
}

PyObject *apply_fused(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return call(a, n, 5, [](Args &x) {
        const PlanKey k = x.key<PlanKey>();
        const at::Tensor *params = x.floats(), *message = x.tensor(at::kByte);
        const float eta = x.number();
        void *s = x.stream();
        if (!x.ok) return 0;
        x.need(params->numel() == k.d && message->numel() == k.message);
        if (!x.ok) return 0;
        float *xp = f32(params);
        const void *in = message->data_ptr();
        return unlocked([&] { return F.apply_fused(k.plan, xp, in, eta, s); });
    });
}

PyObject *compressor_quality(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return call(a, n, 4, [](Args &x) {
        const PlanKey k = x.key<PlanKey>();
        const at::Tensor *v = x.floats(), *out = x.tensor(at::kDouble);
        void *s = x.stream();
        if (!x.ok) return 0;
        x.need(has_rows(*v) && out->numel() == 2 * rows(*v));
        if (!x.ok) return 0;
        const float *vp = f32(v);
        double *op = static_cast<double *>(out->data_ptr());
        const int nv = (int)rows(*v);
        const int64_t vs = stride(*v);
        return unlocked([&] { return F.compressor_quality(k.plan, nv, vp, vs, op, s); });
    });
}

// bind(addresses): the entry points' addresses, in the order of Entries.
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    constexpr Py_ssize_t count = sizeof(Entries) / sizeof(void *);
    void *p[count];
    if (n != count) {
        PyErr_SetString(PyExc_TypeError, "bind: one address for each entry point");
        return nullptr;
    }
    for (Py_ssize_t i = 0; i < count; ++i) {
        p[i] = PyLong_AsVoidPtr(a[i]);
        if (!p[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "bind: null address");
            return nullptr;
        }
    }
    memcpy(&F, p, sizeof F);
    Py_RETURN_NONE;
}

#define EF_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {EF_METHOD(bind),
                         EF_METHOD(worker_step),
                         EF_METHOD(worker_step_sgd),
                         EF_METHOD(worker_step_fused),
                         EF_METHOD(worker_step_state),
                         EF_METHOD(server_step),
                         EF_METHOD(server_step_state),
                         EF_METHOD(server_step_fused),
                         EF_METHOD(apply),
                         EF_METHOD(apply_wd),
                         EF_METHOD(apply_fused),
                         EF_METHOD(compressor_quality),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_ef_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__ef_binding(void)
{
    PyObject *m = PyModule_Create(&module);
    // what the loader asks for before it binds any entry point
    if (m && PyModule_AddStringConstant(m, "built_for", EF_BUILT_FOR) < 0) Py_CLEAR(m);
    return m;
}
