// The recurrent step's way from Python to osdn_step, for a call whose arguments are what they should be.
//
// A decode step of few sequences takes the device 4 us; checking eleven tensors, allocating two and marshalling fifteen
// arguments in Python took 12 (8 chains of 128 x 128, one token: 11.8 us a call, so 6.0).  Anything out of the
// ordinary (a subclass of Tensor, a torch function mode, another device, a wrong type, shape or layout, a value outside its field) is left
// to the Python code, which says what is wrong with it: then this returns None and has done nothing.
#include <Python.h>

#include <cfloat>
#include <climits>
#include <cmath>
#include <cstring>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <ATen/ops/empty_like.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/osdn.h"

namespace {

typedef int (*StepFn)(const osdn_params *, const void *, const void *, const void *, const float *, const float *, const float *,
                      const float *, const float *, void *, float *, float *, void *);
StepFn g_step = nullptr;
PyObject *g_names[10];       // interned: the fields of Hyper, in the order of HyperField
enum HyperField { SCALE, ETA, D_MIN, D_MAX, EPS, BETA_AWARE, SEGMENTS, P1_PIECES, P1_PIECE_SWEEPS, P1_SOLVED };
const char *const kNames[10] = {"scale", "eta", "d_min", "d_max", "eps", "beta_aware", "segments", "p1_pieces", "p1_piece_sweeps", "p1_solved"};

// a plain dense tensor of this type and shape on device `dev`
bool plain(const at::Tensor &t, at::ScalarType type, int64_t dev, at::IntArrayRef shape) {
    return t.is_cuda() && t.layout() == at::kStrided && t.has_storage() && t.scalar_type() == type && t.device().index() == dev &&
           t.sizes() == shape && t.is_contiguous();
}
bool as_float(PyObject *hp, int f, float &out) {
    PyObject *o = PyObject_GetAttr(hp, g_names[f]);
    if (!o) { PyErr_Clear(); return false; }
    const bool ok = PyFloat_CheckExact(o);
    const double x = ok ? PyFloat_AS_DOUBLE(o) : 0.0;
    Py_DECREF(o);
    if (!ok || (std::isfinite(x) && std::fabs(x) > FLT_MAX)) return false;
    out = (float)x;
    return true;
}
bool as_int(PyObject *hp, int f, int32_t &out) {
    PyObject *o = PyObject_GetAttr(hp, g_names[f]);
    if (!o) { PyErr_Clear(); return false; }
    int over = 0;
    const bool ok = PyLong_CheckExact(o) || PyBool_Check(o);
    const long x = ok ? PyLong_AsLongAndOverflow(o, &over) : 0;
    Py_DECREF(o);
    if (!ok || over || x < INT_MIN || x > INT_MAX) return false;
    out = (int32_t)x;
    return true;
}

// step(q, k, v, beta, log_alpha, retention, d_in, S_in, hp, in_place, device, stream): (o, S_out, d_out), the status
// of a call that failed, or None
PyObject *step(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (!g_step || n != 12 || at::impl::PythonTorchFunctionTLS::stack_len() > 0) Py_RETURN_NONE;
    const at::Tensor *t[8];
    for (int i = 0; i < 8; ++i) {
        t[i] = nullptr;
        if (a[i] == Py_None) {
            if (i < 4) Py_RETURN_NONE;
        } else if (THPVariable_CheckExact(a[i])) {
            t[i] = &THPVariable_Unpack(a[i]);
        } else {
            Py_RETURN_NONE;
        }
    }
    const at::Tensor &q = *t[0], &k = *t[1], &v = *t[2];
    const long dev = PyLong_AsLong(a[10]);
    void *stream = PyLong_AsVoidPtr(a[11]);
    if (PyErr_Occurred()) { PyErr_Clear(); Py_RETURN_NONE; }
    if (!PyBool_Check(a[9]) || k.dim() != 4 || v.dim() != 4) Py_RETURN_NONE;
    const int64_t B = k.size(0), T = k.size(1), H = k.size(2), K = k.size(3), V = v.size(3);
    for (int64_t x : {B, T, H, K, V})
        if (x > INT_MAX) Py_RETURN_NONE;
    const at::ScalarType io = k.scalar_type() == at::kBFloat16 ? at::kBFloat16 : at::kFloat, f32 = at::kFloat;
    const bool gate_vec = t[4] && t[4]->dim() == 4, ret_vec = t[5] && t[5]->dim() == 4;
    const int64_t bthk[] = {B, T, H, K}, bthv[] = {B, T, H, V}, bhvk[] = {B, H, V, K}, bhk[] = {B, H, K};
    const at::IntArrayRef th(bthk, 3), thk(bthk, 4);
    if (!plain(q, io, dev, thk) || !plain(k, io, dev, thk) || !plain(v, io, dev, at::IntArrayRef(bthv, 4)) || !plain(*t[3], f32, dev, th) ||
        (t[4] && !plain(*t[4], f32, dev, gate_vec ? thk : th)) || (t[5] && !plain(*t[5], f32, dev, ret_vec ? thk : th)) ||
        (t[6] && !plain(*t[6], f32, dev, at::IntArrayRef(bhk, 3))) || (t[7] && !plain(*t[7], f32, dev, at::IntArrayRef(bhvk, 4))))
        Py_RETURN_NONE;
    osdn_params p{};
    p.B = (int32_t)B; p.T = (int32_t)T; p.H = (int32_t)H; p.K = (int32_t)K; p.V = (int32_t)V; p.chunk = 64;
    p.io_dtype = io == at::kBFloat16 ? OSDN_BF16 : OSDN_F32;
    PyObject *hp = a[8], *scale = PyObject_GetAttr(hp, g_names[SCALE]);
    if (!scale) { PyErr_Clear(); Py_RETURN_NONE; }
    const bool no_scale = scale == Py_None;
    Py_DECREF(scale);
    if (no_scale) p.scale = (float)std::pow((double)K, -0.5);
    else if (!as_float(hp, SCALE, p.scale)) Py_RETURN_NONE;
    if (!as_float(hp, ETA, p.eta) || !as_float(hp, D_MIN, p.d_min) || !as_float(hp, D_MAX, p.d_max) || !as_float(hp, EPS, p.eps) ||
        !as_int(hp, BETA_AWARE, p.beta_aware) || !as_int(hp, SEGMENTS, p.segments) || !as_int(hp, P1_PIECES, p.p1_pieces) ||
        !as_int(hp, P1_PIECE_SWEEPS, p.p1_piece_sweeps) || !as_int(hp, P1_SOLVED, p.p1_solved))
        Py_RETURN_NONE;
    p.retention_per_channel = ret_vec;
    p.gate_per_channel = gate_vec;

    const at::TensorOptions f32_on = k.options().dtype(f32);
    const bool in_place = a[9] == Py_True && t[7];
    at::Tensor o = at::empty_like(v), d = at::empty(at::IntArrayRef(bhk, 3), f32_on);
    at::Tensor S = in_place ? *t[7] : at::empty(at::IntArrayRef(bhvk, 4), f32_on);
    auto ptr = [](const at::Tensor *x) { return x ? static_cast<const float *>(x->data_ptr()) : nullptr; };
    const void *qp = q.data_ptr(), *kp = k.data_ptr(), *vp = v.data_ptr();
    const float *bp = ptr(t[3]), *gp = ptr(t[4]), *rp = ptr(t[5]), *dp = ptr(t[6]), *sp = ptr(t[7]);
    void *op = o.data_ptr();
    float *So = static_cast<float *>(S.data_ptr()), *d_out = static_cast<float *>(d.data_ptr());
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = g_step(&p, qp, kp, vp, bp, gp, rp, dp, sp, op, So, d_out, stream);
    Py_END_ALLOW_THREADS
    if (rc != OSDN_OK) return PyLong_FromLong(rc);
    PyObject *out = PyTuple_New(3);
    if (!out) return nullptr;
    PyTuple_SET_ITEM(out, 0, THPVariable_Wrap(o));
    if (in_place) {
        Py_INCREF(a[7]);
        PyTuple_SET_ITEM(out, 1, a[7]);
    } else {
        PyTuple_SET_ITEM(out, 1, THPVariable_Wrap(S));
    }
    PyTuple_SET_ITEM(out, 2, THPVariable_Wrap(d));
    return out;
    END_HANDLE_TH_ERRORS
}

// bind(address, size, version): where osdn_step is.  Refused where its struct or the tensor library are not those this was built for.
PyObject *bind(PyObject *, PyObject *args) {
    PyObject *addr;
    Py_ssize_t size;
    const char *version;
    if (!PyArg_ParseTuple(args, "Ons", &addr, &size, &version)) return nullptr;
    void *p = PyLong_AsVoidPtr(addr);
    if (PyErr_Occurred()) return nullptr;
    if (size != (Py_ssize_t)sizeof(osdn_params))
        return PyErr_Format(PyExc_ImportError, "built for an osdn_params of %zd bytes, not %zd", (Py_ssize_t)sizeof(osdn_params), size);
    if (std::strcmp(version, OSDN_TORCH_VERSION) != 0)
        return PyErr_Format(PyExc_ImportError, "built for torch " OSDN_TORCH_VERSION ", not %s", version);
    g_step = reinterpret_cast<StepFn>(p);
    Py_RETURN_NONE;
}

PyMethodDef kMethods[] = {
    {"step", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(step)), METH_FASTCALL, "osdn_step on plain tensors, or None"},
    {"bind", bind, METH_VARARGS, "address of osdn_step, size of osdn_params, version of the tensor library"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) {
    for (int i = 0; i < 10; ++i) {
        g_names[i] = PyUnicode_InternFromString(kNames[i]);
        if (!g_names[i]) return nullptr;
    }
    return PyModule_Create(&kModule);
}
