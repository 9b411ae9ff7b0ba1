// The step calls' way from Python objects to the C ABI.  A small shard's step costs the host more than the device: an Adam step on
// 4099 elements takes the device 3.3 us, and Python bytecode, struct packing and ctypes took 1 us of the host's 6.1, of a call with a
// whole tensor's descriptor 2 us of 7.3.  Here the argument structs are filled from the objects' own fields.
//
// Only what needs no conversion is taken: a Plan with an integer handle, exactly a Hyper whose fields are plain numbers in range, an
// exact torch.Tensor or an integer address, the current stream.  Everything else is not taken: the call returns 1, which no entry
// point does, and binding.py's conversions, whose errors are the definition, decide.  The GIL is released around the library's call,
// as ctypes does.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cmath>
#include <cstdint>
#include <cstring>
#include <initializer_list>

#include "ccfused.h"

namespace {

typedef int (*StepFn)(cc_plan *, const cc_hparams *, int32_t *, void *);
typedef int (*StaticFn)(const cc_tensor *, int32_t, const cc_hparams *, int32_t *, void *);
typedef int (*EpilogueFn)(const cc_epilogue *, void *);

// Set by bind(), once, before the first call.
PyTypeObject *g_plan, *g_hyper, *g_tensor_args, *g_tensor, *g_parameter;
PyObject *g_get_device, *g_raw_stream;
PyCFunction g_data_ptr, g_numel;

enum Field { kLr, kBeta1, kBeta2, kEps, kLossScale, kStep, kGradAverage, kAdamMode, kSkipMode, kHandle, kNumel, kWIn, kMIn, kVIn, kWOut, kMOut, kVOut, kW16Out, kGrad, kWeightDecay, kFields };
const char *const kNames[kFields] = {"lr", "beta1", "beta2", "eps", "loss_scale", "step", "grad_average", "adam_mode", "skip_mode", "handle",
                                     "numel", "w_in", "m_in", "v_in", "w_out", "m_out", "v_out", "w16_out", "grad", "weight_decay"};
PyObject *g_names[kFields];

// The dictionary of an object of exactly this type.
struct Fields {
    PyObject *dict = nullptr;
    Fields(PyObject *o, PyTypeObject *type)
    {
        PyObject **d = Py_TYPE(o) == type ? _PyObject_GetDictPtr(o) : nullptr;
        if (d) Py_XINCREF(dict = *d);
    }
    ~Fields() { Py_XDECREF(dict); }
    Fields(const Fields &) = delete;
    PyObject *operator[](Field f) const { return dict ? PyDict_GetItemWithError(dict, g_names[f]) : nullptr; }
};

// False: not a plain number, or out of range (an error may be set; the callers clear it).
bool to_float(PyObject *x, float *out)
{
    double d;
    if (x && PyFloat_CheckExact(x)) d = PyFloat_AS_DOUBLE(x);
    else if (x && PyLong_CheckExact(x)) {
        d = PyLong_AsDouble(x);
        if (d == -1.0 && PyErr_Occurred()) return false;
    } else return false;
    *out = (float)d;
    return !std::isfinite(d) || std::isfinite(*out);
}
bool to_int(PyObject *x, int32_t *out)
{
    if (!x || !PyLong_Check(x)) return false;
    int overflow;
    const long long v = PyLong_AsLongLongAndOverflow(x, &overflow);
    if (overflow || v < INT32_MIN || v > INT32_MAX) return false;
    *out = (int32_t)v;
    return true;
}
bool to_u64(PyObject *x, uint64_t *out)
{
    if (!x || !PyLong_CheckExact(x)) return false;
    *out = PyLong_AsUnsignedLongLong(x);
    return !(*out == (uint64_t)-1 && PyErr_Occurred());
}
bool is_tensor(PyObject *x) { return x && (Py_TYPE(x) == g_tensor || Py_TYPE(x) == g_parameter); }
template <class P> bool address(PyObject *tensor, P *out)
{
    if (!is_tensor(tensor)) return false;
    Py_INCREF(tensor);                   // a torch function mode runs other code in here
    PyObject *p = g_data_ptr(tensor, nullptr);
    Py_DECREF(tensor);
    uint64_t v = 0;
    const bool good = p && to_u64(p, &v);
    Py_XDECREF(p);
    *out = reinterpret_cast<P>((uintptr_t)v);
    return good;
}
bool to_flag(PyObject *x, int32_t **out)
{
    if (!PyLong_CheckExact(x)) return address(x, out);
    uint64_t v;
    if (!to_u64(x, &v)) return false;
    *out = reinterpret_cast<int32_t *>((uintptr_t)v);
    return true;
}

bool to_hparams(PyObject *hp, cc_hparams *c)
{
    const Fields d(hp, g_hyper);
    return to_float(d[kLr], &c->lr) && to_float(d[kBeta1], &c->beta1) && to_float(d[kBeta2], &c->beta2) && to_float(d[kEps], &c->eps) &&
           to_float(d[kLossScale], &c->loss_scale) && to_int(d[kStep], &c->step) && to_int(d[kGradAverage], &c->grad_average) &&
           to_int(d[kAdamMode], &c->adam_mode) && to_int(d[kSkipMode], &c->skip_mode);
}

// The current device's current stream.
bool current_stream(PyObject *stream, void **out)
{
    if (stream != Py_None) return false;
    PyObject *device = PyObject_CallNoArgs(g_get_device);
    PyObject *raw = device ? PyObject_CallOneArg(g_raw_stream, device) : nullptr;
    uint64_t v = 0;
    const bool good = raw && to_u64(raw, &v);
    Py_XDECREF(device);
    Py_XDECREF(raw);
    *out = reinterpret_cast<void *>((uintptr_t)v);
    return good;
}

// Up to CC_MAX_R slices; the rest stay null.
template <class P> bool addresses(PyObject *list, P (&out)[CC_MAX_R], Py_ssize_t *count)
{
    if (!list || !(PyList_CheckExact(list) || PyTuple_CheckExact(list))) return false;
    Py_INCREF(list);
    bool good = true;
    for (Py_ssize_t r = 0; good && r < PySequence_Fast_GET_SIZE(list) && r < CC_MAX_R; ++r) good = address(PySequence_Fast_GET_ITEM(list, r), &out[r]);
    *count = PySequence_Fast_GET_SIZE(list);
    Py_DECREF(list);
    return good;
}

PyObject *not_taken()
{
    PyErr_Clear();
    return PyLong_FromLong(1);
}
template <class Call> PyObject *called(Call call)
{
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = call();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}
template <class Fn> Fn function(PyObject *address) { return reinterpret_cast<Fn>(PyLong_AsVoidPtr(address)); }

// step(function, plan, hp, flag, stream)
PyObject *step(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    cc_hparams hp;
    int32_t *flag;
    void *stream;
    uint64_t handle;
    if (n != 5) return not_taken();
    const Fields plan(a[1], g_plan);
    if (!to_u64(plan[kHandle], &handle) || !to_hparams(a[2], &hp) || !to_flag(a[3], &flag) || !current_stream(a[4], &stream)) return not_taken();
    const StepFn fn = function<StepFn>(a[0]);
    return called([&] { return fn(reinterpret_cast<cc_plan *>((uintptr_t)handle), &hp, flag, stream); });
}

// static_step(function, tensor, R, hp, flag, stream)
PyObject *static_step(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    cc_hparams hp;
    int32_t *flag, R;
    void *stream;
    Py_ssize_t slices;
    if (n != 6) return not_taken();
    const Fields d(a[1], g_tensor_args);
    cc_tensor t;
    std::memset(&t, 0, sizeof(t));
    if (!to_u64(d[kNumel], &t.numel) || !address(d[kWIn], &t.w_in) || !address(d[kMIn], &t.m_in) ||
        !address(d[kVIn], &t.v_in) || !address(d[kWOut], &t.w_out) || !address(d[kMOut], &t.m_out) ||
        !address(d[kVOut], &t.v_out) || !address(d[kW16Out], &t.w16_out) || !addresses(d[kGrad], t.grad, &slices) ||
        !to_float(d[kWeightDecay], &t.weight_decay) || !to_int(a[2], &R) || !to_hparams(a[3], &hp) || !to_flag(a[4], &flag) ||
        !current_stream(a[5], &stream))
        return not_taken();
    const StaticFn fn = function<StaticFn>(a[0]);
    return called([&] { return fn(&t, R, &hp, flag, stream); });
}

// epilogue(function, partials, bias, residual, out, first, hidden, dropout_p, seed, stream, numel)
PyObject *epilogue(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    cc_epilogue e;
    std::memset(&e, 0, sizeof(e));
    Py_ssize_t slices;
    uint64_t hidden;
    void *stream;
    if (n != 11 || !addresses(a[1], e.partial, &slices) || !address(a[2], &e.bias) || !address(a[3], &e.residual) || !address(a[4], &e.out) ||
        !to_u64(a[5], &e.first) || !to_u64(a[6], &hidden) || hidden > UINT32_MAX || slices > INT32_MAX || !to_float(a[7], &e.dropout_p) ||
        !to_u64(a[8], &e.seed) || !current_stream(a[9], &stream))
        return not_taken();
    if (a[10] != Py_None) {
        if (!to_u64(a[10], &e.numel)) return not_taken();
    } else {
        PyObject *k = g_numel(a[3], nullptr);
        const bool good = k && to_u64(k, &e.numel);
        Py_XDECREF(k);
        if (!good) return not_taken();
    }
    e.hidden = (uint32_t)hidden;
    e.R = (int32_t)slices;
    const EpilogueFn fn = function<EpilogueFn>(a[0]);
    return called([&] { return fn(&e, stream); });
}

// A method of torch.Tensor that takes no arguments, as the C function behind it, if torch.Tensor and Parameter both have it as it is.
PyCFunction no_args_method(const char *name)
{
    PyObject *m = PyObject_GetAttrString((PyObject *)g_tensor, name), *same = m ? PyObject_GetAttrString((PyObject *)g_parameter, name) : nullptr;
    PyCFunction f = nullptr;
    if (same && m == same && Py_TYPE(m) == &PyMethodDescr_Type && ((PyMethodDescrObject *)m)->d_method->ml_flags == METH_NOARGS)
        f = ((PyMethodDescrObject *)m)->d_method->ml_meth;
    Py_XDECREF(m);
    Py_XDECREF(same);
    if (!f) PyErr_Clear();
    return f;
}

// bind(Plan, Hyper, Tensor, torch.Tensor, torch.nn.Parameter, current device, current raw stream): whether the calls above can be used.
PyObject *bind(PyObject *, PyObject *args)
{
    PyObject *plan, *hyper, *tensor_args, *tensor, *parameter, *device, *raw;
    if (!PyArg_ParseTuple(args, "O!O!O!O!O!OO", &PyType_Type, &plan, &PyType_Type, &hyper, &PyType_Type, &tensor_args, &PyType_Type, &tensor, &PyType_Type, &parameter, &device, &raw)) return nullptr;
    for (PyObject *o : {plan, hyper, tensor_args, tensor, parameter, device, raw}) Py_INCREF(o);          // for as long as the process runs
    g_plan = (PyTypeObject *)plan;
    g_hyper = (PyTypeObject *)hyper;
    g_tensor_args = (PyTypeObject *)tensor_args;
    g_tensor = (PyTypeObject *)tensor;
    g_parameter = (PyTypeObject *)parameter;
    g_get_device = device;
    g_raw_stream = raw;
    g_data_ptr = no_args_method("data_ptr");
    g_numel = no_args_method("numel");
    for (int k = 0; k < kFields; ++k)
        if (!g_names[k] && !(g_names[k] = PyUnicode_InternFromString(kNames[k]))) return nullptr;
    return PyBool_FromLong(g_data_ptr && g_numel);
}

PyMethodDef g_methods[] = {{"bind", bind, METH_VARARGS, nullptr},
                           {"step", (PyCFunction)(void *)step, METH_FASTCALL, nullptr},
                           {"static_step", (PyCFunction)(void *)static_step, METH_FASTCALL, nullptr},
                           {"epilogue", (PyCFunction)(void *)epilogue, METH_FASTCALL, nullptr},
                           {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_step_calls", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__step_calls(void) { return PyModule_Create(&g_module); }
