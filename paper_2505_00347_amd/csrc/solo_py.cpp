// The step calls of the Python binding, marshalled natively.
//
// A step of a small tensor takes the GPU 4-6 us; a ctypes call with eleven or thirteen arguments,
// seven data_ptr() calls from Python and a torch.cuda.current_stream() object took the host 7.8 us
// beside an MI355X (launch included), so the caller was what bounded it: 3.5 us through this module,
// and the call of 4096 elements went from 7.8 to 4.5 us.
// Nothing is kept between calls but the entry points of libsolo and torch's two functions that name
// the current stream: every pointer is asked for on every call.  What only ctypes can pass (its own
// integer objects, anything with _as_parameter_) goes to the binding's calls through ctypes.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

#include "../../include/solo.h"

namespace {

decltype(&solo_adamw_step_mp) g_step = nullptr;
decltype(&solo_adamw_step_multi) g_multi = nullptr;
PyObject *g_config_type = nullptr;      // the ctypes mirror of solo_config
PyObject *g_argument_error = nullptr;   // ctypes.ArgumentError
PyObject *g_ctypes_object = nullptr;    // base class of ctypes' integers and pointers
PyObject *g_ctypes_step = nullptr, *g_ctypes_multi = nullptr;    // the same calls through ctypes
PyObject *g_slow_stream = nullptr;      // Python: the current stream's handle, initialising torch's GPU side if need be
PyObject *g_get_device = nullptr, *g_raw_stream = nullptr;   // torch's own, or null where it has none
PyObject *g_data_ptr = nullptr, *g_cuda_stream = nullptr, *g_as_parameter = nullptr;    // interned names
bool g_gpu_ready = false;               // g_slow_stream has succeeded in this process

bool refuse(const char *what, PyObject *got)
{
    PyErr_Format(g_argument_error, "%s expected, got %s", what, Py_TYPE(got)->tp_name);
    return false;
}

// An integer argument, as ctypes passes one: wrapped to the width of its C type.  False without an
// exception: one for ctypes.
bool integer(PyObject *o, uint64_t &out)
{
    if (!PyLong_Check(o)) {
        const int is = PyObject_IsInstance(o, g_ctypes_object);
        if (is < 0) return false;
        return is || PyObject_HasAttr(o, g_as_parameter) ? false : refuse("an int", o);
    }
    out = PyLong_AsUnsignedLongLongMask(o);
    return !(out == (uint64_t)-1 && PyErr_Occurred());
}

// None, an address, or a tensor.
template <typename T>
bool pointer(PyObject *o, T *&out)
{
    uint64_t v = 0;
    if (o != Py_None) {
        if (PyLong_Check(o)) {
            if (!integer(o, v)) return false;
        } else {
            PyObject *r = PyObject_CallMethodNoArgs(o, g_data_ptr);
            if (!r) return false;
            const bool ok = r == Py_None || integer(r, v);
            Py_DECREF(r);
            if (!ok) return false;
        }
    }
    out = reinterpret_cast<T *>(v);
    return true;
}

// None (torch's current stream), a handle, or a stream object.
bool stream_of(PyObject *o, void *&out)
{
    uint64_t v = 0;
    PyObject *r = nullptr;
    if (o == Py_None) {
        if (g_gpu_ready && g_raw_stream) {
            PyObject *dev = PyObject_CallNoArgs(g_get_device);
            if (!dev) return false;
            r = PyObject_CallOneArg(g_raw_stream, dev);
            Py_DECREF(dev);
        } else {
            r = PyObject_CallNoArgs(g_slow_stream);
            if (r) g_gpu_ready = true;
        }
    } else if (PyLong_Check(o)) {
        Py_INCREF(o);
        r = o;
    } else {
        r = PyObject_GetAttr(o, g_cuda_stream);
    }
    if (!r) return false;
    const bool ok = r == Py_None || integer(r, v);      // (None: the default stream)
    Py_DECREF(r);
    out = reinterpret_cast<void *>(v);
    return ok;
}

struct Config {
    Py_buffer view;
    bool held = false;
    bool get(PyObject *o)
    {
        const int is = PyObject_IsInstance(o, g_config_type);
        if (is < 0) return false;
        if (!is) return refuse("a solo_config", o);
        if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) return false;
        held = true;
        if (view.len < (Py_ssize_t)sizeof(solo_config)) return refuse("a solo_config", o);
        return true;
    }
    const solo_config *ptr() const { return static_cast<const solo_config *>(view.buf); }
    ~Config() { if (held) PyBuffer_Release(&view); }
};

bool count_args(Py_ssize_t got, Py_ssize_t want)
{
    if (g_step && got == want) return true;
    PyErr_Format(PyExc_TypeError, "%zd arguments expected, got %zd", want, got);
    return false;
}

PyObject *by_ctypes(PyObject *call, PyObject *const *a, Py_ssize_t count)
{
    return PyErr_Occurred() ? nullptr : PyObject_Vectorcall(call, a, (size_t)count, nullptr);
}

// step(param, param_bf16, grad, grad_scale, m_codes, m_scale, v_codes, v_scale, v_base, n, step, cfg, stream)
PyObject *step(PyObject *, PyObject *const *a, Py_ssize_t count)
{
    float *param, *m_scale, *v_scale, *v_base;
    uint16_t *param_bf16;
    const void *grad;
    const float *grad_scale;
    uint32_t *m_codes, *v_codes;
    uint64_t n, t;
    void *stream = nullptr;
    Config cfg;
    if (!count_args(count, 13)) return nullptr;
    if (!pointer(a[0], param) || !pointer(a[1], param_bf16) || !pointer(a[2], grad) ||
        !pointer(a[3], grad_scale) || !pointer(a[4], m_codes) || !pointer(a[5], m_scale) || !pointer(a[6], v_codes) ||
        !pointer(a[7], v_scale) || !pointer(a[8], v_base) || !integer(a[9], n) || !integer(a[10], t) || !cfg.get(a[11]) ||
        (n != 0 && !stream_of(a[12], stream)))
        return by_ctypes(g_ctypes_step, a, count);
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = g_step(param, param_bf16, grad, grad_scale, m_codes, m_scale, v_codes, v_scale, v_base, n, t, cfg.ptr(), stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// multi(table, count, units, table_flags, grad_scale, step, cfg, stream)
PyObject *multi(PyObject *, PyObject *const *a, Py_ssize_t count)
{
    const void *table;
    const float *grad_scale;
    uint64_t tensors, units, flags, t;
    void *stream = nullptr;
    Config cfg;
    if (!count_args(count, 8)) return nullptr;
    if (!pointer(a[0], table) || !integer(a[1], tensors) || !integer(a[2], units) ||
        !integer(a[3], flags) || !pointer(a[4], grad_scale) || !integer(a[5], t) || !cfg.get(a[6]) ||
        (units != 0 && !stream_of(a[7], stream)))
        return by_ctypes(g_ctypes_multi, a, count);
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = g_multi(table, (uint32_t)tensors, units, (uint32_t)flags, grad_scale, t, cfg.ptr(), stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// bind(address of solo_adamw_step_mp, of solo_adamw_step_multi, config type, its size, ArgumentError, ctypes' base
//      class, the step through ctypes, the multi-tensor step through ctypes, slow stream, torch's current
//      device, torch's raw stream of a device): the last two may be None
PyObject *bind(PyObject *, PyObject *args)
{
    unsigned long long s, m;
    Py_ssize_t size;
    PyObject *type, *error, *object, *step_c, *multi_c, *slow, *device, *raw;
    if (!PyArg_ParseTuple(args, "KKOnOOOOOOO", &s, &m, &type, &size, &error, &object, &step_c, &multi_c, &slow, &device, &raw))
        return nullptr;
    if (size != (Py_ssize_t)sizeof(solo_config)) {
        PyErr_Format(PyExc_ImportError, "built for a solo_config of %zu bytes, not %zd", sizeof(solo_config), size);
        return nullptr;
    }
    g_step = reinterpret_cast<decltype(g_step)>((uintptr_t)s);
    g_multi = reinterpret_cast<decltype(g_multi)>((uintptr_t)m);
    const bool fast = device != Py_None && raw != Py_None;
    struct { PyObject **to, *from; } kept[] = {
        {&g_config_type, type}, {&g_argument_error, error}, {&g_ctypes_object, object}, {&g_ctypes_step, step_c},
        {&g_ctypes_multi, multi_c}, {&g_slow_stream, slow}, {&g_get_device, fast ? device : nullptr},
        {&g_raw_stream, fast ? raw : nullptr}};
    for (auto &k : kept) {
        Py_XINCREF(k.from);
        Py_XSETREF(*k.to, k.from);
    }
    g_gpu_ready = false;
    Py_RETURN_NONE;
}

// A forked child has no GPU of its parent's: the next call asks torch again, which says so.
PyObject *forked(PyObject *, PyObject *)
{
    g_gpu_ready = false;
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"step", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(step)), METH_FASTCALL, "solo_adamw_step_mp"},
    {"multi", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(multi)), METH_FASTCALL, "solo_adamw_step_multi"},
    {"bind", bind, METH_VARARGS, "the entry points and types of the binding"},
    {"forked", forked, METH_NOARGS, "called in a forked child"},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_solo_native", "step calls of libsolo", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__solo_native()
{
    g_data_ptr = PyUnicode_InternFromString("data_ptr");
    g_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    g_as_parameter = PyUnicode_InternFromString("_as_parameter_");
    if (!g_data_ptr || !g_cuda_stream || !g_as_parameter) return nullptr;
    return PyModule_Create(&module);
}
