// The entry points that a Python program calls once per kernel or inference, as a CPython
// extension.  Through ctypes the conversion of ten arguments costs 1.3 us, half of what the HIP
// launch itself takes on the host; vectorcall functions that read the integers directly cost 0.2.
//
// Every function returns the call's status, or None when an argument is not a plain integer (or
// None for a pointer): the caller then goes through ctypes, which knows all other forms.  As there,
// integers are truncated to the C type and the interpreter lock is released during the call.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include "sgprs.h"

namespace {

struct Args {
    PyObject* const* v;
    Py_ssize_t n, at = 0;
    bool ok = true;
    unsigned long long word(bool none_ok)
    {
        PyObject* o = v[at++];
        if (PyLong_Check(o)) return PyLong_AsUnsignedLongLongMask(o);
        if (!none_ok || o != Py_None) ok = false;
        return 0;
    }
    int i() { return (int)word(false); }
    size_t z() { return (size_t)word(false); }
    template <class T = void> T* p() { return (T*)word(true); }
};

// One method: FIELDS declares the arguments in order, CALL uses them.
#define METHOD(name, count, FIELDS, CALL)                                                         \
    PyObject* name(PyObject*, PyObject* const* argv, Py_ssize_t n)                                \
    {                                                                                             \
        if (n != count) {                                                                         \
            PyErr_Format(PyExc_TypeError, #name " takes %d arguments (%zd given)", count, n);     \
            return nullptr;                                                                       \
        }                                                                                         \
        Args a{argv, n};                                                                          \
        FIELDS;                                                                                   \
        if (!a.ok) {                                                                              \
            PyErr_Clear();                                                                        \
            Py_RETURN_NONE;                                                                       \
        }                                                                                         \
        int rc;                                                                                   \
        Py_BEGIN_ALLOW_THREADS rc = CALL;                                                         \
        Py_END_ALLOW_THREADS return PyLong_FromLong(rc);                                          \
    }

METHOD(conv2d, 11, auto* d = a.p<sgprs_conv_desc_t>(); auto* x = a.p(); auto* w = a.p(); auto* sc = a.p<float>(); auto* sh = a.p<float>();
       auto* res = a.p(); auto* y = a.p(); auto* ws = a.p(); size_t wb = a.z(); auto* pool = a.p<sgprs_pool_t>(); int part = a.i(),
       sgprs_conv2d(d, x, w, sc, sh, res, y, ws, wb, pool, part))
METHOD(maxpool2d, 9, int dt = a.i(); int nn = a.i(); int h = a.i(); int w = a.i(); int c = a.i(); auto* x = a.p(); auto* y = a.p();
       auto* pool = a.p<sgprs_pool_t>(); int part = a.i(), sgprs_maxpool2d(dt, nn, h, w, c, x, y, pool, part))
METHOD(bn_relu, 9, int dt = a.i(); size_t px = a.z(); int c = a.i(); auto* x = a.p(); auto* sc = a.p<float>(); auto* sh = a.p<float>();
       auto* y = a.p(); auto* pool = a.p<sgprs_pool_t>(); int part = a.i(), sgprs_bn_relu(dt, px, c, x, sc, sh, y, pool, part))
METHOD(add_relu, 8, int dt = a.i(); size_t cnt = a.z(); auto* x = a.p(); auto* b = a.p(); auto* y = a.p(); int relu = a.i();
       auto* pool = a.p<sgprs_pool_t>(); int part = a.i(), sgprs_add_relu(dt, cnt, x, b, y, relu, pool, part))
METHOD(avgpool_fc, 12, int dt = a.i(); int nn = a.i(); int hw = a.i(); int cin = a.i(); int cout = a.i(); auto* x = a.p(); auto* w = a.p();
       auto* bias = a.p<float>(); auto* lg = a.p<float>(); auto* ws = a.p<float>(); auto* pool = a.p<sgprs_pool_t>(); int part = a.i(),
       sgprs_avgpool_fc(dt, nn, hw, cin, cout, x, w, bias, lg, ws, pool, part))
METHOD(avgpool_fc_static, 11, int dt = a.i(); int nn = a.i(); int hw = a.i(); int cin = a.i(); int cout = a.i(); auto* x = a.p();
       auto* w = a.p(); auto* bias = a.p<float>(); auto* lg = a.p<float>(); auto* pool = a.p<sgprs_pool_t>(); int part = a.i(),
       sgprs_avgpool_fc_static(dt, nn, hw, cin, cout, x, w, bias, lg, pool, part))
METHOD(global_avgpool, 8, int dt = a.i(); int nn = a.i(); int hw = a.i(); int c = a.i(); auto* x = a.p(); auto* y = a.p<float>();
       auto* pool = a.p<sgprs_pool_t>(); int part = a.i(), sgprs_global_avgpool(dt, nn, hw, c, x, y, pool, part))
METHOD(stage_run, 7, auto* t = a.p<sgprs_task_t>(); int st = a.i(); int b = a.i(); auto* in = a.p(); auto* out = a.p();
       auto* pool = a.p<sgprs_pool_t>(); int part = a.i(), sgprs_stage_run(t, st, b, in, out, pool, part))
METHOD(task_run, 6, auto* t = a.p<sgprs_task_t>(); int b = a.i(); auto* in = a.p(); auto* lg = a.p<float>();
       auto* pool = a.p<sgprs_pool_t>(); int part = a.i(), sgprs_task_run(t, b, in, lg, pool, part, nullptr))

#define ENTRY(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {ENTRY(conv2d), ENTRY(maxpool2d), ENTRY(bn_relu), ENTRY(add_relu), ENTRY(avgpool_fc), ENTRY(avgpool_fc_static),
                         ENTRY(global_avgpool), ENTRY(stage_run), ENTRY(task_run), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", "Hot entry points of libsgprs.", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls(void) { return PyModule_Create(&module); }
