// Argument marshalling of the calls that a serving loop makes once per layer (tc_prefill_attn and its
// non-allocating variant), as a small CPython module: through ctypes and numpy's address objects the
// marshalling alone took 6-7 us per call, as much as the launches it leads to; here it takes under 1 us.
// Nothing is kept from one call for the next.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstdint>

namespace {

typedef int32_t (*prefill_fn)(void *, int32_t, const void *, const void *, const void *, void *, const int32_t *,
                              const int32_t *, int32_t, const int32_t *, const int32_t *, int32_t, float, void *);

PyObject *s_data_ptr, *s_cuda_stream, *s_ctypes, *s_data;
PyObject *g_as_int32;                   // callable: anything array-like -> contiguous int32 array

bool as_address(PyObject *x, void **out)
{
    if (x == Py_None) { *out = nullptr; return true; }
    PyObject *v = nullptr;
    if (PyLong_Check(x)) { v = x; Py_INCREF(v); }
    else if ((v = PyObject_CallMethodNoArgs(x, s_data_ptr)) == nullptr) {       // torch tensor, or else a numpy array
        if (!PyErr_ExceptionMatches(PyExc_AttributeError)) return false;
        PyErr_Clear();
        PyObject *c = PyObject_GetAttr(x, s_ctypes);
        if (!c) return false;
        v = PyObject_GetAttr(c, s_data);
        Py_DECREF(c);
        if (!v) return false;
    }
    *out = PyLong_AsVoidPtr(v);
    Py_DECREF(v);
    return !(*out == nullptr && PyErr_Occurred());
}

// A view of an int32 array that holds on to its memory for the length of the call.
struct Ints {
    Py_buffer view{};
    bool held = false;
    ~Ints() { if (held) PyBuffer_Release(&view); }
    bool plain() const
    {
        const char *f = view.format;
        return view.itemsize == 4 && f && (f[0] == 'i' || f[0] == 'l') && f[1] == 0;
    }
    bool take(PyObject *x)
    {
        if (PyObject_CheckBuffer(x) && PyObject_GetBuffer(x, &view, PyBUF_ND | PyBUF_FORMAT | PyBUF_C_CONTIGUOUS) == 0) {
            held = true;
            if (plain()) return true;
            PyBuffer_Release(&view);
            held = false;
        }
        PyErr_Clear();
        PyObject *a = PyObject_CallOneArg(g_as_int32, x);
        if (!a) return false;
        const int rc = PyObject_GetBuffer(a, &view, PyBUF_ND | PyBUF_FORMAT | PyBUF_C_CONTIGUOUS);
        Py_DECREF(a);                       // the view keeps it alive
        held = rc == 0;
        return held;
    }
    const int32_t *data() const { return (const int32_t *)view.buf; }
    Py_ssize_t size() const { return view.len / 4; }
};

// prefill(function address, context address, layer, q, k_new, v_new, out, cu_seqlens, block_table,
//         prefix_len, suffix_len, sm_scale, stream) -> status
PyObject *prefill(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != 13) { PyErr_SetString(PyExc_TypeError, "prefill takes 13 arguments"); return nullptr; }
    void *fn, *ctx, *q, *k, *v, *out, *stream = nullptr;
    if (!as_address(args[0], &fn) || !as_address(args[1], &ctx)) return nullptr;
    const long layer = PyLong_AsLong(args[2]);
    if (layer == -1 && PyErr_Occurred()) return nullptr;
    if (!as_address(args[3], &q) || !as_address(args[4], &k) || !as_address(args[5], &v) || !as_address(args[6], &out)) return nullptr;
    Ints cu, bt, pl, sl;
    if (!cu.take(args[7]) || !bt.take(args[8]) || !pl.take(args[9]) || !sl.take(args[10])) return nullptr;
    const double scale = PyFloat_AsDouble(args[11]);
    if (scale == -1.0 && PyErr_Occurred()) return nullptr;
    PyObject *s = args[12];
    if (s == Py_None || PyLong_Check(s)) {
        if (!as_address(s, &stream)) return nullptr;
    } else {
        PyObject *a = PyObject_GetAttr(s, s_cuda_stream);
        if (!a) return nullptr;
        const bool ok = as_address(a, &stream);
        Py_DECREF(a);
        if (!ok) return nullptr;
    }
    const Py_ssize_t B = pl.size();
    const Py_ssize_t max_blocks = bt.view.ndim == 2 ? bt.view.shape[1] : (B ? bt.size() / B : 0);
    int32_t rc;
    Py_BEGIN_ALLOW_THREADS
    rc = ((prefill_fn)fn)(ctx, (int32_t)layer, q, k, v, out, cu.data(), bt.data(), (int32_t)max_blocks, pl.data(), sl.data(),
                          (int32_t)B, (float)scale, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

PyObject *set_converter(PyObject *, PyObject *f)
{
    Py_XDECREF(g_as_int32);
    Py_INCREF(f);
    g_as_int32 = f;
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"prefill", (PyCFunction)(void (*)(void))prefill, METH_FASTCALL, "marshal one tc_prefill_attn call"},
    {"set_converter", set_converter, METH_O, "callable that turns anything array-like into a contiguous int32 array"},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_py_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__py_call(void)
{
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    s_ctypes = PyUnicode_InternFromString("ctypes");
    s_data = PyUnicode_InternFromString("data");
    return PyModule_Create(&module);
}
