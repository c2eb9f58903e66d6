// Calls of the C ABI from Python: converts the arguments (a tensor by its data_ptr(), an address, None, an integer), releases the
// interpreter lock and calls the entry point.  One decoded token's GEMM takes 5 us on the device and 27 arguments; converted by ctypes
// and in Python they took longer than that.  The entry points' addresses come from binding.py, which loads the library.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <tuple>
#include <type_traits>
#include <utility>

#include "aweq.h"

namespace {

PyObject* s_data_ptr;

template <class T>
bool convert(PyObject* o, T& v)
{
    if constexpr (std::is_pointer<T>::value) {
        if (o == Py_None) { v = nullptr; return true; }
        unsigned long long a;
        if (PyLong_Check(o)) {
            a = PyLong_AsUnsignedLongLongMask(o);
        } else {
            PyObject* const r = PyObject_CallMethodNoArgs(o, s_data_ptr);
            if (!r) return false;
            a = PyLong_AsUnsignedLongLongMask(r);
            Py_DECREF(r);
        }
        if (a == (unsigned long long)-1 && PyErr_Occurred()) return false;
        v = reinterpret_cast<T>((uintptr_t)a);
    } else {
        const unsigned long long a = PyLong_AsUnsignedLongLongMask(o);   // (the low bits, whatever the integer's sign and size: as ctypes converts)
        if (a == (unsigned long long)-1 && PyErr_Occurred()) return false;
        v = (T)a;
    }
    return true;
}

template <class T> struct Entry;
template <class... A>
struct Entry<int (*)(A...)> {
    template <size_t... I>
    static PyObject* run(int (*fn)(A...), PyObject* const* o, std::index_sequence<I...>)
    {
        std::tuple<A...> a;
        if (!(convert(o[I], std::get<I>(a)) && ...)) return nullptr;
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = fn(std::get<I>(a)...);
        Py_END_ALLOW_THREADS
        return PyLong_FromLong(rc);
    }
    static PyObject* call(int (*fn)(A...), PyObject* const* o, Py_ssize_t n)
    {
        if (!fn) { PyErr_SetString(PyExc_RuntimeError, "the library is not loaded"); return nullptr; }
        if (n != (Py_ssize_t)sizeof...(A)) { PyErr_Format(PyExc_TypeError, "%zd arguments instead of %zd", n, (Py_ssize_t)sizeof...(A)); return nullptr; }
        return run(fn, o, std::index_sequence_for<A...>());
    }
};

#define ENTRIES(X)                                                                                                     \
    X(aweq_calib_stats) X(aweq_calib_stats_static) X(aweq_equalize) X(aweq_quant_weight) X(aweq_fold_quant_weight)     \
    X(aweq_quant_act) X(aweq_w8a8_gemm) X(aweq_w8a8_gemm_fused) X(aweq_bias_correct) X(aweq_wonly_gemm)

#define X(name)                                                                                                        \
    decltype(&::name) p_##name;                                                                                        \
    PyObject* call_##name(PyObject*, PyObject* const* o, Py_ssize_t n) { return Entry<decltype(&::name)>::call(p_##name, o, n); }
ENTRIES(X)
#undef X
decltype(&::aweq_calibrate) p_aweq_calibrate;

// the fields of a structure in order, from a sequence
struct Fields {
    PyObject* seq;
    Py_ssize_t at = 0;
    bool ok = true;
    explicit Fields(PyObject* o) : seq(PySequence_Fast(o, "a sequence of fields")) { ok = seq != nullptr; }
    ~Fields() { Py_XDECREF(seq); }
    template <class T>
    Fields& operator>>(T& v)
    {
        if (!ok) return *this;
        if (at >= PySequence_Fast_GET_SIZE(seq)) { PyErr_SetString(PyExc_TypeError, "a field is missing"); ok = false; return *this; }
        ok = convert(PySequence_Fast_GET_ITEM(seq, at), v);
        ++at;
        return *this;
    }
    // every field has been taken (the count is what there is to check a structure's layout by)
    bool done()
    {
        if (ok && at != PySequence_Fast_GET_SIZE(seq)) { PyErr_Format(PyExc_TypeError, "%zd fields instead of %zd", PySequence_Fast_GET_SIZE(seq), at); ok = false; }
        return ok;
    }
};

PyObject* call_aweq_calibrate(PyObject*, PyObject* const* o, Py_ssize_t n)
{
    if (!p_aweq_calibrate) { PyErr_SetString(PyExc_RuntimeError, "the library is not loaded"); return nullptr; }
    if (n != 3) { PyErr_SetString(PyExc_TypeError, "layer, weights, stream"); return nullptr; }
    aweq_calib_layer l;
    Fields f(o[0]);
    f >> l.X >> l.dt >> l.T >> l.K >> l.ldx >> l.xmin >> l.xmax >> l.xsum >> l.count >> l.r_x >> l.R_x >> l.p_x >> l.wmin >> l.wmax >> l.wcount >> l.r_w >>
        l.R_w >> l.p_w >> l.s >> l.inv_s >> l.xhat_range >> l.mu_xhat >> l.act_step >> l.act_zero >> l.xq >> l.rowsum_x >> l.colsum_xq >>
        l.enable_awe >> l.enable_bc >> l.bits >> l.group >> l.w8a8 >> l.forward >> l.fused_weight_pass >> l.ws >> l.ws_bytes >> l.status;
    if (!f.done()) return nullptr;
    PyObject* const members = PySequence_Fast(o[1], "a sequence of weights");
    if (!members) return nullptr;
    const Py_ssize_t count = PySequence_Fast_GET_SIZE(members);
    aweq_calib_weight few[4];
    aweq_calib_weight* const w = count <= 4 ? few : static_cast<aweq_calib_weight*>(PyMem_Malloc(count * sizeof(aweq_calib_weight)));
    PyObject* result = nullptr;
    void* stream = nullptr;
    bool ok = w != nullptr;
    if (!ok) PyErr_NoMemory();
    for (Py_ssize_t i = 0; ok && i < count; ++i) {
        Fields m(PySequence_Fast_GET_ITEM(members, i));
        m >> w[i].W >> w[i].N >> w[i].ldw >> w[i].W_hat >> w[i].ldwh >> w[i].codes >> w[i].step_w >> w[i].zero_w >> w[i].rowsum_w >> w[i].bias_in >>
            w[i].delta >> w[i].bias_out >> w[i].out_i32 >> w[i].out_deq >> w[i].colsum_acc;
        ok = m.done();
    }
    if (ok && convert(o[2], stream)) {
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = p_aweq_calibrate(&l, w, (int)count, stream);
        Py_END_ALLOW_THREADS
        result = PyLong_FromLong(rc);
    }
    if (w != few) PyMem_Free(w);
    Py_DECREF(members);
    return result;
}

// bind(name, address)
PyObject* bind_entry(PyObject*, PyObject* args)
{
    const char* name;
    unsigned long long address;
    if (!PyArg_ParseTuple(args, "sK", &name, &address)) return nullptr;
    const auto is = [&](const char* s) { return __builtin_strcmp(name, s) == 0; };
#define X(n) if (is(#n)) { p_##n = reinterpret_cast<decltype(p_##n)>((uintptr_t)address); Py_RETURN_NONE; }
    ENTRIES(X)
    X(aweq_calibrate)
#undef X
    PyErr_SetString(PyExc_KeyError, name);
    return nullptr;
}

#define X(n) {#n, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(call_##n)), METH_FASTCALL, nullptr},
PyMethodDef methods[] = {ENTRIES(X) X(aweq_calibrate) {"bind", bind_entry, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
#undef X
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native()
{
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    return s_data_ptr ? PyModule_Create(&module) : nullptr;
}
