// CPython extension over the C ABI (include/e2eg.h): one function per entry point, same name, same argument
// order.  It exists for the time of a call: through ctypes, with every tensor's address fetched in
// Python, the arguments of e2eg_propagate_fwd take 4 us, here under 1 us.
//
// A pointer argument may be None, an int address or an object with data_ptr() (a torch tensor).  The
// library runs without the interpreter lock.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstdint>
#include <tuple>
#include <type_traits>
#include <utility>

#include "../../include/e2eg.h"

namespace {

PyObject* g_data_ptr = nullptr;   // the interned method name

template <typename T>
bool convert(PyObject* o, T* out) {
    if constexpr (std::is_pointer<T>::value) {
        void* p = nullptr;
        if (o == Py_None) {
        } else if (PyLong_Check(o)) {
            p = PyLong_AsVoidPtr(o);
        } else {
            PyObject* r = PyObject_CallMethodNoArgs(o, g_data_ptr);
            if (!r) return false;
            p = PyLong_AsVoidPtr(r);
            Py_DECREF(r);
        }
        if (!p && PyErr_Occurred()) return false;
        *out = static_cast<T>(p);
    } else if constexpr (std::is_floating_point<T>::value) {
        const double v = PyFloat_AsDouble(o);
        if (v == -1.0 && PyErr_Occurred()) return false;
        *out = static_cast<T>(v);
    } else {   // as ctypes: no check of the range
        const unsigned long long v = PyLong_AsUnsignedLongLongMask(o);
        if (v == ~0ull && PyErr_Occurred()) return false;
        *out = static_cast<T>(v);
    }
    return true;
}

template <typename R, typename... A, size_t... I>
PyObject* call(R (*f)(A...), PyObject* const* args, std::index_sequence<I...>) {
    std::tuple<A...> a{};
    if (!(convert<A>(args[I], &std::get<I>(a)) && ...)) return nullptr;
    R r;
    Py_BEGIN_ALLOW_THREADS
    r = f(std::get<I>(a)...);
    Py_END_ALLOW_THREADS
    if constexpr (std::is_unsigned<R>::value) return PyLong_FromUnsignedLongLong(r);
    else return PyLong_FromLongLong(r);
}

template <typename R, typename... A>
PyObject* check_and_call(R (*f)(A...), PyObject* const* args, Py_ssize_t n) {
    if (n != (Py_ssize_t)sizeof...(A)) {
        PyErr_Format(PyExc_TypeError, "expected %d arguments, got %zd", (int)sizeof...(A), n);
        return nullptr;
    }
    return call(f, args, std::index_sequence_for<A...>());
}

template <auto F>
PyObject* wrap(PyObject*, PyObject* const* args, Py_ssize_t n) {
    return check_and_call(F, args, n);
}

#define ENTRY(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(&wrap<&name>)), METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {
    ENTRY(e2eg_build_csr_workspace_bytes),
    ENTRY(e2eg_build_csr),
    ENTRY(e2eg_sched_bytes),
    ENTRY(e2eg_sched_weighted_bytes),
    ENTRY(e2eg_normalize_workspace_bytes),
    ENTRY(e2eg_normalize),
    ENTRY(e2eg_normalize_weighted),
    ENTRY(e2eg_normalize_built),
    ENTRY(e2eg_sched_check_symmetric),
    ENTRY(e2eg_propagate_workspace_bytes),
    ENTRY(e2eg_propagate_fwd),
    ENTRY(e2eg_propagate_bwd),
    ENTRY(e2eg_propagate_weighted_fwd),
    ENTRY(e2eg_propagate_weighted_bwd),
    ENTRY(e2eg_edge_weights),
    ENTRY(e2eg_sampling_weights),
    ENTRY(e2eg_sampler_table_bytes),
    ENTRY(e2eg_sampler_prepare_workspace_bytes),
    ENTRY(e2eg_sampler_prepare),
    ENTRY(e2eg_sample_capacity),
    ENTRY(e2eg_sample_subgraph_workspace_bytes),
    ENTRY(e2eg_sample_subgraph),
    ENTRY(e2eg_layer_transform_workspace_bytes),
    ENTRY(e2eg_layer_transform),
    ENTRY(e2eg_layer_transform_noalloc),
    ENTRY(e2eg_readout_mean),
    ENTRY(e2eg_gfae_loss_workspace_bytes),
    ENTRY(e2eg_gfae_loss),
    ENTRY(e2eg_aggregate_workspace_bytes),
    ENTRY(e2eg_aggregate),
    ENTRY(e2eg_block_norms_workspace_bytes),
    ENTRY(e2eg_block_norms),
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_native", "libe2eg.so's entry points", -1, g_methods,
                        nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() {
    g_data_ptr = PyUnicode_InternFromString("data_ptr");
    if (!g_data_ptr) return nullptr;
    return PyModule_Create(&g_module);
}
