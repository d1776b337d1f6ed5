// Calls of libsentencekv's C entry points from Python without ctypes: a pointer argument is a tensor (its data pointer) or None (a null
// pointer), a number an integer.  Addresses as integers are taken for the context and for skv_segment's n_sent_host only, so that an
// argument in another one's place is refused here and does not go to the GPU as an address.  ctypes and the Python code around it took 2.4 to 4.8 us per call (an is_contiguous and a
// data_ptr call for every tensor, argument objects), more than the kernels of a short context run; this takes 0.3 to 0.7.
// Host code only.  The entry points are looked up in the library that `load` is given, once.
#include <Python.h>

#include <dlfcn.h>

#include <tuple>
#include <type_traits>
#include <utility>

#include <torch/csrc/autograd/python_variable.h>

#include "sentencekv.h"

#ifndef SKV_BUILT_FOR
#define SKV_BUILT_FOR ""
#endif

namespace {

// the Python and torch of this build: _build.py looks for it in the file, since the module only runs with them
__attribute__((used)) const char built_for[] = SKV_BUILT_FOR;

bool refuse(PyObject* o, const char* wanted) {
    PyErr_Format(PyExc_TypeError, "%s expected, got %.100s", wanted, Py_TYPE(o)->tp_name);
    return false;
}

// One Python argument as a C one; false with a Python exception set where it cannot be.
template <typename T, bool kAddress>
bool convert(PyObject* o, T* out) {
    if constexpr (kAddress) {
        if (o != Py_None && !PyLong_Check(o)) return refuse(o, "an address or None");
        const unsigned long long v = o == Py_None ? 0 : PyLong_AsUnsignedLongLong(o);
        if (v == (unsigned long long)-1 && PyErr_Occurred()) return false;
        *out = reinterpret_cast<T>(static_cast<uintptr_t>(v));
    } else if constexpr (std::is_pointer_v<T>) {
        if (o == Py_None) {
            *out = nullptr;
        } else if (THPVariable_Check(o)) {
            const at::Tensor& t = THPVariable_Unpack(o);
            if (!t.is_contiguous()) {
                PyErr_SetString(PyExc_AssertionError, "tensors handed to libsentencekv must be contiguous");
                return false;
            }
            *out = static_cast<T>(t.data_ptr());
        } else {
            return refuse(o, "a tensor or None");
        }
    } else {
        if (THPVariable_Check(o)) return refuse(o, "a number");
        const long long v = PyLong_AsLongLong(o);
        if (v == -1 && PyErr_Occurred()) return false;
        *out = static_cast<T>(v);
    }
    return true;
}

template <auto F> struct Call;
template <typename R, typename... A, R (*F)(A...)>
struct Call<F> {
    static inline R (*entry)(A...) = nullptr;      // in the loaded library; F only names the signature

    template <size_t I>
    static constexpr bool takes_address() {
        if constexpr (std::is_same_v<std::tuple_element_t<I, std::tuple<A...>>, skv_ctx*>) return true;
        else if constexpr (std::is_same_v<decltype(F), decltype(&skv_segment)>) return F == &skv_segment && I + 1 == sizeof...(A);
        else return false;
    }

    template <size_t... I>
    static PyObject* run(PyObject* const* args, std::index_sequence<I...>) {
        std::tuple<A...> v{};
        try {
            if (!(convert<A, takes_address<I>()>(args[I], &std::get<I>(v)) && ...)) return nullptr;
        } catch (const std::exception& e) {        // a tensor without storage
            PyErr_SetString(PyExc_RuntimeError, e.what());
            return nullptr;
        }
        R r;
        Py_BEGIN_ALLOW_THREADS
        r = entry(std::get<I>(v)...);
        Py_END_ALLOW_THREADS
        return PyLong_FromLongLong(static_cast<long long>(r));
    }
    static PyObject* method(PyObject*, PyObject* const* args, Py_ssize_t n) {
        if (n != (Py_ssize_t)sizeof...(A) || !entry) {
            PyErr_SetString(entry ? PyExc_TypeError : PyExc_RuntimeError, entry ? "wrong number of arguments" : "no library loaded");
            return nullptr;
        }
        return run(args, std::index_sequence_for<A...>{});
    }
    static bool find(void* lib, const char* name) {
        entry = reinterpret_cast<R (*)(A...)>(dlsym(lib, name));
        return entry != nullptr;
    }
};

#define SKV_CALLS(X)                                                                                                      \
    X(skv_segment) X(skv_build_semvec) X(skv_build_semvec_layers) X(skv_token_importance) X(skv_retain) X(skv_compact_pool) \
    X(skv_query_update) X(skv_score) X(skv_select) X(skv_gather) X(skv_attend) X(skv_decode_step) X(skv_merge_lse)

PyObject* load(PyObject*, PyObject* path) {
    const char* p = PyUnicode_AsUTF8(path);
    if (!p) return nullptr;
    void* lib = dlopen(p, RTLD_NOW | RTLD_LOCAL);
    if (!lib) {
        PyErr_SetString(PyExc_OSError, dlerror());
        return nullptr;
    }
#define FIND(name)                                                     \
    if (!Call<&name>::find(lib, #name)) {                              \
        PyErr_SetString(PyExc_AttributeError, "missing symbol " #name); \
        return nullptr;                                                \
    }
    SKV_CALLS(FIND)
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"load", load, METH_O, "looks the entry points up in the library at this path"},
#define METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&Call<&name>::method)), METH_FASTCALL, nullptr},
    SKV_CALLS(METHOD)
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls() { return PyModule_Create(&module); }
