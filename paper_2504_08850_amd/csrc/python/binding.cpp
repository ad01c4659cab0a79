// Python entry points of libspecee.so that a decode loop calls per layer: argument marshalling only, driven by the
// C signatures of include/specee.h.  An eager specee_predict through ctypes, with a Python object per pointer, took
// 11.4 us beside a kernel of 3.4 us; through this file it takes 4.6 us, a call on a token tree 7.9 instead of 17.4 us.
//
// How a Python argument becomes a C one:
//   const T *            tensor of T's type on the GPU, contiguous, or None
//   T *                  the same without a check of the type (outputs); void *: any tensor
//   const specee_dims *  tuple (d, V, K, H, eps, threshold)
//   const specee_mlp *   tuple (W1, b1, w2, b2) of fp16 tensors or None
//   integers             anything with __index__
//   last argument        the stream: None (the current one) or its handle
// The tensors outlive the call: the caller's argument list holds them.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/version.h>

#include <tuple>
#include <utility>

#include "../../../include/specee.h"

namespace {

bool tensor_ptr(PyObject *o, const c10::ScalarType *type, void **out) {
    *out = nullptr;
    if (o == Py_None) return true;
    if (!THPVariable_Check(o)) {
        PyErr_Format(PyExc_TypeError, "a tensor is expected, not %s", Py_TYPE(o)->tp_name);
        return false;
    }
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.is_cuda() || !t.is_contiguous()) {
        PyErr_SetString(PyExc_AssertionError, "device-resident contiguous tensors only");
        return false;
    }
    if (type && t.scalar_type() != *type) {
        PyErr_Format(PyExc_AssertionError, "a tensor of type %s is expected, not %s", c10::toString(*type),
                     c10::toString(t.scalar_type()));
        return false;
    }
    *out = t.data_ptr();
    return true;
}

template <class T>
struct Elem;
template <>
struct Elem<specee_half> {
    static constexpr c10::ScalarType type = c10::ScalarType::Half;
};
template <>
struct Elem<float> {
    static constexpr c10::ScalarType type = c10::ScalarType::Float;
};
template <>
struct Elem<int32_t> {
    static constexpr c10::ScalarType type = c10::ScalarType::Int;
};
template <>
struct Elem<uint32_t> {  // words travel as int32
    static constexpr c10::ScalarType type = c10::ScalarType::Int;
};

// Arg<A>: storage for one C argument of type A and its conversion
template <class A>
struct Arg;

template <class T>
struct Arg<const T *> {
    void *p;
    bool from(PyObject *o) {
        const c10::ScalarType t = Elem<T>::type;
        return tensor_ptr(o, &t, &p);
    }
    const T *get() { return static_cast<const T *>(p); }
};
template <class T>
struct Arg<T *> {
    void *p;
    bool from(PyObject *o) { return tensor_ptr(o, nullptr, &p); }
    T *get() { return static_cast<T *>(p); }
};

template <class I>
struct IntArg {
    long long v;
    bool from(PyObject *o) {
        v = PyLong_AsLongLong(o);
        return !(v == -1 && PyErr_Occurred());
    }
    I get() { return static_cast<I>(v); }
};
template <>
struct Arg<int> : IntArg<int> {};
template <>
struct Arg<long long> : IntArg<long long> {};
template <>
struct Arg<size_t> : IntArg<size_t> {};

bool tuple_of(PyObject *o, Py_ssize_t n) {
    if (PyTuple_Check(o) && PyTuple_GET_SIZE(o) == n) return true;
    PyErr_Format(PyExc_TypeError, "a tuple of %zd values is expected", n);
    return false;
}

template <>
struct Arg<const specee_dims *> {
    specee_dims dims;
    bool from(PyObject *o) {
        if (!tuple_of(o, 6)) return false;
        int32_t *field[4] = {&dims.d, &dims.V, &dims.K, &dims.H};
        for (int i = 0; i < 4; ++i) {
            const long long v = PyLong_AsLongLong(PyTuple_GET_ITEM(o, i));
            if (v == -1 && PyErr_Occurred()) return false;
            *field[i] = static_cast<int32_t>(v);
        }
        const double eps = PyFloat_AsDouble(PyTuple_GET_ITEM(o, 4));
        if (eps == -1.0 && PyErr_Occurred()) return false;
        const double thr = PyFloat_AsDouble(PyTuple_GET_ITEM(o, 5));
        if (thr == -1.0 && PyErr_Occurred()) return false;
        dims.eps = static_cast<float>(eps);
        dims.threshold = static_cast<float>(thr);
        return true;
    }
    const specee_dims *get() { return &dims; }
};

template <>
struct Arg<const specee_mlp *> {
    specee_mlp mlp;
    bool from(PyObject *o) {
        if (!tuple_of(o, 4)) return false;
        const c10::ScalarType half = c10::ScalarType::Half;
        void *p[4];
        for (int i = 0; i < 4; ++i)
            if (!tensor_ptr(PyTuple_GET_ITEM(o, i), &half, &p[i])) return false;
        mlp.W1 = static_cast<const specee_half *>(p[0]);
        mlp.b1 = static_cast<const specee_half *>(p[1]);
        mlp.w2 = static_cast<const specee_half *>(p[2]);
        mlp.b2 = static_cast<const specee_half *>(p[3]);
        return true;
    }
    const specee_mlp *get() { return &mlp; }
};

bool stream_handle(PyObject *o, void **out) {
    if (o == Py_None) {
        *out = c10::hip::getCurrentHIPStream().stream();
        return true;
    }
    *out = PyLong_AsVoidPtr(o);
    return !PyErr_Occurred();
}

// F: a C entry point whose last parameter is the stream.  Returns its status.
template <class... A, size_t... I>
PyObject *invoke(int (*f)(A...), PyObject *const *args, std::index_sequence<I...>) {
    std::tuple<Arg<std::tuple_element_t<I, std::tuple<A...>>>...> c;
    void *stream = nullptr;
    // in order, the stream last
    if (!((std::get<I>(c).from(args[I])) && ...) || !stream_handle(args[sizeof...(I)], &stream)) return nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f(std::get<I>(c).get()..., stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

template <class... A>
PyObject *checked(int (*f)(A...), PyObject *const *args, Py_ssize_t n) {
    if (n != (Py_ssize_t)sizeof...(A)) {
        PyErr_Format(PyExc_TypeError, "%zu arguments are expected, not %zd", sizeof...(A), n);
        return nullptr;
    }
    try {
        return invoke(f, args, std::make_index_sequence<sizeof...(A) - 1>{});
    } catch (const std::exception &e) {  // a tensor without storage, a stream query that fails
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

template <auto F>
PyObject *entry(PyObject *, PyObject *const *args, Py_ssize_t n) {
    return checked(F, args, n);
}

#define SPECEE_ENTRY(name) {#name, reinterpret_cast<PyCFunction>(&entry<&name>), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    SPECEE_ENTRY(specee_predict),        SPECEE_ENTRY(specee_predict_q4),
    SPECEE_ENTRY(specee_predict_sweep),  SPECEE_ENTRY(specee_predict_tree),
    SPECEE_ENTRY(specee_predict_tree_static), SPECEE_ENTRY(specee_predict_tree_q4),
    SPECEE_ENTRY(lm_head_gemv),          SPECEE_ENTRY(lm_head_gemv_q4),
    SPECEE_ENTRY(specee_verify),         SPECEE_ENTRY(specee_verify_q4),
    SPECEE_ENTRY(specee_layer_loop),     SPECEE_ENTRY(specee_layer_loop_q4),
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", "Argument marshalling of libspecee.so", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void) {
    PyObject *m = PyModule_Create(&module);
    // what this file was compiled against: tensors of another version may be laid out differently
    if (m && PyModule_AddStringConstant(m, "torch_version", TORCH_VERSION) < 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
