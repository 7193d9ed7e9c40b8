// The calls that a program makes per tensor or per step, with the binding's argument checks in native code.
//
// A call on a small tensor is bound by the host: of 4.0 us for a step of a plan on 64 k elements the runtime's launch
// takes 2.4, and marshalling a list of 16 streams in Python took 10 of the 15.7 us of a small decode-and-sum and update.
//
// Every function takes the arguments of the binding's function of the same name, then the binding's `_stream`, which is
// asked for the stream once the arguments are known to be good.  It returns the library's status, or -1 and does nothing
// where an argument is anything but plainly good: the binding's own checks then say what is wrong, or convert it.
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <torch/csrc/autograd/python_variable.h>

#include <climits>

#include "cdsgd.h"

namespace {

struct Library {
    decltype(&cdsgd_quantize_pack) quantize_pack;
    decltype(&cdsgd_decode_sum) decode_sum;
    decltype(&cdsgd_decode_sum_sparse) decode_sum_sparse;
    decltype(&cdsgd_update) update;
    decltype(&cdsgd_sparse_encode) sparse_encode;
    decltype(&cdsgd_sparse_words) sparse_words;
    decltype(&cdsgd_sparse_segments) sparse_segments;
    decltype(&cdsgd_step_fused) step_fused;
    decltype(&cdsgd_step_fused_range) step_fused_range;
    decltype(&cdsgd_step_fused_static) step_fused_static;
} lib;

struct NotPlain {};  // leave it to the binding

size_t packed_words(size_t n) { return (n + 15) / 16; }

// A dense contiguous tensor on the GPU, not of a subclass, with `n` elements (kAny: any number).
constexpr size_t kAny = (size_t)-1;
void *buffer(PyObject *o, at::ScalarType type, size_t n, size_t *numel = nullptr)
{
    if (!THPVariable_CheckExact(o)) throw NotPlain();
    const at::Tensor &t = THPVariable_Unpack(o);
    if (t.scalar_type() != type || !t.is_cuda() || !t.is_contiguous()) throw NotPlain();
    const size_t have = (size_t)t.numel();
    if (n != kAny && have != n) throw NotPlain();
    if (numel) *numel = have;
    return t.data_ptr();
}

float *floats(PyObject *o, size_t n, size_t *numel = nullptr) { return static_cast<float *>(buffer(o, at::kFloat, n, numel)); }
float *floats_or_null(PyObject *o, size_t n) { return o == Py_None ? nullptr : floats(o, n); }
uint32_t *words(PyObject *o, size_t n) { return static_cast<uint32_t *>(buffer(o, at::kInt, n)); }

float number(PyObject *o)
{
    if (PyFloat_CheckExact(o)) return (float)PyFloat_AS_DOUBLE(o);
    throw NotPlain();
}

long whole(PyObject *o)
{
    if (!PyLong_CheckExact(o)) throw NotPlain();
    int over = 0;
    const long v = PyLong_AsLongAndOverflow(o, &over);
    if (over) throw NotPlain();
    return v;
}

int small(PyObject *o)
{
    const long v = whole(o);
    if (v < INT_MIN || v > INT_MAX) throw NotPlain();
    return (int)v;
}

template <typename T>
T *address(PyObject *o)
{
    if (!PyLong_CheckExact(o)) throw NotPlain();
    void *p = PyLong_AsVoidPtr(o);
    if (!p && PyErr_Occurred()) {
        PyErr_Clear();
        throw NotPlain();
    }
    return static_cast<T *>(p);
}

struct Raised {};  // a Python error is set

void *stream_of(PyObject *lookup)
{
    PyObject *s = PyObject_CallNoArgs(lookup);
    if (!s) throw Raised();
    void *p = PyLong_Check(s) ? PyLong_AsVoidPtr(s) : nullptr;
    const bool bad = !PyLong_Check(s) || (!p && PyErr_Occurred());
    Py_DECREF(s);
    if (bad) {
        PyErr_Clear();
        throw NotPlain();
    }
    return p;
}

// `call` does what a function does with its arguments; the lock is given up inside it, around the library's part.
template <typename Call>
PyObject *guarded(Py_ssize_t have, Py_ssize_t want, Call call)
{
    int status = -1;
    if (have == want && lib.update && !at::impl::torch_function_mode_enabled()) {
        try {
            status = call();
        } catch (const Raised &) {
            return nullptr;
        } catch (...) {
            status = -1;  // (a tensor without storage, a layout without strides: the binding says what it is)
        }
    }
    return PyLong_FromLong(status);
}

template <typename Call>
int unlocked(Call call)
{
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = call();
    Py_END_ALLOW_THREADS
    return status;
}

PyObject *quantize_pack(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 5, [&] {
        size_t count;
        const float *grad = floats(a[0], kAny, &count);
        float *residual = floats(a[1], count);
        uint32_t *packed = words(a[2], packed_words(count));
        const float t = number(a[3]);
        void *s = stream_of(a[4]);
        return unlocked([&] { return lib.quantize_pack(grad, residual, packed, count, t, s); });
    });
}

PyObject *decode(PyObject *const *a, Py_ssize_t n, bool sparse)
{
    return guarded(n, 4, [&] {
        if (!PyList_CheckExact(a[0]) && !PyTuple_CheckExact(a[0])) throw NotPlain();
        const Py_ssize_t workers = PySequence_Fast_GET_SIZE(a[0]);
        if (workers < 1 || workers > CDSGD_MAX_WORKERS) throw NotPlain();
        size_t count;
        float *agg = floats(a[1], kAny, &count);
        const size_t each = sparse ? lib.sparse_words(count) : packed_words(count);
        const uint32_t *streams[CDSGD_MAX_WORKERS];
        for (Py_ssize_t j = 0; j < workers; ++j) streams[j] = words(PySequence_Fast_GET_ITEM(a[0], j), each);
        const float t = number(a[2]);
        void *s = stream_of(a[3]);
        const auto f = sparse ? lib.decode_sum_sparse : lib.decode_sum;
        return unlocked([&] { return f(streams, (int)workers, agg, count, t, s); });
    });
}

PyObject *decode_sum(PyObject *, PyObject *const *a, Py_ssize_t n) { return decode(a, n, false); }
PyObject *decode_sum_sparse(PyObject *, PyObject *const *a, Py_ssize_t n) { return decode(a, n, true); }

PyObject *update(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 8, [&] {
        size_t count;
        float *w_global = floats(a[0], kAny, &count);
        float *w_local = floats_or_null(a[1], count);
        const float *grad = floats_or_null(a[2], count);
        const float *agg = floats_or_null(a[3], count);
        const float lr_local = number(a[4]), lr_global = number(a[5]);
        const int workers = small(a[6]);
        void *s = stream_of(a[7]);
        return unlocked([&] { return lib.update(w_global, w_local, grad, agg, count, lr_local, lr_global, workers, s); });
    });
}

PyObject *sparse_encode(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 5, [&] {
        const long count = whole(a[1]);
        if (count < 1) throw NotPlain();
        const uint32_t *packed = words(a[0], packed_words((size_t)count));
        uint32_t *sparse = words(a[2], lib.sparse_words((size_t)count));
        uint32_t *counts = a[3] == Py_None ? nullptr : words(a[3], lib.sparse_segments((size_t)count));
        void *s = stream_of(a[4]);
        return unlocked([&] { return lib.sparse_encode(packed, (size_t)count, sparse, counts, s); });
    });
}

PyObject *step(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 7, [&] {
        cdsgd_plan *plan = address<cdsgd_plan>(a[0]);
        const long i = whole(a[1]);
        const int k = small(a[2]);
        const float t = number(a[3]), lr_local = number(a[4]), lr_global = number(a[5]);
        void *s = stream_of(a[6]);
        return unlocked([&] { return lib.step_fused(plan, i, k, t, lr_local, lr_global, s); });
    });
}

PyObject *step_range(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 9, [&] {
        cdsgd_plan *plan = address<cdsgd_plan>(a[0]);
        const int first = small(a[1]), count = small(a[2]);
        const long i = whole(a[3]);
        const int k = small(a[4]);
        const float t = number(a[5]), lr_local = number(a[6]), lr_global = number(a[7]);
        void *s = stream_of(a[8]);
        return unlocked([&] { return lib.step_fused_range(plan, first, count, i, k, t, lr_local, lr_global, s); });
    });
}

PyObject *step_static(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 12, [&] {
        const cdsgd_tensor *tensors = address<const cdsgd_tensor>(a[0]);
        const int num_tensors = small(a[1]);
        const uint32_t *const *const *peers = address<const uint32_t *const *const>(a[2]);
        const int workers = small(a[3]), self = small(a[4]), dtype = small(a[5]);
        const long i = whole(a[6]);
        const int k = small(a[7]);
        const float t = number(a[8]), lr_local = number(a[9]), lr_global = number(a[10]);
        void *s = stream_of(a[11]);
        return unlocked([&] {
            return lib.step_fused_static(tensors, num_tensors, peers, workers, self, dtype, i, k, t, lr_local, lr_global, s);
        });
    });
}

// bind(addresses of the library's functions, in the order of `Library`)
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    void *p[sizeof(Library) / sizeof(void *)];
    if (n != (Py_ssize_t)(sizeof(p) / sizeof(p[0]))) {
        PyErr_SetString(PyExc_TypeError, "bind takes an address for each of the library's functions");
        return nullptr;
    }
    for (Py_ssize_t i = 0; i < n; ++i) {
        p[i] = PyLong_AsVoidPtr(a[i]);
        if (!p[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "an address is 0");
            return nullptr;
        }
    }
    static_assert(sizeof(Library) == sizeof(p), "nothing but function pointers");
    __builtin_memcpy(&lib, p, sizeof(p));
    Py_RETURN_NONE;
}

template <typename F>
PyMethodDef method(const char *name, F f)
{
    return {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr};
}

PyMethodDef methods[] = {method("bind", bind), method("quantize_pack", quantize_pack), method("decode_sum", decode_sum),
                         method("decode_sum_sparse", decode_sum_sparse), method("update", update),
                         method("sparse_encode", sparse_encode), method("step", step), method("step_range", step_range),
                         method("step_static", step_static), {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

#ifndef CDSGD_BUILD_ID_HEX
#define CDSGD_BUILD_ID_HEX "0000000000000000"
#endif
#ifndef CDSGD_CALLS_LIBRARY
#define CDSGD_CALLS_LIBRARY ""
#define CDSGD_CALLS_TORCH ""
#define CDSGD_CALLS_SOABI ""
#endif

// The identity of what the module was built from; the marker makes it findable in the file.
extern "C" __attribute__((used, visibility("default"))) const char cdsgd_calls_id[] = "CDSGD_BUILD_ID=" CDSGD_BUILD_ID_HEX;

// made_for: the library (its identity), the torch and the Python that the module may be used with.
PyMODINIT_FUNC PyInit__calls(void)
{
    PyObject *m = PyModule_Create(&module);
    if (!m) return nullptr;
    PyObject *made_for = Py_BuildValue("(sss)", CDSGD_CALLS_LIBRARY, CDSGD_CALLS_TORCH, CDSGD_CALLS_SOABI);
    if (!made_for || PyModule_AddObject(m, "made_for", made_for) != 0) {
        Py_XDECREF(made_for);
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
