// The calls that a training or inference loop makes, from Python objects to the C ABI in one step.
// Through ctypes a call spends as much on its arguments as the library does on a launch -- data_ptr() and three properties of
// every tensor, each a Python call, then the conversions: 1.8 us for sparse_linear_forward, 3.3 for
// sparse_linear_backward (with an empty function in the place of either), 0.14 and 0.15 here.  The entry points come as addresses from the library that the
// package has loaded (bind), so that there is one copy of it in the process.  Every call releases the interpreter lock and returns the
// status code.
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

namespace {

using Forward = int (*)(const void *, const float *, int32_t, float *, int32_t, int32_t, void *);
using Backward = int (*)(void *, const float *, int32_t, const float *, int32_t, const float *, int32_t, float *, int32_t, float *, float *,
                         int32_t, void *);
using Update = int (*)(float *, float *, const float *, int64_t, float, float, void *);
using TrainStep = int (*)(void *, const float *, int32_t, const int32_t *, int32_t, float, float, void *, size_t, float *, void *);
using MlpForward = int (*)(void *, const float *, int32_t, int32_t, void *, size_t, void *);

Forward g_forward;
Backward g_backward;
Update g_update, g_update_nesterov;
TrainStep g_train_step;
MlpForward g_mlp_forward;

// Reads the arguments of one call in order; the first that cannot be read leaves a Python exception and `ok` false.
struct Args {
    PyObject *const *v;
    bool ok = true;

    int64_t integer()
    {
        PyObject *o = *v++;
        if (!ok) return 0;
        const long long x = PyLong_AsLongLong(o);
        if (x == -1 && PyErr_Occurred()) ok = false;
        return x;
    }
    float real()
    {
        PyObject *o = *v++;
        if (!ok) return 0.f;
        const double x = PyFloat_AsDouble(o);
        if (x == -1.0 && PyErr_Occurred()) ok = false;
        return static_cast<float>(x);
    }
    // a handle or address as an int, or None
    void *address()
    {
        PyObject *o = *v++;
        if (!ok || o == Py_None) return nullptr;
        void *p = PyLong_AsVoidPtr(o);
        if (!p && PyErr_Occurred()) ok = false;
        return p;
    }
    const at::Tensor *tensor(PyObject *o)
    {
        if (THPVariable_Check(o)) return &THPVariable_Unpack(o);
        PyErr_SetString(PyExc_TypeError, "expected a tensor");
        ok = false;
        return nullptr;
    }
    // a tensor's memory, or None
    void *memory()
    {
        PyObject *o = *v++;
        if (!ok || o == Py_None) return nullptr;
        const at::Tensor *t = tensor(o);
        return t ? t->data_ptr() : nullptr;
    }
    // the same, or an address as an int
    void *memory_or_address()
    {
        if (PyLong_Check(*v)) return address();
        return memory();
    }
    void *buffer(size_t &bytes)
    {
        PyObject *o = *v++;
        bytes = 0;
        const at::Tensor *t = ok ? tensor(o) : nullptr;
        if (!t) return nullptr;
        bytes = t->nbytes();
        return t->data_ptr();
    }
    // a float32 matrix with unit column stride and its leading dimension, or None
    float *matrix(int32_t &ld)
    {
        PyObject *o = *v++;
        ld = 0;
        if (!ok || o == Py_None) return nullptr;
        const at::Tensor *t = tensor(o);
        if (!t) return nullptr;
        if (t->dim() != 2 || t->stride(1) != 1 || t->scalar_type() != at::kFloat) {
            PyErr_SetString(PyExc_AssertionError, "expected a float32 matrix with contiguous rows");
            ok = false;
            return nullptr;
        }
        ld = static_cast<int32_t>(t->stride(0));
        return static_cast<float *>(t->data_ptr());
    }
    // a matrix, or an address, followed by its leading dimension: None takes the matrix's own
    float *matrix_with_ld(int32_t &ld)
    {
        if (v[1] == Py_None) {
            float *p = matrix(ld);
            ++v;
            return p;
        }
        float *p = static_cast<float *>(memory_or_address());
        ld = static_cast<int32_t>(integer());
        return p;
    }
    // None: torch's current stream; a torch stream; or a handle
    void *stream()
    {
        PyObject *o = *v++;
        if (!ok) return nullptr;
        if (o == Py_None) return c10::hip::getCurrentHIPStream().stream();
        if (PyLong_Check(o)) return PyLong_AsVoidPtr(o);
        PyObject *h = PyObject_GetAttrString(o, "cuda_stream");
        if (!h) {
            ok = false;
            return nullptr;
        }
        void *s = PyLong_AsVoidPtr(h);
        Py_DECREF(h);
        if (!s && PyErr_Occurred()) ok = false;
        return s;
    }
};

// Runs `call`, which reads its arguments and returns a closure for the library call.
template <typename F>
PyObject *run(PyObject *const *args, Py_ssize_t n, Py_ssize_t expected, F &&read)
{
    if (n != expected) {
        PyErr_Format(PyExc_TypeError, "%zd arguments, %zd expected", n, expected);
        return nullptr;
    }
    try {
        Args a{args};
        auto call = read(a);
        if (!a.ok) return nullptr;
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = call();
        Py_END_ALLOW_THREADS
        return PyLong_FromLong(rc);
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

// (layer, X, Y, batch, stream)
PyObject *forward(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return run(args, n, 5, [](Args &a) {
        int32_t ldx, ldy;
        const void *layer = a.address();
        const float *X = a.matrix(ldx);
        float *Y = a.matrix(ldy);
        const int32_t batch = static_cast<int32_t>(a.integer());
        void *s = a.stream();
        return [=] { return g_forward(layer, X, ldx, Y, ldy, batch, s); };
    });
}

// (layer, X, Y, dY, dX, dvalues, dbias, batch, stream)
PyObject *backward(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return run(args, n, 9, [](Args &a) {
        int32_t ldx, ldy, lddy, lddx;
        void *layer = a.address();
        const float *X = a.matrix(ldx), *Y = a.matrix(ldy), *dY = a.matrix(lddy);
        float *dX = a.matrix(lddx), *dv = static_cast<float *>(a.memory()), *db = static_cast<float *>(a.memory());
        const int32_t batch = static_cast<int32_t>(a.integer());
        void *s = a.stream();
        return [=] { return g_backward(layer, X, ldx, Y, ldy, dY, lddy, dX, lddx, dv, db, batch, s); };
    });
}

// (values, velocity, grad, n, lr, momentum, nesterov, stream)
PyObject *update(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return run(args, n, 8, [](Args &a) {
        float *w = static_cast<float *>(a.memory()), *v = static_cast<float *>(a.memory());
        const float *g = static_cast<const float *>(a.memory());
        const int64_t count = a.integer();
        const float lr = a.real(), mu = a.real();
        const Update f = a.integer() ? g_update_nesterov : g_update;
        void *s = a.stream();
        return [=] { return f(w, v, g, count, lr, mu, s); };
    });
}

// (mlp, X, ldx, labels, batch, lr, momentum, workspace, loss, stream)
PyObject *train_step(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return run(args, n, 10, [](Args &a) {
        void *mlp = a.address();
        int32_t ldx;
        const float *X = a.matrix_with_ld(ldx);
        const int32_t *labels = static_cast<const int32_t *>(a.memory_or_address());
        const int32_t batch = static_cast<int32_t>(a.integer());
        const float lr = a.real(), mu = a.real();
        size_t bytes;
        void *ws = a.buffer(bytes);
        float *loss = static_cast<float *>(a.memory());
        void *s = a.stream();
        return [=] { return g_train_step(mlp, X, ldx, labels, batch, lr, mu, ws, bytes, loss, s); };
    });
}

// (mlp, X, ldx, batch, workspace, stream)
PyObject *mlp_forward(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return run(args, n, 6, [](Args &a) {
        void *mlp = a.address();
        int32_t ldx;
        const float *X = a.matrix_with_ld(ldx);
        const int32_t batch = static_cast<int32_t>(a.integer());
        size_t bytes;
        void *ws = a.buffer(bytes);
        void *s = a.stream();
        return [=] { return g_mlp_forward(mlp, X, ldx, batch, ws, bytes, s); };
    });
}

// (workspace, rows, batch, ld, offset in floats): the (rows, batch) matrix there
PyObject *view(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != 5) {
        PyErr_Format(PyExc_TypeError, "%zd arguments, 5 expected", n);
        return nullptr;
    }
    try {
        Args a{args + 1};
        const at::Tensor *ws = a.tensor(args[0]);
        const int64_t rows = a.integer(), batch = a.integer(), ld = a.integer(), offset = a.integer();
        if (!a.ok) return nullptr;
        return THPVariable_Wrap(ws->as_strided({rows, batch}, {ld, 1}, ws->storage_offset() + offset));
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

// addresses of sparse_linear_forward, sparse_linear_backward, sgd_update_values, sgd_update_values_nesterov, mlp_train_step, mlp_forward
PyObject *bind(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != 6) {
        PyErr_SetString(PyExc_TypeError, "six addresses expected");
        return nullptr;
    }
    Args a{args};
    g_forward = reinterpret_cast<Forward>(a.address());
    g_backward = reinterpret_cast<Backward>(a.address());
    g_update = reinterpret_cast<Update>(a.address());
    g_update_nesterov = reinterpret_cast<Update>(a.address());
    g_train_step = reinterpret_cast<TrainStep>(a.address());
    g_mlp_forward = reinterpret_cast<MlpForward>(a.address());
    if (!a.ok) return nullptr;
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(bind)), METH_FASTCALL, nullptr},
    {"forward", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(forward)), METH_FASTCALL, nullptr},
    {"backward", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(backward)), METH_FASTCALL, nullptr},
    {"update", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(update)), METH_FASTCALL, nullptr},
    {"train_step", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(train_step)), METH_FASTCALL, nullptr},
    {"mlp_forward", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(mlp_forward)), METH_FASTCALL, nullptr},
    {"view", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(view)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall() { return PyModule_Create(&module); }
