// The per-call host work of the Python binding: arguments in, tensors over the result's device buffers out.
//
// A sampling call of a small bulk takes a few dozen microseconds on the device; building its argument structures with
// ctypes and one tensor per array through the CUDA array interface took as long again (about 15 us per call and 2.2 us
// per array; here 2 us and 0.4 us).  Everything else of the binding stays in bms.py.
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/ATen.h>
#include <vector>

#include "../../include/bms.h"

namespace {

// a tensor over device memory that belongs to `owner`, which it keeps alive
PyObject *view(const void *ptr, int64_t count, at::ScalarType type, int device, PyObject *owner)
{
    const at::TensorOptions opts = at::TensorOptions().dtype(type).device(at::Device(at::kCUDA, (c10::DeviceIndex)device));
    if (!ptr || count == 0)
        return THPVariable_Wrap(at::empty({0}, opts));
    Py_INCREF(owner);
    return THPVariable_Wrap(at::for_blob(const_cast<void *>(ptr), {count})
                                .deleter([owner](void *) {
                                    if (!Py_IsInitialized())
                                        return;
                                    const PyGILState_STATE gil = PyGILState_Ensure();
                                    Py_DECREF(owner);
                                    PyGILState_Release(gil);
                                })
                                .options(opts)
                                .target_device(opts.device())
                                .make_tensor());
}

void set(PyObject *tuple, int i, PyObject *item) { PyTuple_SET_ITEM(tuple, i, item); }

PyObject *none()
{
    Py_INCREF(Py_None);
    return Py_None;
}

bool complete(PyObject *tuple) // every item was made (a failed one left a Python error behind)
{
    for (Py_ssize_t i = 0; i < PyTuple_GET_SIZE(tuple); ++i)
        if (!PyTuple_GET_ITEM(tuple, i))
            return false;
    return true;
}

PyObject *hop_tuple(const bms_hop_view &v, int64_t k, int device, PyObject *owner)
{
    PyObject *t = PyTuple_New(14);
    if (!t)
        return nullptr;
    set(t, 0, PyLong_FromLongLong(v.rows));
    set(t, 1, PyLong_FromLongLong(v.nnz));
    set(t, 2, PyLong_FromLongLong(v.ncols));
    set(t, 3, PyLong_FromLongLong(v.pnnz));
    set(t, 4, view(v.mb_rowoff, k + 1, at::kLong, device, owner));
    set(t, 5, view(v.row_vertex, v.rows, at::kInt, device, owner));
    set(t, 6, view(v.rowptr, v.rows + 1, at::kLong, device, owner));
    set(t, 7, view(v.col, v.nnz, at::kInt, device, owner));
    set(t, 8, view(v.mb_coloff, k + 1, at::kLong, device, owner));
    set(t, 9, view(v.col_vertex, v.ncols, at::kInt, device, owner));
    set(t, 10, v.p_off ? view(v.p_off, k + 1, at::kLong, device, owner) : none());
    set(t, 11, v.p_off ? view(v.p_col, v.pnnz, at::kInt, device, owner) : none());
    set(t, 12, v.p_off ? view(v.p_cnt, v.pnnz, at::kInt, device, owner) : none());
    set(t, 13, v.row_self ? view(v.row_self, v.rows, at::kInt, device, owner) : none());
    if (!complete(t)) {
        Py_DECREF(t);
        return nullptr;
    }
    return t;
}

template <class F>
PyObject *guarded(F f)
{
    try {
        return f();
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

// hop(result, h, k, device, owner) -> the hop's fields, or the error code
PyObject *py_hop(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != 5) {
        PyErr_SetString(PyExc_TypeError, "hop takes 5 arguments");
        return nullptr;
    }
    bms_result *res = static_cast<bms_result *>(PyLong_AsVoidPtr(args[0]));
    const int32_t h = (int32_t)PyLong_AsLong(args[1]);
    const int64_t k = PyLong_AsLongLong(args[2]);
    const int device = (int)PyLong_AsLong(args[3]);
    if (PyErr_Occurred())
        return nullptr;
    bms_hop_view v;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = bms_result_hop(res, h, &v);
    Py_END_ALLOW_THREADS
    if (rc != BMS_OK)
        return PyLong_FromLong(rc);
    return guarded([&] { return hop_tuple(v, k, device, args[4]); });
}

// minibatch(result, h, i, device, owner) -> the minibatch's fields, or the error code
PyObject *py_minibatch(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != 5) {
        PyErr_SetString(PyExc_TypeError, "minibatch takes 5 arguments");
        return nullptr;
    }
    bms_result *res = static_cast<bms_result *>(PyLong_AsVoidPtr(args[0]));
    const int32_t h = (int32_t)PyLong_AsLong(args[1]), i = (int32_t)PyLong_AsLong(args[2]);
    const int device = (int)PyLong_AsLong(args[3]);
    if (PyErr_Occurred())
        return nullptr;
    PyObject *owner = args[4];
    bms_mb_view v;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = bms_result_minibatch(res, h, i, &v);
    Py_END_ALLOW_THREADS
    if (rc != BMS_OK)
        return PyLong_FromLong(rc);
    return guarded([&]() -> PyObject * {
        PyObject *t = PyTuple_New(11);
        if (!t)
            return nullptr;
        set(t, 0, PyLong_FromLongLong(v.rows));
        set(t, 1, PyLong_FromLongLong(v.nnz));
        set(t, 2, PyLong_FromLongLong(v.ncols));
        set(t, 3, PyLong_FromLongLong(v.row0));
        set(t, 4, PyLong_FromLongLong(v.edge0));
        set(t, 5, PyLong_FromLongLong(v.col0));
        set(t, 6, view(v.row_vertex, v.rows, at::kInt, device, owner));
        set(t, 7, view(v.rowptr, v.rows + 1, at::kLong, device, owner));
        set(t, 8, view(v.col, v.nnz, at::kInt, device, owner));
        set(t, 9, view(v.col_vertex, v.ncols, at::kInt, device, owner));
        set(t, 10, v.row_self ? view(v.row_self, v.rows, at::kInt, device, owner) : none());
        if (!complete(t)) {
            Py_DECREF(t);
            return nullptr;
        }
        return t;
    });
}

// sample(ladies, csr, batches, k, b, params, seed, stream, mb_base, flags, recycle, scratch_limit, alloc, dealloc)
// -> (error code, result)
PyObject *py_sample(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != 14 || !PyTuple_Check(args[5])) {
        PyErr_SetString(PyExc_TypeError, "sample takes 14 arguments, the parameters in a tuple");
        return nullptr;
    }
    const int ladies = PyObject_IsTrue(args[0]);
    bms_csr *csr = static_cast<bms_csr *>(PyLong_AsVoidPtr(args[1]));
    const int32_t *batches = static_cast<const int32_t *>(PyLong_AsVoidPtr(args[2]));
    const int32_t k = (int32_t)PyLong_AsLong(args[3]), b = (int32_t)PyLong_AsLong(args[4]);
    const Py_ssize_t L = PyTuple_GET_SIZE(args[5]);
    std::vector<int32_t> params((size_t)L);
    for (Py_ssize_t h = 0; h < L; ++h)
        params[(size_t)h] = (int32_t)PyLong_AsLong(PyTuple_GET_ITEM(args[5], h));
    const uint64_t seed = PyLong_AsUnsignedLongLongMask(args[6]);
    bms_opts o{};
    o.stream = PyLong_AsVoidPtr(args[7]);
    o.mb_base = (int32_t)PyLong_AsLong(args[8]);
    o.flags = (uint32_t)PyLong_AsUnsignedLong(args[9]);
    o.recycle = static_cast<bms_result *>(PyLong_AsVoidPtr(args[10]));
    o.scratch_limit = PyLong_AsLongLong(args[11]);
    o.alloc = reinterpret_cast<void *(*)(size_t, void *)>(PyLong_AsVoidPtr(args[12]));
    o.dealloc = reinterpret_cast<void (*)(void *, void *)>(PyLong_AsVoidPtr(args[13]));
    if (PyErr_Occurred())
        return nullptr;
    bms_result *out = nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS // the allocator's callbacks take the lock by themselves
    rc = (ladies ? bms_sample_ladies : bms_sample_nodewise)(csr, batches, k, b, params.data(), (int32_t)L, seed, &o, &out);
    Py_END_ALLOW_THREADS
    PyObject *t = PyTuple_New(2);
    if (!t)
        return nullptr;
    set(t, 0, PyLong_FromLong(rc));
    set(t, 1, PyLong_FromVoidPtr(out));
    return t;
}

PyMethodDef methods[] = {
    {"sample", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(py_sample)), METH_FASTCALL, nullptr},
    {"hop", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(py_hop)), METH_FASTCALL, nullptr},
    {"minibatch", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(py_minibatch)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

} // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&module); }
