// The calls of a planning step (kvsched_sortedF, kvsched_simulate, kvsched_argmin) from Python: checks, output tensors and the call in
// one native function each.
//
// Bound by the host: for a short backlog the calls' kernels take less time than their arguments.  Of the 9.8 / 8.4 / 5.6 us the three
// took before the Python code returned, 3.3 are the launch; the rest was one tensor after the other made through Python (1.25 us
// each), checked there (0.25) and passed through ctypes (1.2): 6.6 / 5.0 / 4.1 us now, and an order of 61 requests with its timeline 24.6 ->
// 18.5 us.  Whatever is not the plain case (another type, not contiguous, a subclass of Tensor, output tensors of the caller's) gets None here
// and takes the Python path, which also says what is wrong with an argument.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ops/empty.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/version.h>

#include <utility>

#include "../../include/kvsched.h"

namespace {

// The tensor `x` if it is a plain one of this type, contiguous and on a GPU; null otherwise.
const at::Tensor *plain(PyObject *x, at::ScalarType type)
{
    if (!THPVariable_CheckExact(x)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(x);
    return t.is_cuda() && t.scalar_type() == type && t.is_contiguous() ? &t : nullptr;
}

at::Tensor fresh(const at::Tensor &like, at::ScalarType type, at::IntArrayRef sizes) { return at::empty(sizes, like.options().dtype(type)); }

template <class T>
T *data(const at::Tensor &t) { return static_cast<T *>(t.data_ptr()); }

// An int as ctypes passes it on: its lowest bits.
long long number(PyObject *x) { return (long long)PyLong_AsUnsignedLongLongMask(x); }

kvsched_ctx *context(PyObject *x) { return static_cast<kvsched_ctx *>(PyLong_AsVoidPtr(x)); }

// (return code, outputs ...); an undefined tensor is None.
template <class... Tensors>
PyObject *result(int rc, Tensors... outputs)
{
    PyObject *r = PyTuple_New(1 + sizeof...(outputs));
    if (!r) return nullptr;
    PyObject *const items[] = {PyLong_FromLong(rc), THPVariable_Wrap(std::move(outputs))...};
    bool whole = true;
    for (size_t i = 0; i < 1 + sizeof...(outputs); ++i) {
        whole = whole && items[i];
        PyTuple_SET_ITEM(r, (Py_ssize_t)i, items[i]);
    }
    if (!whole) {
        Py_DECREF(r);
        return nullptr;
    }
    return r;
}

// No C++ exception leaves: the Python path makes the call again and raises what there is to raise.
template <class Call>
PyObject *guarded(Call call)
{
    try {
        return call();
    } catch (...) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

// (context, s, o, M, tie_rule, feas_mode, stream) -> (rc, order, batch_end, F, num_batches)
PyObject *sortedF(PyObject *, PyObject *const *a, Py_ssize_t count)
{
    return guarded([&]() -> PyObject * {
        const at::Tensor *s, *o;
        if (count != 7 || !(s = plain(a[1], at::kInt)) || !(o = plain(a[2], at::kInt)) || s->dim() < 1) Py_RETURN_NONE;
        kvsched_ctx *ctx = context(a[0]);
        const long long M = number(a[3]);
        const int32_t tie_rule = (int32_t)number(a[4]), feas_mode = (int32_t)number(a[5]);
        void *stream = PyLong_AsVoidPtr(a[6]);
        if (PyErr_Occurred()) return nullptr;
        const int64_t n = s->size(0);
        at::Tensor order = fresh(*s, at::kInt, {n}), ends = fresh(*s, at::kInt, {n}), F = fresh(*s, at::kDouble, {n}), nb = fresh(*s, at::kInt, {1});
        const int32_t *sp = data<int32_t>(*s), *op = data<int32_t>(*o);
        int32_t *order_p = data<int32_t>(order), *ends_p = data<int32_t>(ends), *nb_p = data<int32_t>(nb);
        double *F_p = data<double>(F);
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = kvsched_sortedF(ctx, (int32_t)n, sp, op, M, tie_rule, feas_mode, order_p, ends_p, F_p, nb_p, stream);
        Py_END_ALLOW_THREADS
        return result(rc, std::move(order), std::move(ends), std::move(F), std::move(nb));
    });
}

// (context, orders, s, o, M, completions, common_prefix, stream) -> (rc, tel, completion or None)
PyObject *simulate(PyObject *, PyObject *const *a, Py_ssize_t count)
{
    return guarded([&]() -> PyObject * {
        const at::Tensor *orders, *s, *o;
        if (count != 8 || !(orders = plain(a[1], at::kInt)) || !(s = plain(a[2], at::kInt)) || !(o = plain(a[3], at::kInt)) || orders->dim() != 2)
            Py_RETURN_NONE;
        kvsched_ctx *ctx = context(a[0]);
        const long long M = number(a[4]);
        const int wanted = PyObject_IsTrue(a[5]);
        const int32_t common_prefix = (int32_t)number(a[6]);
        void *stream = PyLong_AsVoidPtr(a[7]);
        if (PyErr_Occurred()) return nullptr;
        const int64_t C = orders->size(0), n = orders->size(1);
        at::Tensor tel = fresh(*orders, at::kLong, {C}), completion;
        if (wanted) completion = fresh(*orders, at::kInt, {C, n});
        const int32_t *orders_p = data<int32_t>(*orders), *sp = data<int32_t>(*s), *op = data<int32_t>(*o);
        int64_t *tel_p = data<int64_t>(tel);
        int32_t *completion_p = wanted ? data<int32_t>(completion) : nullptr;
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = kvsched_simulate(ctx, orders_p, (int32_t)C, (int32_t)n, sp, op, M, tel_p, completion_p, common_prefix, stream);
        Py_END_ALLOW_THREADS
        return result(rc, std::move(tel), std::move(completion));
    });
}

// (context, tel, stream) -> (rc, result)
PyObject *argmin(PyObject *, PyObject *const *a, Py_ssize_t count)
{
    return guarded([&]() -> PyObject * {
        const at::Tensor *tel;
        if (count != 3 || !(tel = plain(a[1], at::kLong)) || tel->dim() < 1) Py_RETURN_NONE;
        kvsched_ctx *ctx = context(a[0]);
        void *stream = PyLong_AsVoidPtr(a[2]);
        if (PyErr_Occurred()) return nullptr;
        at::Tensor best = fresh(*tel, at::kLong, {2});
        const int64_t *tel_p = data<int64_t>(*tel);
        int64_t *best_p = data<int64_t>(best);
        const int32_t C = (int32_t)tel->size(0);
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = kvsched_argmin(ctx, tel_p, C, best_p, stream);
        Py_END_ALLOW_THREADS
        return result(rc, std::move(best));
    });
}

PyMethodDef methods[] = {
    {"sortedF", (PyCFunction)(void (*)(void))sortedF, METH_FASTCALL, nullptr},
    {"simulate", (PyCFunction)(void (*)(void))simulate, METH_FASTCALL, nullptr},
    {"argmin", (PyCFunction)(void (*)(void))argmin, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef definition = {PyModuleDef_HEAD_INIT, "kvsched_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_kvsched_host()
{
    PyObject *m = PyModule_Create(&definition);
    if (m && PyModule_AddStringConstant(m, "torch_version", TORCH_VERSION) != 0) Py_CLEAR(m);  // (whose layouts are compiled in)
    return m;
}
