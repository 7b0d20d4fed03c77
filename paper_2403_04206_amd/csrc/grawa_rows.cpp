// Argument marshalling of the Python binding in native code: the checks that grawa.py makes on the tensors of a call and what it
// passes on, instead of a dozen attribute look-ups a tensor; and whole calls of those that small models make one after the other.
// Such calls were bound by them: LGRAWA of 4 workers, 270 k columns 9.8 -> 8.4 us, without allocation and 8 workers 12.0 -> 10.7; a round of
// four scored steps and the communication, 4 workers, 9 k columns, takes the host 32.4 us with the checks alone and 24.7 with the calls.  Anything that is not
// plainly in order gives None, and grawa.py looks again and raises.
#include <torch/csrc/autograd/python_variable.h>

namespace {

struct Rows {
    void *p;
    int64_t ld;
    int dt; // GRAWA_F32 or GRAWA_BF16
};

// A plain CUDA tensor: subclasses and proxies go by their own Python attributes.  May throw (tensors of torch's transforms do).
const at::Tensor *plain_tensor(PyObject *o)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || t.layout() != at::kStrided || !t.is_cuda() || !t.has_storage()) return nullptr;
    if (t.key_set().has(c10::DispatchKey::Python) || t.unsafeGetTensorImpl()->has_symbolic_sizes_strides()) return nullptr;
    return &t;
}

// [K, >= P] with unit column stride whose rows do not overlap and whose storage holds them; float32, or with `grads` bfloat16 too.
bool rows_of(PyObject *o, int64_t K, int64_t P, bool grads, Rows &r)
{
    const at::Tensor *t = plain_tensor(o);
    if (!t || t->dim() != 2) return false;
    const at::ScalarType type = t->scalar_type();
    if (type != at::kFloat && !(grads && type == at::kBFloat16)) return false;
    const int64_t size = type == at::kFloat ? 4 : 2, ld = t->stride(0);
    if (t->stride(1) != 1 || K < 1 || P < 1 || t->size(0) != K || t->size(1) < P || (K > 1 && ld < P)) return false;
    const int64_t have = (int64_t)(t->storage().nbytes() / (size_t)size) - t->storage_offset();
    if (have < P || (K > 1 && ld > (have - P) / (K - 1))) return false; // (K - 1) ld + P elements from the view's start
    r = Rows{t->data_ptr(), ld, type == at::kFloat ? 0 : 1};
    return true;
}

// None, or a float32 vector of at least n elements with unit stride.
bool vector_of(PyObject *o, int64_t n, float *&p)
{
    p = nullptr;
    if (o == Py_None) return true;
    const at::Tensor *t = plain_tensor(o);
    if (!t || t->scalar_type() != at::kFloat || t->dim() != 1 || t->stride(0) != 1 || n < 1 || t->size(0) < n) return false;
    if ((int64_t)(t->storage().nbytes() / 4) - t->storage_offset() < n) return false;
    p = static_cast<float *>(t->data_ptr());
    return true;
}

// None, or a contiguous float32 tensor [K, L], with L = 0 [K].
bool table_of(PyObject *o, int64_t K, int64_t L, float *&p)
{
    p = nullptr;
    if (o == Py_None) return true;
    const at::Tensor *t = plain_tensor(o);
    if (!t || t->scalar_type() != at::kFloat || !t->is_contiguous() || t->dim() != (L ? 2 : 1) || t->size(0) != K || (L && t->size(1) != L))
        return false;
    p = static_cast<float *>(t->data_ptr());
    return true;
}

bool number_of(PyObject *o, float &f) // as ctypes makes a C float of float(o)
{
    if (!PyFloat_CheckExact(o)) return false;
    f = (float)PyFloat_AS_DOUBLE(o);
    return true;
}

bool integer_of(PyObject *o, long long &v)
{
    if (!PyLong_CheckExact(o)) return false;
    v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    return true;
}

bool pointer_of(PyObject *o, void *&p)
{
    p = nullptr;
    if (!PyLong_CheckExact(o)) return false;
    p = PyLong_AsVoidPtr(o);
    if (!p && PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    return true;
}

// The handle that `current`, a Python function, gives: asked for last, since it sets torch's CUDA state up.
template <typename Call> PyObject *status_of(PyObject *current, const Call &call)
{
    PyObject *handle = PyObject_CallNoArgs(current);
    if (!handle) return nullptr;
    void *stream;
    const bool ok = pointer_of(handle, stream);
    Py_DECREF(handle);
    if (!ok) Py_RETURN_NONE;
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = call(stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

// rows(t, K, P, grads): (data pointer, row stride, dtype code).
PyObject *rows(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != 4) {
        PyErr_SetString(PyExc_TypeError, "rows(tensor, K, P, grads)");
        return nullptr;
    }
    const long long K = PyLong_AsLongLong(args[1]), P = PyLong_AsLongLong(args[2]);
    const int grads = PyObject_IsTrue(args[3]);
    if (PyErr_Occurred()) return nullptr;
    try { // no C++ exception may leave
        Rows r;
        if (!rows_of(args[0], K, P, grads, r)) Py_RETURN_NONE;
        return Py_BuildValue("KLi", (unsigned long long)reinterpret_cast<uintptr_t>(r.p), (long long)r.ld, r.dt);
    } catch (...) {
        Py_RETURN_NONE;
    }
}

// Whole calls: the status, or None where an argument is not plainly in order.  `function` is the address of the library's function of
// that name, `current` a function that gives the stream's handle; the GIL is released as ctypes does.

// scored(function, plan, x, g, K, P, lr, gamma, center, mu, tau, current): grawa_local_step_scored
PyObject *scored(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    typedef int (*Function)(void *, float *, int64_t, const void *, int64_t, int, float, const float *, float, float, float, void *);
    void *function, *plan;
    long long K, P;
    float lr, gamma, mu, tau, *center;
    Rows x, g;
    try {
        if (n != 12 || !pointer_of(args[0], function) || !pointer_of(args[1], plan) || !integer_of(args[4], K) || !integer_of(args[5], P) ||
            !rows_of(args[2], K, P, false, x) || !rows_of(args[3], K, P, true, g) || !number_of(args[6], lr) || !number_of(args[7], gamma) ||
            !vector_of(args[8], P, center) || !number_of(args[9], mu) || !number_of(args[10], tau))
            Py_RETURN_NONE;
    } catch (...) {
        Py_RETURN_NONE;
    }
    return status_of(args[11], [&](void *stream) {
        return reinterpret_cast<Function>(function)(plan, static_cast<float *>(x.p), x.ld, g.p, g.ld, g.dt, lr, center, mu, tau, gamma, stream);
    });
}

// local(function, plan, x, K, P, L, per_layer, lam, center_out, weights_out, est_out, current): grawa_local_lgrawa_update, grawa_local_mgrawa_update
PyObject *local(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    typedef int (*Function)(void *, float *, int64_t, float, float *, float *, float *, void *);
    void *function, *plan;
    long long K, P, L, per_layer;
    float lam, *center, *weights, *est;
    Rows x;
    try {
        if (n != 12 || !pointer_of(args[0], function) || !pointer_of(args[1], plan) || !integer_of(args[3], K) || !integer_of(args[4], P) ||
            !integer_of(args[5], L) || !integer_of(args[6], per_layer) || L < 1 || !rows_of(args[2], K, P, false, x) || !number_of(args[7], lam) ||
            !vector_of(args[8], P, center) || !table_of(args[9], K, per_layer ? L : 0, weights) || !table_of(args[10], K, L, est))
            Py_RETURN_NONE;
    } catch (...) {
        Py_RETURN_NONE;
    }
    return status_of(args[11], [&](void *stream) {
        return reinterpret_cast<Function>(function)(plan, static_cast<float *>(x.p), x.ld, lam, center, weights, est, stream);
    });
}

// lgrawa(function, plan, x, g, K, P, L, lam, center_out, weights_out, current): grawa_lgrawa_update
PyObject *lgrawa(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    typedef int (*Function)(void *, float *, int64_t, const void *, int64_t, int, float, float *, float *, void *);
    void *function, *plan;
    long long K, P, L;
    float lam, *center, *weights;
    Rows x, g;
    try {
        if (n != 11 || !pointer_of(args[0], function) || !pointer_of(args[1], plan) || !integer_of(args[4], K) || !integer_of(args[5], P) ||
            !integer_of(args[6], L) || L < 1 || !rows_of(args[2], K, P, false, x) || !rows_of(args[3], K, P, true, g) || !number_of(args[7], lam) ||
            !vector_of(args[8], P, center) || !table_of(args[9], K, L, weights))
            Py_RETURN_NONE;
    } catch (...) {
        Py_RETURN_NONE;
    }
    return status_of(args[10], [&](void *stream) {
        return reinterpret_cast<Function>(function)(plan, static_cast<float *>(x.p), x.ld, g.p, g.ld, g.dt, lam, center, weights, stream);
    });
}

#define GRAWA_METHOD(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(f)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {GRAWA_METHOD(rows), GRAWA_METHOD(scored), GRAWA_METHOD(local), GRAWA_METHOD(lgrawa), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_rows", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

} // namespace

// The functions above read torch's objects through the headers this file was compiled with, so the module names the torch
// and the Python that it is for, and grawa.py uses it with no other.
PyMODINIT_FUNC PyInit__rows()
{
    PyObject *m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "built_for", GRAWA_ROWS_BUILT_FOR) != 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
