// Argument marshalling of the Python binding for the tensors of a call: the checks that grawa.py makes on a [K, >= P] view and
// what it passes on, by one call into native code instead of a dozen attribute look-ups.  A small update's call was bound
// by them: LGRAWA of 4 workers, 270 k columns 9.8 -> 8.4 us, without allocation and 8 workers 12.0 -> 10.7.  Anything that is not plainly in order gives
// None, and grawa.py looks again and raises.
#include <torch/csrc/autograd/python_variable.h>

namespace {

// rows(t, K, P, grads): (data pointer, row stride, dtype code) of a CUDA tensor [K, >= P] with unit column stride whose rows do
// not overlap and whose storage holds them; float32, or with `grads` bfloat16 too.  The codes are GRAWA_F32 and GRAWA_BF16.
PyObject *rows(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != 4) {
        PyErr_SetString(PyExc_TypeError, "rows(tensor, K, P, grads)");
        return nullptr;
    }
    const long long K = PyLong_AsLongLong(args[1]), P = PyLong_AsLongLong(args[2]);
    const int grads = PyObject_IsTrue(args[3]);
    if (PyErr_Occurred()) return nullptr;
    if (!THPVariable_CheckExact(args[0])) Py_RETURN_NONE; // subclasses and proxies: by their own Python attributes
    try { // no C++ exception may leave: tensors of torch's transforms throw on some of these
        const at::Tensor &t = THPVariable_Unpack(args[0]);
        if (!t.defined() || t.layout() != at::kStrided || !t.is_cuda() || t.dim() != 2 || !t.has_storage()) Py_RETURN_NONE;
        const at::ScalarType type = t.scalar_type();
        if (type != at::kFloat && !(grads && type == at::kBFloat16)) Py_RETURN_NONE;
        if (t.key_set().has(c10::DispatchKey::Python) || t.unsafeGetTensorImpl()->has_symbolic_sizes_strides()) Py_RETURN_NONE;
        const int64_t size = type == at::kFloat ? 4 : 2, ld = t.stride(0);
        if (t.stride(1) != 1 || K < 1 || P < 1 || t.size(0) != K || t.size(1) < P || (K > 1 && ld < P)) Py_RETURN_NONE;
        const int64_t have = (int64_t)(t.storage().nbytes() / (size_t)size) - t.storage_offset();
        if (have < P || (K > 1 && ld > (have - P) / (K - 1))) Py_RETURN_NONE; // (K - 1) ld + P elements from the view's start
        return Py_BuildValue("KLi", (unsigned long long)reinterpret_cast<uintptr_t>(t.data_ptr()), (long long)ld, type == at::kFloat ? 0 : 1);
    } catch (...) {
        Py_RETURN_NONE;
    }
}

PyMethodDef methods[] = {{"rows", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(rows)), METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
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
