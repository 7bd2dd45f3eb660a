// CPython extension module `_native_call`: the marshalling of a GEMM call from tensors to the C ABI.
//
// A single-row product takes about 5 us on the GPU and 2.9 us of library and launch on the host; checking and unpacking
// six tensors in Python and the foreign-function call took another 2.9 us, so that a stream of small calls was bound by
// Python.  Here the same takes 0.4 us.  Calls that are not plain - another tensor type, a wrong dtype, device, shape or
// stride, a transform's wrapper - are left to the Python code, which states what is wrong: every function returns None
// for them and has done nothing.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <limits.h>

#include <ATen/core/Tensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

namespace {

// gptq_w4a16_gemm, gptq_w4a16_gemm_static and gptq_w4a16_gemm_prepared have one signature
using gemm_fn = int (*)(const void *, const void *, const void *, const void *, const void *, void *, int, int, int, int,
                        void *);

// A contiguous tensor on the GPU of exactly torch.Tensor's type (or a Parameter), or null.
const at::Tensor *plain(PyObject *obj, at::ScalarType type, int64_t dim)
{
    if (!THPVariable_CheckExact(obj))
        return nullptr;
    const at::Tensor &t = THPVariable_Unpack(obj);
    if (!t.defined() || !t.is_cuda() || t.scalar_type() != type || t.dim() != dim || !t.is_contiguous())
        return nullptr;
    return &t;
}

// (function address, x, qweight, qzeros, scales, index or None, out, group_size) -> status code, or None
PyObject *gemm(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != 8 || !PyLong_CheckExact(args[0]) || !PyLong_CheckExact(args[7]))
        Py_RETURN_NONE;
    const gemm_fn fn = reinterpret_cast<gemm_fn>(PyLong_AsVoidPtr(args[0]));
    const long group = PyLong_AsLong(args[7]);
    if (PyErr_Occurred()) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    int rc;
    try {
        const at::Tensor *x = plain(args[1], at::kHalf, 2), *qweight = plain(args[2], at::kInt, 2);
        const at::Tensor *qzeros = plain(args[3], at::kInt, 2), *scales = plain(args[4], at::kHalf, 2);
        const bool indexed = args[5] != Py_None;
        const at::Tensor *index = indexed ? plain(args[5], at::kInt, 1) : nullptr;
        const at::Tensor *out = plain(args[6], at::kHalf, 2);
        if (!fn || !x || !qweight || !qzeros || !scales || !out || (indexed && !index))
            Py_RETURN_NONE;
        const int64_t M = x->size(0), K = qweight->size(0) * 8, N = qweight->size(1);
        if (group <= 0 || group > INT_MAX || M > INT_MAX || K > INT_MAX || N > INT_MAX || K % group != 0 || N % 8 != 0 ||
            x->size(1) != K || qzeros->size(0) != K / group || qzeros->size(1) != N / 8 || scales->size(0) != K / group ||
            scales->size(1) != N || (indexed && index->size(0) != K) || out->size(0) != M || out->size(1) != N)
            Py_RETURN_NONE;
        const void *px = x->data_ptr(), *pw = qweight->data_ptr(), *pz = qzeros->data_ptr(), *ps = scales->data_ptr();
        const void *pi = indexed ? index->data_ptr() : nullptr;
        void *po = out->data_ptr();
        void *const stream = c10::hip::getCurrentHIPStream().stream();
        Py_BEGIN_ALLOW_THREADS
        rc = fn(px, pw, pz, ps, pi, po, (int)M, (int)K, (int)N, (int)group, stream);
        Py_END_ALLOW_THREADS
    } catch (...) {
        Py_RETURN_NONE;  // (a wrapper without storage, for one: Python meets the same and says so)
    }
    return PyLong_FromLong(rc);
}

PyMethodDef methods[] = {
    {"gemm", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(gemm)), METH_FASTCALL,
     "gemm(address, x, qweight, qzeros, scales, index, out, group_size) -> status code, or None for a call that is not plain"},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native_call(void)
{
    return PyModule_Create(&module);
}
