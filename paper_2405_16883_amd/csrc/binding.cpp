// Python entry points of the execution calls: tensors and sizes in, one call of the C ABI, its status out.
//
// Argument marshalling only.  The calls are short (a kernel launch takes 2 to 3 us of host time), so reading seven tensors'
// pointers, types and strides through Python costs more than the call itself: 9.3 us per planned SpMM of a small graph
// through ctypes.  binding.py keeps the signatures, the error type and everything that is not on the hot path.
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>
#include <exception>

#include "scorch_spmm.h"

namespace {

// Arguments of one call; `ok` turns false, with the Python error set, at the first one that does not fit.
struct Args {
    PyObject *const *v;
    bool ok = true;

    int32_t i32(int i) {
        if (!ok) return 0;
        const long long x = PyLong_AsLongLong(v[i]);
        if (x == -1 && PyErr_Occurred()) ok = false;
        return (int32_t)x;
    }

    // Device pointer of a tensor; nullptr for None and for a tensor without elements.
    void *ptr(int i, at::ScalarType type, const char *name) {
        if (!ok || v[i] == Py_None) return nullptr;
        if (!THPVariable_Check(v[i])) {
            PyErr_Format(PyExc_TypeError, "%s must be a tensor", name);
            ok = false;
            return nullptr;
        }
        const at::Tensor &t = THPVariable_Unpack(v[i]);
        if (!t.is_cuda()) {
            PyErr_Format(PyExc_ValueError, "%s must live on the GPU", name);
            ok = false;
        } else if (t.scalar_type() != type) {
            PyObject *got = PyObject_GetAttrString(v[i], "dtype");
            if (got) PyErr_Format(PyExc_ValueError, "%s must be %s, got %S", name, type == at::kInt ? "torch.int32" : "torch.float32", got);
            Py_XDECREF(got);
            ok = false;
        }
        return ok && t.numel() > 0 ? t.data_ptr() : nullptr;
    }
    int32_t *ints(int i, const char *name) { return static_cast<int32_t *>(ptr(i, at::kInt, name)); }
    float *floats(int i, const char *name) { return static_cast<float *>(ptr(i, at::kFloat, name)); }

    // Row stride of a matrix whose rows are contiguous.
    int32_t ld(int i, const char *name) {
        if (!ok) return 0;
        if (!THPVariable_Check(v[i])) {
            PyErr_Format(PyExc_TypeError, "%s must be a tensor", name);
            ok = false;
            return 0;
        }
        const at::Tensor &t = THPVariable_Unpack(v[i]);
        if (t.dim() != 2 || (t.numel() > 0 && t.stride(1) != 1)) {
            PyErr_Format(PyExc_ValueError, "%s must be 2-D with unit column stride", name);
            ok = false;
            return 0;
        }
        return (int32_t)(t.size(0) > 1 ? t.stride(0) : std::max(t.stride(0), t.size(1)));
    }

    // stream: None for the current stream of the current device
    void *stream(int i) {
        if (!ok) return nullptr;
        if (v[i] == Py_None) return c10::hip::getCurrentHIPStream().stream();
        PyObject *h = PyObject_GetAttrString(v[i], "cuda_stream");
        void *s = h ? PyLong_AsVoidPtr(h) : nullptr;
        Py_XDECREF(h);
        if (PyErr_Occurred()) ok = false;
        return s;
    }
};

bool count_is(Py_ssize_t nargs, Py_ssize_t want) {
    if (nargs != want) PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, nargs);
    return nargs == want;
}

template <typename F> PyObject *status_of(const Args &a, F call) {
    if (!a.ok) return nullptr;
    scorch_status_t st;
    Py_BEGIN_ALLOW_THREADS
    st = call();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
}

// (m, k, n, rowptr, colidx, vals, B, C, stream)
template <scorch_status_t (*CALL)(int32_t, int32_t, int32_t, const int32_t *, const int32_t *, const float *, const float *,
                                  int32_t, float *, int32_t, void *)>
PyObject *spmm(PyObject *, PyObject *const *v, Py_ssize_t nargs) {
    if (!count_is(nargs, 9)) return nullptr;
    Args a{v};
    const int32_t m = a.i32(0), k = a.i32(1), n = a.i32(2);
    const int32_t *rp = a.ints(3, "rowptr"), *ci = a.ints(4, "colidx");
    const float *x = a.floats(5, "vals"), *B = a.floats(6, "B");
    const int32_t ldb = a.ld(6, "B");
    float *C = a.floats(7, "C");
    const int32_t ldc = a.ld(7, "C");
    void *s = a.stream(8);
    return status_of(a, [&] { return CALL(m, k, n, rp, ci, x, B, ldb, C, ldc, s); });
}

const scorch_spmm_plan_t *plan_of(Args &a, int i) {
    if (!a.ok) return nullptr;
    void *p = PyLong_AsVoidPtr(a.v[i]);
    if (PyErr_Occurred()) a.ok = false;
    return static_cast<const scorch_spmm_plan_t *>(p);
}

// (plan handle, rowptr, colidx, vals, B, C, stream)
PyObject *spmm_planned(PyObject *, PyObject *const *v, Py_ssize_t nargs) {
    if (!count_is(nargs, 7)) return nullptr;
    Args a{v};
    const scorch_spmm_plan_t *plan = plan_of(a, 0);
    const int32_t *rp = a.ints(1, "rowptr"), *ci = a.ints(2, "colidx");
    const float *x = a.floats(3, "vals"), *B = a.floats(4, "B");
    const int32_t ldb = a.ld(4, "B");
    float *C = a.floats(5, "C");
    const int32_t ldc = a.ld(5, "C");
    void *s = a.stream(6);
    return status_of(a, [&] { return scorch_spmm_csr_planned(plan, rp, ci, x, B, ldb, C, ldc, s); });
}

// (plan handle, rowptr, colidx, vals, B, bias, activation, C, stream)
PyObject *spmm_planned_epilogue(PyObject *, PyObject *const *v, Py_ssize_t nargs) {
    if (!count_is(nargs, 9)) return nullptr;
    Args a{v};
    const scorch_spmm_plan_t *plan = plan_of(a, 0);
    const int32_t *rp = a.ints(1, "rowptr"), *ci = a.ints(2, "colidx");
    const float *x = a.floats(3, "vals"), *B = a.floats(4, "B");
    const int32_t ldb = a.ld(4, "B");
    const float *bias = a.floats(5, "bias");
    const int32_t act = a.i32(6);
    float *C = a.floats(7, "C");
    const int32_t ldc = a.ld(7, "C");
    void *s = a.stream(8);
    return status_of(a, [&] { return scorch_spmm_csr_planned_epilogue(plan, rp, ci, x, B, ldb, bias, act, C, ldc, s); });
}

// (m, k, d, rowptr, colidx, vals, B, Ct, out_vals, stream)
PyObject *sddmm(PyObject *, PyObject *const *v, Py_ssize_t nargs) {
    if (!count_is(nargs, 10)) return nullptr;
    Args a{v};
    const int32_t m = a.i32(0), k = a.i32(1), d = a.i32(2);
    const int32_t *rp = a.ints(3, "rowptr"), *ci = a.ints(4, "colidx");
    const float *x = a.floats(5, "vals"), *B = a.floats(6, "B");
    const int32_t ldb = a.ld(6, "B");
    const float *Ct = a.floats(7, "Ct");
    const int32_t ldct = a.ld(7, "Ct");
    float *out = a.floats(8, "out_vals");
    void *s = a.stream(9);
    return status_of(a, [&] { return scorch_sddmm_csr(m, k, d, rp, ci, x, B, ldb, Ct, ldct, out, s); });
}

// (plan handle, d, rowptr, colidx, vals, B, Ct, out_vals, stream)
PyObject *sddmm_planned(PyObject *, PyObject *const *v, Py_ssize_t nargs) {
    if (!count_is(nargs, 9)) return nullptr;
    Args a{v};
    const scorch_spmm_plan_t *plan = plan_of(a, 0);
    const int32_t d = a.i32(1);
    const int32_t *rp = a.ints(2, "rowptr"), *ci = a.ints(3, "colidx");
    const float *x = a.floats(4, "vals"), *B = a.floats(5, "B");
    const int32_t ldb = a.ld(5, "B");
    const float *Ct = a.floats(6, "Ct");
    const int32_t ldct = a.ld(6, "Ct");
    float *out = a.floats(7, "out_vals");
    void *s = a.stream(8);
    return status_of(a, [&] { return scorch_sddmm_csr_planned(plan, d, rp, ci, x, B, ldb, Ct, ldct, out, s); });
}

// (X, W, bias, activation, Y, stream)
PyObject *dense_layer(PyObject *, PyObject *const *v, Py_ssize_t nargs) {
    if (!count_is(nargs, 6)) return nullptr;
    Args a{v};
    const float *X = a.floats(0, "X"), *W = a.floats(1, "W");
    const int32_t ldx = a.ld(0, "X"), ldw = a.ld(1, "W");
    const float *bias = a.floats(2, "bias");
    const int32_t act = a.i32(3);
    float *Y = a.floats(4, "Y");
    const int32_t ldy = a.ld(4, "Y");
    void *s = a.stream(5);
    if (!a.ok) return nullptr;
    const at::Tensor &x = THPVariable_Unpack(v[0]), &w = THPVariable_Unpack(v[1]), &y = THPVariable_Unpack(v[4]);
    if (x.size(1) != w.size(0) || y.size(0) != x.size(0) || y.size(1) != w.size(1) ||
        (v[2] != Py_None && THPVariable_Unpack(v[2]).numel() != w.size(1))) {
        PyErr_SetString(PyExc_ValueError, "X, W, bias and Y do not fit together");
        return nullptr;
    }
    const int32_t m = (int32_t)x.size(0), k = (int32_t)x.size(1), n = (int32_t)w.size(1);
    return status_of(a, [&] { return scorch_dense_layer(m, k, n, X, ldx, W, ldw, bias, act, Y, ldy, s); });
}

// (m, row_idx, rowptr_out, bad_flag, stream)
PyObject *coo_to_csr_rowptr(PyObject *, PyObject *const *v, Py_ssize_t nargs) {
    if (!count_is(nargs, 5)) return nullptr;
    Args a{v};
    const int32_t m = a.i32(0);
    const int32_t *rows = a.ints(1, "row_idx");
    int32_t *out = a.ints(2, "rowptr_out"), *bad = a.ints(3, "bad_flag");
    void *s = a.stream(4);
    if (a.ok && (v[1] == Py_None || v[2] == Py_None)) {
        PyErr_SetString(PyExc_TypeError, "row_idx and rowptr_out must be tensors");
        return nullptr;
    }
    if (a.ok && THPVariable_Unpack(v[2]).numel() != (int64_t)m + 1) {
        PyErr_SetString(PyExc_ValueError, "rowptr_out must have m + 1 entries");
        return nullptr;
    }
    const int64_t nnz = a.ok ? THPVariable_Unpack(v[1]).numel() : 0;
    return status_of(a, [&] { return scorch_coo_to_csr_rowptr(m, nnz, rows, out, bad, s); });
}

// What the interpreter calls.  A tensor without plain memory (sparse, fake, wrapped by a transform) and a missing GPU make torch
// throw; the exception becomes a Python error here, it must not reach the interpreter's C frames.
typedef PyObject *(*method)(PyObject *, PyObject *const *, Py_ssize_t);
template <method F> PyObject *guarded(PyObject *self, PyObject *const *v, Py_ssize_t nargs) {
    try {
        return F(self, v, nargs);
    } catch (...) {
        torch::translate_exception_to_python(std::current_exception());
        return nullptr;
    }
}
template <method F> PyMethodDef entry(const char *name) {
    return {name, (PyCFunction)(void (*)(void))guarded<F>, METH_FASTCALL, nullptr};
}

PyMethodDef kMethods[] = {
    entry<spmm<scorch_spmm_csr>>("spmm_csr"),
    entry<spmm<scorch_spmm_csr_static>>("spmm_csr_static"),
    entry<spmm_planned>("spmm_csr_planned"),
    entry<spmm_planned_epilogue>("spmm_csr_planned_epilogue"),
    entry<sddmm>("sddmm_csr"),
    entry<sddmm_planned>("sddmm_csr_planned"),
    entry<dense_layer>("dense_layer"),
    entry<coo_to_csr_rowptr>("coo_to_csr_rowptr"),
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_scorch_binding", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__scorch_binding(void) { return PyModule_Create(&kModule); }
