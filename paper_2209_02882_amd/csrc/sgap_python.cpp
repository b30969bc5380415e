// The way from a Python call to the C ABI, in native code: reads the tensors' device pointers, checks what binding.py
// checks and calls the library on torch's current stream.  A call of a small matrix is over on the GPU in about 4 us;
// reading five tensors, the stream and fifteen ctypes arguments in Python took 8 us of host time per call, which is
// what such calls were bound by (1,024 rows of 10 entries, N = 32: 9.6 us a call, 4 us of it kernel).
//
// Every function returns the library's status, or -1 if an argument is not what the quick way takes (no tensor, not on
// the GPU, another type or length): nothing has been done then, and binding.py's own checks say what is wrong.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/sgap.h"

namespace {

constexpr int kNotTaken = -1;

struct Call {
    PyObject* const* arg;
    bool ok = true;

    int64_t number(int n)
    {
        PyObject* o = arg[n];
        if (!PyLong_CheckExact(o)) return ok = false, 0;
        int overflow = 0;
        const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
        if (overflow) ok = false;
        return v;
    }
    // a C int: what does not fit is not taken (ctypes would cut it off: left to the slow way)
    int small(int n)
    {
        const int64_t v = number(n);
        if (v != (int)v) ok = false;
        return (int)v;
    }
    const at::Tensor* tensor(int n)
    {
        if (!ok || !THPVariable_Check(arg[n])) return ok = false, nullptr;
        return &THPVariable_Unpack(arg[n]);
    }
    // device pointer of a contiguous tensor of `count` elements (null for an empty one)
    void* data(int n, at::ScalarType type, int64_t count)
    {
        const at::Tensor* t = tensor(n);
        if (!t) return nullptr;
        if (!t->is_cuda() || t->scalar_type() != type || t->numel() != count || !t->is_contiguous()) {
            ok = false;
            return nullptr;
        }
        return count ? t->data_ptr() : nullptr;
    }
    int32_t* ints(int n, int64_t count) { return static_cast<int32_t*>(data(n, at::kInt, count)); }
    float* floats(int n, int64_t count) { return static_cast<float*>(data(n, at::kFloat, count)); }
    int64_t length(int n)
    {
        const at::Tensor* t = tensor(n);
        return t ? t->numel() : 0;
    }
    int64_t number_or(int n, int64_t otherwise) { return arg[n] == Py_None ? otherwise : number(n); }
    // a torch stream; None: torch's current stream on the current device
    void* stream(int n)
    {
        if (!ok) return nullptr;
        if (arg[n] == Py_None) return c10::hip::getCurrentHIPStream().stream();
        PyObject* handle = PyObject_GetAttrString(arg[n], "cuda_stream");
        void* s = handle && PyLong_Check(handle) ? PyLong_AsVoidPtr(handle) : nullptr;
        if (!handle || !PyLong_Check(handle) || PyErr_Occurred()) {
            PyErr_Clear();
            ok = false;
        }
        Py_XDECREF(handle);
        return s;
    }
    // None, or a CUDA uint8 tensor
    void* workspace(int n, int64_t* bytes)
    {
        *bytes = 0;
        if (arg[n] == Py_None) return nullptr;
        const at::Tensor* t = tensor(n);
        if (!t) return nullptr;
        if (!t->is_cuda() || t->scalar_type() != at::kByte) {
            ok = false;
            return nullptr;
        }
        *bytes = t->numel();
        return *bytes ? t->data_ptr() : nullptr;
    }
};

struct Matrix {
    int64_t M, K, N, nnz;
    const int32_t *rowptr, *colidx;
    const float *vals, *B;
    float* C;
    // arguments 0 .. 7: M, K, N, rowptr, colidx, vals, B, C
    explicit Matrix(Call& c)
    {
        M = c.number(0); K = c.number(1); N = c.number(2);
        if (!c.ok || M < 0 || K < 0 || N < 0 || M > INT32_MAX || K > INT32_MAX || N > INT32_MAX) {
            c.ok = false;
            return;
        }
        nnz = c.length(4);
        rowptr = c.ints(3, M + 1);
        colidx = c.ints(4, nnz);
        vals = c.floats(5, nnz);
        B = c.floats(6, K * N);
        C = c.floats(7, M * N);
    }
};

PyObject* status(int st) { return PyLong_FromLong(st); }

// the library call itself, without the interpreter's lock: a launch may wait for room in the queue
template <typename F>
PyObject* enqueue(F&& f)
{
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = f();
    Py_END_ALLOW_THREADS
    return status(st);
}

// M, K, N, rowptr, colidx, vals, B, C, group_size, strategy, schedule, nnz_hint, stream; sgap_ttm_csf has the same
// arguments with fibers for rows, and forwards to the same code in the library
PyObject* spmm_csr_ex(PyObject*, PyObject* const* arg, Py_ssize_t n)
{
    Call c{arg};
    if (n != 13) return status(kNotTaken);
    const Matrix m(c);
    const int group = c.small(8), strategy = c.small(9), schedule = c.small(10);
    const int64_t hint = c.number_or(11, m.nnz);
    void* stream = c.stream(12);
    if (!c.ok) return status(kNotTaken);
    return enqueue([&] {
        return sgap_spmm_csr_ex(m.M, m.K, m.N, m.rowptr, m.colidx, m.vals, m.B, m.C, group, strategy, schedule, hint,
                                   stream);
    });
}

// M, K, N, rowptr, colidx, vals, B, C, config, nnz_hint, workspace, stream
PyObject* spmm_csr_cfg(PyObject*, PyObject* const* arg, Py_ssize_t n)
{
    Call c{arg};
    if (n != 12) return status(kNotTaken);
    const Matrix m(c);
    const int64_t hint = c.number_or(9, m.nnz);
    int64_t bytes = 0;
    void* ws = c.workspace(10, &bytes);
    void* stream = c.stream(11);
    if (!c.ok) return status(kNotTaken);
    Py_buffer config;  // a ctypes structure lends its memory
    if (PyObject_GetBuffer(arg[8], &config, PyBUF_SIMPLE) != 0) {
        PyErr_Clear();
        return status(kNotTaken);
    }
    PyObject* st = config.len != (Py_ssize_t)sizeof(sgap_config) ? status(kNotTaken) : enqueue([&] {
        return sgap_spmm_csr_cfg(m.M, m.K, m.N, m.rowptr, m.colidx, m.vals, m.B, m.C,
                                 static_cast<const sgap_config*>(config.buf), hint, ws, bytes, stream);
    });
    PyBuffer_Release(&config);
    return st;
}

struct Sampled {
    int64_t M, K, J, nnz;
    const int32_t *rowptr, *colidx;
    const float *vals, *X1, *X2T;
    float* out;
    // arguments 0 .. 8: M, K, J, rowptr, colidx, vals, X1, X2T, out_vals
    explicit Sampled(Call& c)
    {
        M = c.number(0); K = c.number(1); J = c.number(2);
        if (!c.ok || M < 0 || K < 0 || J < 0 || M > INT32_MAX || K > INT32_MAX || J > INT32_MAX) {
            c.ok = false;
            return;
        }
        nnz = c.length(4);
        rowptr = c.ints(3, M + 1);
        colidx = c.ints(4, nnz);
        vals = c.floats(5, nnz);
        X1 = c.floats(6, M * J);
        X2T = c.floats(7, K * J);
        out = c.floats(8, nnz);
    }
};

// M, K, J, rowptr, colidx, vals, X1, X2T, out_vals, group_size, strategy, nnz_hint, stream
PyObject* sddmm_csr(PyObject*, PyObject* const* arg, Py_ssize_t n)
{
    Call c{arg};
    if (n != 13) return status(kNotTaken);
    const Sampled s(c);
    const int group = c.small(9), strategy = c.small(10);
    const int64_t hint = c.number_or(11, s.nnz);
    void* stream = c.stream(12);
    if (!c.ok) return status(kNotTaken);
    return enqueue([&] {
        return sgap_sddmm_csr(s.M, s.K, s.J, s.rowptr, s.colidx, s.vals, s.X1, s.X2T, s.out, group, strategy, hint,
                                 stream);
    });
}

// ..., group_size, strategy, nnz_hint, long_row_min, window_kb, max_long_rows, workspace, stream
PyObject* sddmm_csr_windows(PyObject*, PyObject* const* arg, Py_ssize_t n)
{
    Call c{arg};
    if (n != 17) return status(kNotTaken);
    const Sampled s(c);
    const int group = c.small(9), strategy = c.small(10);
    const int64_t hint = c.number_or(11, s.nnz);
    const int long_row_min = c.small(12), window_kb = c.small(13), max_long_rows = c.small(14);
    int64_t bytes = 0;
    void* ws = c.workspace(15, &bytes);
    void* stream = c.stream(16);
    if (!c.ok) return status(kNotTaken);
    return enqueue([&] {
        return sgap_sddmm_csr_windows(s.M, s.K, s.J, s.rowptr, s.colidx, s.vals, s.X1, s.X2T, s.out, group, strategy,
                                         hint, long_row_min, window_kb, max_long_rows, ws, bytes, stream);
    });
}

// I, K, L, J, fptr, fidx, eptr, eidx, vals, X1, X2, Y, group_size, strategy, schedule, nnz_hint, stream
PyObject* mttkrp_csf_ex(PyObject*, PyObject* const* arg, Py_ssize_t n)
{
    Call c{arg};
    if (n != 17) return status(kNotTaken);
    const int64_t I = c.number(0), K = c.number(1), L = c.number(2), J = c.number(3);
    if (!c.ok || I < 0 || K < 0 || L < 0 || J < 0 || I > INT32_MAX || K > INT32_MAX || L > INT32_MAX || J > INT32_MAX)
        return status(kNotTaken);
    const int64_t fibers = c.length(5), nnz = c.length(8);
    const int32_t *fptr = c.ints(4, I + 1), *fidx = c.ints(5, fibers), *eptr = c.ints(6, fibers + 1), *eidx = c.ints(7, nnz);
    const float *vals = c.floats(8, nnz), *X1 = c.floats(9, K * J), *X2 = c.floats(10, L * J);
    float* Y = c.floats(11, I * J);
    const int group = c.small(12), strategy = c.small(13), schedule = c.small(14);
    const int64_t hint = c.number_or(15, nnz);
    void* stream = c.stream(16);
    if (!c.ok) return status(kNotTaken);
    return enqueue([&] {
        return sgap_mttkrp_csf_ex(I, K, L, J, fptr, fidx, eptr, eidx, vals, X1, X2, Y, group, strategy, schedule, hint,
                                     stream);
    });
}

PyMethodDef kMethods[] = {
    {"spmm_csr_ex", (PyCFunction)(void (*)())spmm_csr_ex, METH_FASTCALL, nullptr},
    {"spmm_csr_cfg", (PyCFunction)(void (*)())spmm_csr_cfg, METH_FASTCALL, nullptr},
    {"sddmm_csr", (PyCFunction)(void (*)())sddmm_csr, METH_FASTCALL, nullptr},
    {"sddmm_csr_windows", (PyCFunction)(void (*)())sddmm_csr_windows, METH_FASTCALL, nullptr},
    {"mttkrp_csf_ex", (PyCFunction)(void (*)())mttkrp_csf_ex, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&kModule); }
