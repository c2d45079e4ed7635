// hs_torch.cpp -- the ordinary call of each device entry point from Python, in
// native code: tensor checks, output and workspace allocation and the C ABI
// call.  A small product's kernels take less time than the interpreter needs to
// marshal the call (12 to 22 us of host time per call in Python against 4 to 7
// here), so that time is what such a call costs.
//
// Every function takes the arguments already resolved by binding.py and
// returns the result, the hs_status as an int where the library refused the
// call, or None where the arguments are not the ordinary ones (a tensor
// subclass, a lazy view, another dtype, shape, stride or device, an empty matrix);
// binding.py then takes its general path, which answers the call or raises the
// error that belongs to it.
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "hs.h"

namespace {

// the library's entry points, handed over by binding.py
decltype(&hs_workspace_size) f_workspace_size;
decltype(&hs_gemm) f_gemm;
decltype(&hs_gemm_tn) f_gemm_tn;
decltype(&hs_gemm_noalloc) f_gemm_noalloc;
decltype(&hs_gemv) f_gemv;
decltype(&hs_gemm_backward) f_backward;
decltype(&hs_nbody) f_nbody;

struct NoGil {
    PyThreadState *s = PyEval_SaveThread();
    ~NoGil() { PyEval_RestoreThread(s); }
};

PyObject *none() { Py_RETURN_NONE; }

bool known(int dt) { return dt >= HS_F64 && dt <= HS_C32_SPLIT2_F16; }
bool complex_form(int dt) { return dt == HS_C32 || dt == HS_C32_SPLIT3_BF16 || dt == HS_C32_SPLIT2_F16; }

at::ScalarType in_type(int dt) {
    if (complex_form(dt)) return at::kComplexFloat;
    return dt == HS_F64 ? at::kDouble : dt == HS_BF16 ? at::kBFloat16 : dt == HS_F16 ? at::kHalf : at::kFloat;
}
at::ScalarType out_type(int dt) {
    return complex_form(dt) ? at::kComplexFloat : dt == HS_F64 ? at::kDouble : at::kFloat;
}

// A plain GPU tensor of this dtype and dimension that stores its values (no lazy
// conjugate or negative view), or nullptr.
const at::Tensor *plain(PyObject *o, at::ScalarType st, int64_t dim) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || t.dim() != dim || t.scalar_type() != st ||
        t.is_conj() || t.is_neg() || !t.has_storage() || t.unsafeGetTensorImpl()->has_symbolic_sizes_strides())
        return nullptr;
    return &t;
}

// Leading dimension of a non-empty row-major matrix, or 0 if the C ABI
// cannot address it (row_layout in binding.py).
int64_t leading(const at::Tensor &t) {
    const int64_t rows = t.size(0), cols = t.size(1);
    if (rows == 0 || cols == 0) return 0;
    if (cols > 1 && t.stride(1) != 1) return 0;
    if (rows > 1 && t.stride(0) < cols) return 0;
    return rows > 1 ? t.stride(0) : cols;
}

at::Tensor empty(at::IntArrayRef size, at::ScalarType st, const at::Tensor &like) {
    return at::empty(size, at::TensorOptions().dtype(st).device(like.device()));
}

// The workspace of a call (undefined if none is needed or the arguments are
// invalid: the call itself then says so).
struct Workspace {
    at::Tensor t;
    size_t bytes = 0;
    Workspace(size_t n, const at::Tensor &like) {
        if (n == 0 || n == SIZE_MAX) return;
        t = empty({(int64_t)n}, at::kByte, like);
        bytes = n;
    }
    void *ptr() const { return bytes ? t.data_ptr() : nullptr; }
};

void *current_stream() { return (void *)c10::hip::getCurrentHIPStream().stream(); }

bool ints(PyObject *const *a, int n, long *v) {
    for (int i = 0; i < n; ++i) {
        v[i] = PyLong_AsLong(a[i]);
        if (v[i] == -1 && PyErr_Occurred()) {
            PyErr_Clear();
            return false;
        }
        if (v[i] != (int32_t)v[i]) return false;
    }
    return true;
}

PyObject *status_or(hs_status st, const at::Tensor &t) {
    return st == HS_OK ? THPVariable_Wrap(t) : PyLong_FromLong(st);
}

// product(kind, A, B, out, dt, p, K): kind 0 hs_gemm, 1 hs_gemm_tn, 2 hs_gemm_noalloc
PyObject *product(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    long v[3], kind;
    if (n != 7 || !ints(a, 1, &kind) || !ints(a + 4, 3, v)) return none();
    const int dt = (int)v[0];
    if (!known(dt)) return none();
    const hs_schedule s{(int32_t)v[1], (int32_t)v[2]};
    const at::Tensor *A = plain(a[1], in_type(dt), 2), *B = plain(a[2], in_type(dt), 2);
    if (!A || !B) return none();
    const int64_t lda = leading(*A), ldb = leading(*B);
    if (!lda || !ldb) return none();
    const bool tn = kind == 1;
    const int64_t m = A->size(tn ? 1 : 0), k = A->size(tn ? 0 : 1), nc = B->size(1);
    if (B->size(0) != k) return none();
    at::Tensor C;
    if (a[3] == Py_None) {
        if (kind == 2) return none();
        C = empty({m, nc}, out_type(dt), *A);
    } else {
        const at::Tensor *o = plain(a[3], out_type(dt), 2);
        if (!o || o->device() != A->device() || o->size(0) != m || o->size(1) != nc || !leading(*o)) return none();
        C = *o;
    }
    const int64_t ldc = leading(C);
    void *st = current_stream();
    if (kind == 2) {
        hs_status r;
        {
            NoGil g;
            r = f_gemm_noalloc(m, nc, k, dt, s, A->data_ptr(), lda, B->data_ptr(), ldb, C.data_ptr(), ldc, st);
        }
        return status_or(r, C);
    }
    const Workspace ws(f_workspace_size(tn ? HS_OP_GEMM_TN : HS_OP_GEMM, m, nc, k, dt, s), *A);
    hs_status r;
    {
        NoGil g;
        r = (tn ? f_gemm_tn : f_gemm)(m, nc, k, dt, s, A->data_ptr(), lda, B->data_ptr(), ldb, C.data_ptr(), ldc,
                                      ws.ptr(), ws.bytes, st);
    }
    return status_or(r, C);
    END_HANDLE_TH_ERRORS
}

// backward(A, B, G, dt, p, K, need_a, need_b)
PyObject *backward(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    long v[5];
    if (n != 8 || !ints(a + 3, 5, v)) return none();
    const int dt = (int)v[0];
    if (!known(dt)) return none();
    const hs_schedule s{(int32_t)v[1], (int32_t)v[2]};
    const at::ScalarType it = in_type(dt);
    const at::Tensor *A = plain(a[0], it, 2), *B = plain(a[1], it, 2), *G = plain(a[2], it, 2);
    if (!A || !B || !G) return none();
    const int64_t lda = leading(*A), ldb = leading(*B), ldg = leading(*G);
    const int64_t m = A->size(0), k = A->size(1), nc = B->size(1);
    if (!lda || !ldb || !ldg || B->size(0) != k || G->size(0) != m || G->size(1) != nc) return none();
    at::Tensor dA, dB;
    if (v[3]) dA = empty({m, k}, out_type(dt), *A);
    if (v[4]) dB = empty({k, nc}, out_type(dt), *A);
    const Workspace ws(f_workspace_size(HS_OP_BACKWARD, m, nc, k, dt, s), *A);
    void *st = current_stream();
    hs_status r;
    {
        NoGil g;
        r = f_backward(m, nc, k, dt, s, A->data_ptr(), lda, B->data_ptr(), ldb, G->data_ptr(), ldg,
                       v[3] ? dA.data_ptr() : nullptr, k, v[4] ? dB.data_ptr() : nullptr, nc, ws.ptr(), ws.bytes, st);
    }
    if (r != HS_OK) return PyLong_FromLong(r);
    PyObject *x = THPVariable_Wrap(dA), *y = THPVariable_Wrap(dB);   // undefined: None
    if (!x || !y) {
        Py_XDECREF(x);
        Py_XDECREF(y);
        return nullptr;
    }
    PyObject *t = PyTuple_Pack(2, x, y);
    Py_DECREF(x);
    Py_DECREF(y);
    return t;
    END_HANDLE_TH_ERRORS
}

// gemv(A, x, out, dt, p, K)
PyObject *gemv(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    long v[3];
    if (n != 6 || !ints(a + 3, 3, v)) return none();
    const int dt = (int)v[0];
    if (!known(dt)) return none();
    const hs_schedule s{(int32_t)v[1], (int32_t)v[2]};
    const at::Tensor *A = plain(a[0], in_type(dt), 2), *x = plain(a[1], in_type(dt), 1);
    if (!A || !x) return none();
    const int64_t lda = leading(*A), m = A->size(0), nc = A->size(1);
    if (!lda || x->size(0) != nc || x->device() != A->device() || !x->is_contiguous()) return none();
    at::Tensor y;
    if (a[2] == Py_None) {
        y = empty({m}, in_type(dt), *A);
    } else {
        const at::Tensor *o = plain(a[2], in_type(dt), 1);
        if (!o || o->device() != A->device() || o->size(0) != m || o->stride(0) != 1) return none();
        y = *o;
    }
    void *st = current_stream();
    hs_status r;
    {
        NoGil g;
        r = f_gemv(m, nc, dt, s, A->data_ptr(), lda, x->data_ptr(), y.data_ptr(), nullptr, 0, st);
    }
    return status_or(r, y);
    END_HANDLE_TH_ERRORS
}

// nbody(bodies, eps2, out, dt, p, K)
PyObject *nbody(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    long v[3];
    if (n != 6 || !PyFloat_CheckExact(a[1]) || !ints(a + 3, 3, v)) return none();
    const int dt = (int)v[0];
    if (dt != HS_F32 && dt != HS_F64) return none();
    const hs_schedule s{(int32_t)v[1], (int32_t)v[2]};
    const at::Tensor *b = plain(a[0], in_type(dt), 2);
    if (!b || b->size(0) == 0 || b->size(1) != 4 || !b->is_contiguous()) return none();
    const int64_t nb = b->size(0);
    at::Tensor o;
    if (a[2] == Py_None) {
        o = empty({nb, 4}, in_type(dt), *b);
    } else {
        const at::Tensor *g = plain(a[2], in_type(dt), 2);
        if (!g || g->device() != b->device() || g->size(0) != nb || g->size(1) != 4 || !g->is_contiguous()) return none();
        o = *g;
    }
    const Workspace ws(f_workspace_size(HS_OP_NBODY, nb, 0, 0, dt, s), *b);
    void *st = current_stream();
    hs_status r;
    {
        NoGil g;
        r = f_nbody(nb, dt, s, b->data_ptr(), PyFloat_AS_DOUBLE(a[1]), o.data_ptr(), ws.ptr(), ws.bytes, st);
    }
    return status_or(r, o);
    END_HANDLE_TH_ERRORS
}

// connect(addresses of workspace_size, gemm, gemm_tn, gemm_noalloc, gemv, backward, nbody)
PyObject *connect(PyObject *, PyObject *const *a, Py_ssize_t n) {
    void *p[7];
    if (n != 7) return PyErr_Format(PyExc_TypeError, "connect takes 7 addresses");
    for (int i = 0; i < 7; ++i) {
        p[i] = PyLong_AsVoidPtr(a[i]);
        if (PyErr_Occurred()) return nullptr;
    }
    f_workspace_size = (decltype(f_workspace_size))p[0];
    f_gemm = (decltype(f_gemm))p[1];
    f_gemm_tn = (decltype(f_gemm_tn))p[2];
    f_gemm_noalloc = (decltype(f_gemm_noalloc))p[3];
    f_gemv = (decltype(f_gemv))p[4];
    f_backward = (decltype(f_backward))p[5];
    f_nbody = (decltype(f_nbody))p[6];
    Py_RETURN_NONE;
}

#define HS_M(f) {#f, (PyCFunction)(void (*)(void))f, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {HS_M(connect), HS_M(product), HS_M(backward), HS_M(gemv), HS_M(nbody), {}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_hs_torch", nullptr, -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__hs_torch(void) { return PyModule_Create(&module); }
