// Argument marshalling of the Python binding's hot calls.  A call of a small network or a small matrix product takes the
// GPU less time than its checks and ctypes conversions took in Python (gradient of 64-32-10: 17 us of checks and
// conversions for 10 us of kernels), so the same checks are made here on the tensors themselves.
//
// Every function returns the library's status, or None when ANY argument is not exactly what the fast path covers (a
// check that would fail, a tensor subclass, a missing result or workspace): the caller then takes the Python path, which
// makes the same checks one by one and raises the precise error.  Nothing is kept between calls.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <limits>

#include "../../include/ulsnn.h"

namespace {

struct Library {
    decltype(&ulsnn_sgemm) sgemm;
    decltype(&ulsnn_sgemm_ws) sgemm_ws;
    decltype(&ulsnn_mlp_grad) grad;
    decltype(&ulsnn_mlp_grad_mse) grad_mse;
    decltype(&ulsnn_mlp_loss) loss;
    decltype(&ulsnn_mlp_mse) mse;
    decltype(&ulsnn_mlp_grad_epoch) epoch;
    decltype(&ulsnn_cg_direction) cg;
    decltype(&ulsnn_dot) dot;
    decltype(&ulsnn_axpy) axpy;
} lib = {};

// A contiguous tensor on the GPU (torch.Tensor or Parameter itself, no subclass), or null.
const at::Tensor *gpu_tensor(PyObject *o)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    return t.defined() && t.is_cuda() && t.layout() == at::kStrided && t.is_contiguous() ? &t : nullptr;
}
const at::Tensor *typed(PyObject *o, at::ScalarType type)
{
    const at::Tensor *t = gpu_tensor(o);
    return t && t->scalar_type() == type ? t : nullptr;
}
const at::Tensor *f32_of(PyObject *o, int64_t numel)
{
    const at::Tensor *t = typed(o, at::kFloat);
    return t && t->numel() == numel ? t : nullptr;
}
bool is_matrix(const at::Tensor *t, int64_t rows, int64_t cols)
{
    return t && t->dim() == 2 && t->size(0) == rows && t->size(1) == cols;
}
template <class T = void>
T *data(const at::Tensor *t)
{
    return t ? static_cast<T *>(t->data_ptr()) : nullptr;
}
bool as_int(PyObject *o, int &v)
{
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    const long long x = PyLong_AsLongLongAndOverflow(o, &overflow);
    if (overflow || x < std::numeric_limits<int>::min() || x > std::numeric_limits<int>::max()) return false;
    v = (int)x;
    return true;
}
bool as_float(PyObject *o, float &v)
{
    if (PyFloat_CheckExact(o)) v = (float)PyFloat_AS_DOUBLE(o);
    else {
        int i = 0;
        if (!as_int(o, i)) return false;
        v = (float)i;
    }
    return true;
}
bool as_pointer(PyObject *o, void *&p)
{
    if (!PyLong_CheckExact(o)) return false;
    p = PyLong_AsVoidPtr(o);
    if (PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    return true;
}
bool as_trans(PyObject *o, char &c)
{
    if (!PyUnicode_CheckExact(o) || PyUnicode_GET_LENGTH(o) < 1) return false;
    const Py_UCS4 u = PyUnicode_READ_CHAR(o, 0);
    if (u != 'N' && u != 'n' && u != 'T' && u != 't' && u != 'C' && u != 'c') return false;
    c = (char)u;
    return true;
}

// A tensor that has no storage to point at (a functorch wrapper, say) throws from the calls above: such a call takes the
// Python path, where the same calls raise their error.
template <PyObject *(*F)(PyObject *const *, Py_ssize_t)>
PyObject *guarded(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    try {
        return F(a, n);
    } catch (...) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

template <class F>
PyObject *run(F &&call)
{
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = call();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// sgemm(transa, transb, m, n, k, alpha, A, lda, B, ldb, beta, C, ldc, workspace or None, stream)
PyObject *fast_sgemm(PyObject *const *a, Py_ssize_t n_args)
{
    char ta, tb;
    int m, n, k, lda, ldb, ldc;
    float alpha, beta;
    void *stream;
    if (n_args != 15 || !lib.sgemm || !as_trans(a[0], ta) || !as_trans(a[1], tb) || !as_int(a[2], m) || !as_int(a[3], n) ||
        !as_int(a[4], k) || !as_float(a[5], alpha) || !as_int(a[7], lda) || !as_int(a[9], ldb) || !as_float(a[10], beta) ||
        !as_int(a[12], ldc) || !as_pointer(a[14], stream))
        Py_RETURN_NONE;
    const at::Tensor *A = typed(a[6], at::kFloat), *B = typed(a[8], at::kFloat), *C = typed(a[11], at::kFloat), *ws = nullptr;
    if (!A || !B || !C || m < 1 || n < 1 || k < 1) Py_RETURN_NONE;
    if (a[13] != Py_None && !(ws = gpu_tensor(a[13]))) Py_RETURN_NONE;
    // every element the product touches lies inside its tensor
    auto holds = [](const at::Tensor *t, int64_t rows, int64_t cols, int64_t ld) {
        return ld >= cols && (rows - 1) * ld + cols <= t->numel();
    };
    const bool na = ta == 'N' || ta == 'n', nb = tb == 'N' || tb == 'n';
    if (!holds(C, m, n, ldc) || !holds(A, na ? m : k, na ? k : m, lda) || !holds(B, nb ? k : n, nb ? n : k, ldb)) Py_RETURN_NONE;
    const float *pa = data<float>(A), *pb = data<float>(B);
    float *pc = data<float>(C);
    if (a[13] == Py_None) return run([&] { return lib.sgemm(ta, tb, m, n, k, alpha, pa, lda, pb, ldb, beta, pc, ldc, stream); });
    void *pw = data(ws);
    const size_t bytes = ws->numel() * ws->element_size();
    return run([&] { return lib.sgemm_ws(ta, tb, m, n, k, alpha, pa, lda, pb, ldb, beta, pc, ldc, pw, bytes, stream); });
}

enum Form { GRAD = 0, GRAD_MSE = 1, LOSS = 2, MSE = 3, EPOCH = 4 };

// mlp(form, W1, W2, X, labels or T, b1, b2, dW1, dW2, loss, db1, db2, accumulate, chunk, workspace, stream); an error-only
// form takes None for the gradients
PyObject *fast_mlp(PyObject *const *a, Py_ssize_t n_args)
{
    int form, chunk;
    void *stream;
    if (n_args != 16 || !lib.grad || !as_int(a[0], form) || (a[12] != Py_True && a[12] != Py_False) || !as_int(a[13], chunk) ||
        !as_pointer(a[15], stream))
        Py_RETURN_NONE;
    const bool dense = form == GRAD_MSE || form == MSE, backward = form != LOSS && form != MSE;
    const at::Tensor *W1 = gpu_tensor(a[1]);
    if (!W1 || W1->dim() != 2) Py_RETURN_NONE;
    const at::ScalarType type = W1->scalar_type();
    if (type != at::kFloat && type != at::kBFloat16) Py_RETURN_NONE;
    const at::Tensor *W2 = typed(a[2], type), *X = typed(a[3], type), *ws = gpu_tensor(a[14]);
    const at::Tensor *T = typed(a[4], dense ? at::kFloat : at::kInt), *loss = f32_of(a[9], 1);
    if (!W2 || !X || !T || !ws || !loss || W2->dim() != 2 || X->dim() != 2) Py_RETURN_NONE;
    const int64_t n_in = W1->size(0), n_hid = W1->size(1), n_out = W2->size(1), batch = X->size(0);
    const int64_t most = std::numeric_limits<int>::max();
    if (W2->size(0) != n_hid || X->size(1) != n_in || n_in > most || n_hid > most || n_out > most ||
        (form != EPOCH && batch > most))
        Py_RETURN_NONE;
    if (dense ? !is_matrix(T, batch, n_out) : (T->dim() < 1 || T->size(0) != batch)) Py_RETURN_NONE;
    ulsnn_mlp_desc d = {};
    const bool biases = a[5] != Py_None;
    if (biases != (a[6] != Py_None)) Py_RETURN_NONE;
    if (biases) {
        const at::Tensor *b1 = f32_of(a[5], n_hid), *b2 = f32_of(a[6], n_out);
        if (!b1 || !b2) Py_RETURN_NONE;
        d.b1 = data<float>(b1);
        d.b2 = data<float>(b2);
    }
    const at::Tensor *dW1 = nullptr, *dW2 = nullptr;
    if (backward) {
        dW1 = typed(a[7], at::kFloat);
        dW2 = typed(a[8], at::kFloat);
        if (!is_matrix(dW1, n_in, n_hid) || !is_matrix(dW2, n_hid, n_out)) Py_RETURN_NONE;
        if (biases) {
            const at::Tensor *db1 = f32_of(a[10], n_hid), *db2 = f32_of(a[11], n_out);
            if (!db1 || !db2) Py_RETURN_NONE;
            d.db1 = data<float>(db1);
            d.db2 = data<float>(db2);
        } else if (a[10] != Py_None || a[11] != Py_None) {
            Py_RETURN_NONE;
        }
    }
    d.n_in = (int)n_in; d.n_hid = (int)n_hid; d.n_out = (int)n_out;
    d.accumulate = a[12] == Py_True;
    d.operand_dtype = type == at::kBFloat16;
    d.workspace = data(ws);
    d.workspace_bytes = ws->numel() * ws->element_size();
    d.hip_stream = stream;
    const void *w1 = data(W1), *w2 = data(W2), *x = data(X);
    const int32_t *y = dense ? nullptr : data<int32_t>(T);
    const float *t = dense ? data<float>(T) : nullptr;
    float *g1 = data<float>(dW1), *g2 = data<float>(dW2), *l = data<float>(loss);
    return run([&] {
        switch (form) {
            case GRAD: return lib.grad(&d, w1, w2, x, y, (int)batch, g1, g2, l);
            case GRAD_MSE: return lib.grad_mse(&d, w1, w2, x, t, (int)batch, g1, g2, l);
            case LOSS: return lib.loss(&d, w1, w2, x, y, (int)batch, l);
            case MSE: return lib.mse(&d, w1, w2, x, t, (int)batch, l);
            default: return lib.epoch(&d, w1, w2, x, y, batch, chunk, g1, g2, l);
        }
    });
}

// cg(g_new, g_old or None, d, beta, workspace, stream)
PyObject *fast_cg(PyObject *const *a, Py_ssize_t n_args)
{
    void *stream;
    if (n_args != 6 || !lib.cg || !as_pointer(a[5], stream)) Py_RETURN_NONE;
    const at::Tensor *g = typed(a[0], at::kFloat), *ws = gpu_tensor(a[4]), *old = nullptr;
    if (!g || !ws || ws->element_size() != 1) Py_RETURN_NONE;
    const int64_t n = g->numel();
    const at::Tensor *d = f32_of(a[2], n), *beta = f32_of(a[3], 1);
    if (!d || !beta || (a[1] != Py_None && !(old = f32_of(a[1], n)))) Py_RETURN_NONE;
    const float *pg = data<float>(g), *po = data<float>(old);
    float *pd = data<float>(d), *pb = data<float>(beta);
    void *pw = data(ws);
    const size_t bytes = ws->numel() * ws->element_size();
    return run([&] { return lib.cg(n, pg, po, pd, pb, pw, bytes, stream); });
}

// dot(x, y, out, workspace, stream)
PyObject *fast_dot(PyObject *const *a, Py_ssize_t n_args)
{
    void *stream;
    if (n_args != 5 || !lib.dot || !as_pointer(a[4], stream)) Py_RETURN_NONE;
    const at::Tensor *x = typed(a[0], at::kFloat), *ws = gpu_tensor(a[3]);
    if (!x || !ws || ws->element_size() != 1) Py_RETURN_NONE;
    const at::Tensor *y = f32_of(a[1], x->numel()), *out = f32_of(a[2], 1);
    if (!y || !out) Py_RETURN_NONE;
    const int64_t n = x->numel();
    const float *px = data<float>(x), *py = data<float>(y);
    float *po = data<float>(out);
    void *pw = data(ws);
    const size_t bytes = ws->numel() * ws->element_size();
    return run([&] { return lib.dot(n, px, py, po, pw, bytes, stream); });
}

// axpy(alpha, x, y, stream)
PyObject *fast_axpy(PyObject *const *a, Py_ssize_t n_args)
{
    void *stream;
    float alpha;
    if (n_args != 4 || !lib.axpy || !as_float(a[0], alpha) || !as_pointer(a[3], stream)) Py_RETURN_NONE;
    const at::Tensor *x = typed(a[1], at::kFloat);
    if (!x) Py_RETURN_NONE;
    const at::Tensor *y = f32_of(a[2], x->numel());
    if (!y) Py_RETURN_NONE;
    const int64_t n = x->numel();
    const float *px = data<float>(x);
    float *py = data<float>(y);
    return run([&] { return lib.axpy(n, alpha, px, py, stream); });
}

// bind(address, ...): the library's entry points in the order of struct Library
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n_args)
{
    void *p[10];
    if (n_args != 10) {
        PyErr_SetString(PyExc_TypeError, "bind: ten addresses");
        return nullptr;
    }
    for (int i = 0; i < 10; ++i) {
        if (!as_pointer(a[i], p[i])) {
            PyErr_SetString(PyExc_TypeError, "bind: addresses are integers");
            return nullptr;
        }
    }
    lib.sgemm = (decltype(lib.sgemm))p[0]; lib.sgemm_ws = (decltype(lib.sgemm_ws))p[1];
    lib.grad = (decltype(lib.grad))p[2]; lib.grad_mse = (decltype(lib.grad_mse))p[3];
    lib.loss = (decltype(lib.loss))p[4]; lib.mse = (decltype(lib.mse))p[5];
    lib.epoch = (decltype(lib.epoch))p[6]; lib.cg = (decltype(lib.cg))p[7];
    lib.dot = (decltype(lib.dot))p[8]; lib.axpy = (decltype(lib.axpy))p[9];
    Py_RETURN_NONE;
}

#define FAST(f) (PyCFunction)(void (*)(void))(f), METH_FASTCALL, nullptr
PyMethodDef methods[] = {{"bind", FAST(bind)}, {"sgemm", FAST(guarded<fast_sgemm>)}, {"mlp", FAST(guarded<fast_mlp>)}, {"cg", FAST(guarded<fast_cg>)},
                         {"dot", FAST(guarded<fast_dot>)}, {"axpy", FAST(guarded<fast_axpy>)}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fast_call", nullptr, -1, methods};

}  // namespace

// torch_version: the torch whose tensors this file was compiled to read; the binding uses the module with no other.
PyMODINIT_FUNC PyInit__fast_call(void)
{
    PyObject *m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "torch_version", BUILT_WITH_TORCH) != 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
