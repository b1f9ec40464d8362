/* The binding's small calls, in native code: what stands between a Python call and the launch (reading the tensors,
 * allocating the outputs, the current stream, the foreign call) took 7 - 11 us a call in Python, more than the kernels of
 * a decode step; here 3 - 4.  Each function returns NotImplemented for whatever is out of the ordinary (other argument
 * types, tensor subclasses, an active torch function mode, arguments that the checks refuse): the Python
 * form of the call then does it, or raises.  A number is the status of a refused call.  Marshalling only, like the rest of the binding. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "bitlinear.h"

namespace {

typedef bl_status (*quant_fn)(const uint16_t*, int64_t, int64_t, int8_t*, float*, int32_t*, bl_stream);
typedef bl_status (*product_fn)(const uint8_t*, const float*, int, const int8_t*, const float*, const int32_t*, int64_t,
                                int64_t, int64_t, int32_t*, float*, void*, bl_stream);
typedef bl_status (*decode_fn)(const uint8_t*, const float*, int, const uint16_t*, int64_t, int64_t, int64_t, int32_t*,
                               float*, int8_t*, float*, bl_stream);
quant_fn g_quant;
product_fn g_product[2];                 /* gemv, gemm */
decode_fn g_decode;
typedef bl_status (*run_fn)(void*, const bl_stack_plan*, bl_stream);
run_fn g_run;

/* A tensor argument: exactly torch.Tensor or None. */
bool get(PyObject* o, const at::Tensor** t) {
    if (o == Py_None) {
        *t = nullptr;
        return true;
    }
    if (!THPVariable_CheckExact(o)) return false;
    *t = &THPVariable_Unpack(o);
    return true;
}
void* ptr(const at::Tensor* t) { return t ? t->data_ptr() : nullptr; }
void* ptr(const at::Tensor& t) { return t.defined() ? t.data_ptr() : nullptr; }
bool get(PyObject* o, int64_t* v) {
    if (!PyLong_CheckExact(o)) return false;
    *v = PyLong_AsLongLong(o);
    if (*v == -1 && PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    return true;
}
bool get(PyObject* o, bool* v) {
    *v = o == Py_True;
    return o == Py_True || o == Py_False;
}
at::Tensor empty(c10::IntArrayRef size, at::ScalarType type, const at::Tensor& like) {
    return at::empty(size, at::TensorOptions().dtype(type).device(like.device()));
}
/* The 2-d device matrix that a call works on. */
bool matrix(const at::Tensor* t, at::ScalarType type) {
    return t && t->is_cuda() && t->scalar_type() == type && t->dim() == 2 && t->is_contiguous();
}
bool plain() { return at::impl::PythonTorchFunctionTLS::stack_len() == 0; }
int64_t padded(int64_t K) { return K >= 1 && K <= (int64_t)1 << 24 ? (K + 63) / 64 * 64 : 0; }
bl_stream stream() { return (bl_stream)c10::hip::getCurrentHIPStream().stream(); }
PyObject* wrap(at::Tensor t) {
    if (!t.defined()) Py_RETURN_NONE;
    return THPVariable_Wrap(std::move(t));
}
PyObject* other_way() { Py_RETURN_NOTIMPLEMENTED; }

/* f(): the call's result, or nullptr for the Python form; what torch throws (a tensor without storage, memory) goes there too. */
template <typename F>
PyObject* guarded(F f) {
    try {
        if (PyObject* r = f()) return r;
        if (PyErr_Occurred()) return nullptr;
    } catch (...) {
        PyErr_Clear();
    }
    return other_way();
}

PyObject* quant(PyObject*, PyObject* const* a, Py_ssize_t n) {   /* X, want_rowsum */
    return guarded([&]() -> PyObject* {
        const at::Tensor* X;
        bool want;
        if (n != 2 || !plain() || !get(a[0], &X) || !get(a[1], &want) || !matrix(X, at::kBFloat16)) return nullptr;
        const int64_t M = X->size(0), K = X->size(1);
        at::Tensor q = empty({M, padded(K)}, at::kChar, *X), scale = empty({M}, at::kFloat, *X), sum;
        if (want) sum = empty({M}, at::kInt, *X);
        const void* x = ptr(X);
        int8_t* qp = (int8_t*)ptr(q);
        float* sp = (float*)ptr(scale);
        int32_t* rp = (int32_t*)ptr(sum);
        const bl_stream st = stream();
        bl_status rc;
        Py_BEGIN_ALLOW_THREADS
        rc = g_quant((const uint16_t*)x, M, K, qp, sp, rp, st);
        Py_END_ALLOW_THREADS
        if (rc != BL_OK) return PyLong_FromLong(rc);
        return Py_BuildValue("(NNN)", wrap(std::move(q)), wrap(std::move(scale)), wrap(std::move(sum)));
    });
}

/* which, packed, beta, layout, q, scale, rowsum, N, want_acc, want_y, acc, y, workspace, K */
PyObject* product(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&]() -> PyObject* {
        int64_t which, layout, N, K;
        const at::Tensor *packed, *beta, *q, *scale, *rowsum, *acc, *y, *ws;
        bool want_acc, want_y;
        if (n != 14 || !plain() || !get(a[0], &which) || which < 0 || which > 1 || !get(a[1], &packed) || !get(a[2], &beta) ||
            !get(a[3], &layout) || layout != (int)layout || !get(a[4], &q) || !get(a[5], &scale) || !get(a[6], &rowsum) ||
            !get(a[7], &N) || N < 0 || !get(a[8], &want_acc) || !get(a[9], &want_y) || !get(a[10], &acc) || !get(a[11], &y) ||
            !get(a[12], &ws) || !matrix(q, at::kChar) || (!ws && !rowsum))
            return nullptr;
        const int64_t M = q->size(0);
        if (a[13] == Py_None) K = q->size(1);
        else if (!get(a[13], &K)) return nullptr;
        if (q->size(1) != padded(K)) return nullptr;
        at::Tensor acc_new, y_new;
        if (want_acc && !acc) acc_new = empty({M, N}, at::kInt, *q);
        if (want_y && !y) y_new = empty({M, N}, at::kFloat, *q);
        const void *p = ptr(packed), *b = ptr(beta), *qp = ptr(q), *s = ptr(scale), *r = ptr(rowsum);
        void *ap = acc ? ptr(acc) : ptr(acc_new), *yp = y ? ptr(y) : ptr(y_new), *w = ptr(ws);
        const bl_stream st = stream();
        bl_status rc;
        Py_BEGIN_ALLOW_THREADS
        rc = g_product[which]((const uint8_t*)p, (const float*)b, (int)layout, (const int8_t*)qp, (const float*)s,
                              (const int32_t*)r, M, N, K, (int32_t*)ap, (float*)yp, w, st);
        Py_END_ALLOW_THREADS
        if (rc != BL_OK) return PyLong_FromLong(rc);
        PyObject* ao = acc ? Py_NewRef(a[10]) : wrap(std::move(acc_new));
        PyObject* yo = y ? Py_NewRef(a[11]) : wrap(std::move(y_new));
        return Py_BuildValue("(NN)", ao, yo);
    });
}

/* packed, beta, layout, X, N, want_acc, want_y, want_q, acc, y */
PyObject* decode(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&]() -> PyObject* {
        int64_t layout, N;
        const at::Tensor *packed, *beta, *X, *acc, *y;
        bool want_acc, want_y, want_q;
        if (n != 10 || !plain() || !get(a[0], &packed) || !get(a[1], &beta) || !get(a[2], &layout) || layout != (int)layout ||
            !get(a[3], &X) || !get(a[4], &N) || N < 0 || !get(a[5], &want_acc) || !get(a[6], &want_y) || !get(a[7], &want_q) ||
            !get(a[8], &acc) || !get(a[9], &y) || !matrix(X, at::kBFloat16))
            return nullptr;
        const int64_t M = X->size(0), K = X->size(1);
        at::Tensor acc_new, y_new, q, scale;
        if (want_acc && !acc) acc_new = empty({M, N}, at::kInt, *X);
        if (want_y && !y) y_new = empty({M, N}, at::kFloat, *X);
        if (want_q) {
            q = empty({M, K}, at::kChar, *X);
            scale = empty({M}, at::kFloat, *X);
        }
        const void *p = ptr(packed), *b = ptr(beta), *x = ptr(X);
        void *ap = acc ? ptr(acc) : ptr(acc_new), *yp = y ? ptr(y) : ptr(y_new), *qp = ptr(q), *sp = ptr(scale);
        const bl_stream st = stream();
        bl_status rc;
        Py_BEGIN_ALLOW_THREADS
        rc = g_decode((const uint8_t*)p, (const float*)b, (int)layout, (const uint16_t*)x, M, N, K, (int32_t*)ap, (float*)yp,
                      (int8_t*)qp, (float*)sp, st);
        Py_END_ALLOW_THREADS
        if (rc != BL_OK) return PyLong_FromLong(rc);
        PyObject* ao = acc ? Py_NewRef(a[8]) : wrap(std::move(acc_new));
        PyObject* yo = y ? Py_NewRef(a[9]) : wrap(std::move(y_new));
        return Py_BuildValue("(NNNN)", ao, yo, wrap(std::move(q)), wrap(std::move(scale)));
    });
}

/* table, address of the host's bl_stack_plan */
PyObject* run(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&]() -> PyObject* {
        const at::Tensor* table;
        int64_t plan;
        if (n != 2 || !plain() || !get(a[0], &table) || !table || !get(a[1], &plan) || !plan) return nullptr;
        void* t = ptr(table);
        const bl_stream st = stream();
        bl_status rc;
        Py_BEGIN_ALLOW_THREADS
        rc = g_run(t, (const bl_stack_plan*)plan, st);
        Py_END_ALLOW_THREADS
        if (rc != BL_OK) return PyLong_FromLong(rc);
        Py_RETURN_NONE;
    });
}

/* The addresses of bl_quant_act_int8, bl_gemv_w158a8, bl_gemm_w158a8, bl_bitlinear_decode and bl_stack_run in the
 * loaded library. */
PyObject* bind(PyObject*, PyObject* args) {
    unsigned long long f[5];
    if (!PyArg_ParseTuple(args, "KKKKK", f, f + 1, f + 2, f + 3, f + 4)) return nullptr;
    g_run = (run_fn)f[4];
    g_quant = (quant_fn)f[0];
    g_product[0] = (product_fn)f[1];
    g_product[1] = (product_fn)f[2];
    g_decode = (decode_fn)f[3];
    Py_RETURN_NONE;
}

/* The current stream as the calls above see it (compared with the binding's own in a test). */
PyObject* current_stream(PyObject*, PyObject*) { return PyLong_FromUnsignedLongLong((unsigned long long)stream()); }

PyMethodDef methods[] = {{"quant", (PyCFunction)(void (*)(void))quant, METH_FASTCALL, nullptr},
                         {"product", (PyCFunction)(void (*)(void))product, METH_FASTCALL, nullptr},
                         {"decode", (PyCFunction)(void (*)(void))decode, METH_FASTCALL, nullptr},
                         {"run", (PyCFunction)(void (*)(void))run, METH_FASTCALL, nullptr},
                         {"bind", bind, METH_VARARGS, nullptr},
                         {"current_stream", current_stream, METH_NOARGS, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
/* (the doc string is what tells a build against another torch) */
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_bl_torch", "built for torch " BL_TORCH_VERSION, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__bl_torch(void) { return PyModule_Create(&module); }
