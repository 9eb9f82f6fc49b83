// Argument marshalling of binding.py in native code: the checks that the Python functions make, the output tensors, the current
// stream and the call of the C entry point.  In Python these bound what a latency-bound program gets: host time of a call with its
// launches, Python -> here, one query over a ragged corpus 9.2 -> 4.4 us, over a uniform one 8.5 -> 4.2, forward with argmax 10.5 -> 5.1,
// cross-entropy gradient 9.2 -> 5.1, backward 11.9 -> 5.4, a training step of 16 x 16 31.7 -> 15.2.
//
// A function returns the Python function's result, an int (the error code of the C entry point), or None where anything about the
// call is out of the ordinary -- a tensor of another class, kind, type, shape, device or memory layout, an active
// mode that watches torch calls, a value it does not know.  binding.py then does the same work in Python and raises what there is to raise.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/TensorSubclassLikeUtils.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <climits>

#include "../../include/maxsim.h"

namespace {

struct Entries {
    decltype(&maxsim_forward) forward;
    decltype(&maxsim_forward_ragged) forward_ragged;
    decltype(&maxsim_backward) backward;
    decltype(&maxsim_backward_ragged) backward_ragged;
    decltype(&maxsim_ce_grad) ce_grad;
    decltype(&maxsim_quantize_rows_i8) quantize;
    decltype(&maxsim_forward_i8) forward_i8;
    decltype(&maxsim_forward_i8_ragged) forward_i8_ragged;
} entry;

// One call's arguments.  ok() after everything has been looked at: nothing was out of the ordinary.
class Call {
public:
    explicit Call(PyObject *first) { ok_ = !c10::impl::TorchDispatchModeTLS::any_modes_set() && !at::impl::torch_function_mode_enabled() && plain(first) != nullptr; }

    bool ok() const { return ok_; }
    void require(bool x) { ok_ = ok_ && x; }

    // A contiguous tensor of the call's GPU, which is that of the first one and the current one
    const at::Tensor &tensor(PyObject *o, int dims)
    {
        const at::Tensor *t = ok_ ? plain(o) : nullptr;
        if (!t || t->dim() != dims || !t->is_contiguous()) {
            ok_ = false;
            return none();
        }
        if (device_ < 0) {
            device_ = t->get_device();
            ok_ = device_ == c10::hip::current_device();
        }
        ok_ = ok_ && t->get_device() == device_;
        return *t;
    }
    const at::Tensor &tensor(PyObject *o, at::IntArrayRef shape, at::ScalarType type)
    {
        const at::Tensor &t = tensor(o, (int)shape.size());
        ok_ = ok_ && t.scalar_type() == type && t.sizes() == shape;
        return ok_ ? t : none();
    }
    // The caller's output or, for None, a new one
    at::Tensor output(PyObject *o, at::IntArrayRef shape, at::ScalarType type)
    {
        if (o != Py_None)
            return tensor(o, shape, type);
        return ok_ ? at::empty(shape, at::TensorOptions().dtype(type).device(at::kCUDA, device_)) : at::Tensor();
    }
    int size(int64_t n)
    {
        ok_ = ok_ && n >= 0 && n <= INT_MAX;
        return ok_ ? (int)n : 0;
    }
    maxsim_dtype dtype(const at::Tensor &t)
    {
        switch (ok_ ? t.scalar_type() : at::ScalarType::Undefined) {
        case at::ScalarType::Float: return MAXSIM_F32;
        case at::ScalarType::Half: return MAXSIM_F16;
        case at::ScalarType::BFloat16: return MAXSIM_BF16;
        default: ok_ = false; return MAXSIM_F32;
        }
    }
    void *stream() const { return c10::hip::getCurrentHIPStream((c10::DeviceIndex)device_).stream(); }

private:
    static const at::Tensor &none() // (not looked at: ok() is false)
    {
        static const at::Tensor t;
        return t;
    }
    static const at::Tensor *plain(PyObject *o)
    {
        if (!THPVariable_CheckExact(o))
            return nullptr;
        const at::Tensor &t = THPVariable_Unpack(o);
        return t.defined() && t.is_cuda() && !at::isTensorSubclassLike(t) && t.layout() == at::kStrided && !t.is_neg() && !t.is_conj() ? &t : nullptr;
    }
    bool ok_ = false;
    int device_ = -1;
};

const void *in(const at::Tensor &t) { return t.data_ptr(); }
template <typename T> T *at_ptr(const at::Tensor &t) { return static_cast<T *>(t.data_ptr()); }

PyObject *give(PyObject *given, const at::Tensor &t) // the caller's own object, or the new tensor
{
    if (given == Py_None)
        return THPVariable_Wrap(t);
    Py_INCREF(given);
    return given;
}
PyObject *give2(PyObject *g0, const at::Tensor &t0, PyObject *g1, const at::Tensor &t1)
{
    PyObject *a = give(g0, t0);
    PyObject *b = a ? give(g1, t1) : nullptr;
    PyObject *r = b ? PyTuple_Pack(2, a, b) : nullptr;
    Py_XDECREF(a);
    Py_XDECREF(b);
    return r;
}

template <typename F> int without_gil(F &&f)
{
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f();
    Py_END_ALLOW_THREADS
    return rc;
}

#define ARGUMENTS(N)                                                                                                   \
    if (n != (N)) {                                                                                                    \
        PyErr_SetString(PyExc_TypeError, "wrong number of arguments");                                                 \
        return nullptr;                                                                                                \
    }

// (Q, D, scores, argmax, want_argmax)
PyObject *forward(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    ARGUMENTS(5)
    Call c(a[0]);
    const at::Tensor &Q = c.tensor(a[0], 3), &D = c.tensor(a[1], 3);
    const maxsim_dtype dt = c.dtype(Q);
    c.require(c.ok() && D.scalar_type() == Q.scalar_type() && D.size(2) == Q.size(2));
    if (!c.ok())
        Py_RETURN_NONE;
    const int n_q = c.size(Q.size(0)), l_q = c.size(Q.size(1)), d = c.size(Q.size(2)), l_d = c.size(D.size(1));
    const int64_t b = D.size(0);
    const int want = a[3] != Py_None ? 1 : PyObject_IsTrue(a[4]);
    if (want < 0)
        return nullptr;
    const at::Tensor scores = c.output(a[2], {n_q, b}, at::kFloat);
    const at::Tensor argmax = want ? c.output(a[3], {n_q, b, l_q}, at::kInt) : at::Tensor();
    if (!c.ok())
        Py_RETURN_NONE;
    const int rc = without_gil([&] {
        return entry.forward(in(Q), n_q, l_q, in(D), b, l_d, d, dt, at_ptr<float>(scores), want ? at_ptr<int32_t>(argmax) : nullptr, c.stream());
    });
    if (rc != 0)
        return PyLong_FromLong(rc);
    return want ? give2(a[2], scores, a[3], argmax) : give(a[2], scores);
    END_HANDLE_TH_ERRORS
}

// (Q, D_packed, doc_offsets, scores, argmax, want_argmax): all rows of D_packed
PyObject *forward_ragged(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    ARGUMENTS(6)
    Call c(a[0]);
    const at::Tensor &Q = c.tensor(a[0], 3), &D = c.tensor(a[1], 2), &off = c.tensor(a[2], 1);
    const maxsim_dtype dt = c.dtype(Q);
    c.require(c.ok() && D.scalar_type() == Q.scalar_type() && D.size(1) == Q.size(2) && off.scalar_type() == at::kInt && off.size(0) >= 2);
    if (!c.ok())
        Py_RETURN_NONE;
    const int n_q = c.size(Q.size(0)), l_q = c.size(Q.size(1)), d = c.size(Q.size(2));
    const int64_t b = off.size(0) - 1, tokens = D.size(0);
    const int want = a[4] != Py_None ? 1 : PyObject_IsTrue(a[5]);
    if (want < 0)
        return nullptr;
    const at::Tensor scores = c.output(a[3], {n_q, b}, at::kFloat);
    const at::Tensor argmax = want ? c.output(a[4], {n_q, b, l_q}, at::kInt) : at::Tensor();
    if (!c.ok())
        Py_RETURN_NONE;
    const int rc = without_gil([&] {
        return entry.forward_ragged(in(Q), n_q, l_q, in(D), at_ptr<int32_t>(off), b, tokens, d, dt, at_ptr<float>(scores), want ? at_ptr<int32_t>(argmax) : nullptr, c.stream());
    });
    if (rc != 0)
        return PyLong_FromLong(rc);
    return want ? give2(a[3], scores, a[4], argmax) : give(a[3], scores);
    END_HANDLE_TH_ERRORS
}

// (Q, D, argmax, dscore, dQ, dD)
PyObject *backward(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    ARGUMENTS(6)
    Call c(a[0]);
    const at::Tensor &Q = c.tensor(a[0], 3), &D = c.tensor(a[1], 3);
    const maxsim_dtype dt = c.dtype(Q);
    c.require(c.ok() && D.scalar_type() == Q.scalar_type() && D.size(2) == Q.size(2));
    if (!c.ok())
        Py_RETURN_NONE;
    const int n_q = c.size(Q.size(0)), l_q = c.size(Q.size(1)), d = c.size(Q.size(2)), l_d = c.size(D.size(1));
    const int64_t b = D.size(0);
    const at::Tensor &A = c.tensor(a[2], {n_q, b, l_q}, at::kInt), &g = c.tensor(a[3], {n_q, b}, at::kFloat);
    const at::Tensor dQ = c.output(a[4], {n_q, l_q, d}, at::kFloat);
    const at::Tensor dD = c.output(a[5], {b, l_d, d}, at::kFloat);
    if (!c.ok())
        Py_RETURN_NONE;
    const int rc = without_gil([&] {
        return entry.backward(in(Q), n_q, l_q, in(D), b, l_d, d, dt, at_ptr<int32_t>(A), at_ptr<float>(g), at_ptr<float>(dQ), at_ptr<float>(dD), c.stream());
    });
    return rc != 0 ? PyLong_FromLong(rc) : give2(a[4], dQ, a[5], dD);
    END_HANDLE_TH_ERRORS
}

// (Q, D_packed, doc_offsets, argmax, dscore, dQ, dD): all rows of D_packed
PyObject *backward_ragged(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    ARGUMENTS(7)
    Call c(a[0]);
    const at::Tensor &Q = c.tensor(a[0], 3), &D = c.tensor(a[1], 2), &off = c.tensor(a[2], 1);
    const maxsim_dtype dt = c.dtype(Q);
    c.require(c.ok() && D.scalar_type() == Q.scalar_type() && D.size(1) == Q.size(2) && off.scalar_type() == at::kInt && off.size(0) >= 2);
    if (!c.ok())
        Py_RETURN_NONE;
    const int n_q = c.size(Q.size(0)), l_q = c.size(Q.size(1)), d = c.size(Q.size(2));
    const int64_t b = off.size(0) - 1, tokens = D.size(0);
    const at::Tensor &A = c.tensor(a[3], {n_q, b, l_q}, at::kInt), &g = c.tensor(a[4], {n_q, b}, at::kFloat);
    const at::Tensor dQ = c.output(a[5], {n_q, l_q, d}, at::kFloat);
    const at::Tensor dD = c.output(a[6], {tokens, d}, at::kFloat);
    if (!c.ok())
        Py_RETURN_NONE;
    const int rc = without_gil([&] {
        return entry.backward_ragged(in(Q), n_q, l_q, in(D), at_ptr<int32_t>(off), b, tokens, d, dt, at_ptr<int32_t>(A), at_ptr<float>(g), at_ptr<float>(dQ), at_ptr<float>(dD),
                                     c.stream());
    });
    return rc != 0 ? PyLong_FromLong(rc) : give2(a[5], dQ, a[6], dD);
    END_HANDLE_TH_ERRORS
}

// (scores, tau, g, loss)
PyObject *ce_grad(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    ARGUMENTS(4)
    Call c(a[0]);
    const at::Tensor &s = c.tensor(a[0], 2);
    if (!c.ok() || s.scalar_type() != at::kFloat || !PyFloat_CheckExact(a[1]))
        Py_RETURN_NONE;
    const int rows = c.size(s.size(0)), b = c.size(s.size(1));
    const float tau = (float)PyFloat_AS_DOUBLE(a[1]);
    const at::Tensor g = c.output(a[2], {rows, b}, at::kFloat);
    const at::Tensor loss = c.output(a[3], {1}, at::kFloat);
    if (!c.ok())
        Py_RETURN_NONE;
    const int rc = without_gil([&] { return entry.ce_grad(at_ptr<float>(s), rows, b, tau, at_ptr<float>(g), at_ptr<float>(loss), c.stream()); });
    return rc != 0 ? PyLong_FromLong(rc) : give2(a[2], g, a[3], loss);
    END_HANDLE_TH_ERRORS
}

// (X, X_i8, scale): X of two or three dimensions
PyObject *quantize(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    ARGUMENTS(3)
    Call c(a[0]);
    if (!c.ok())
        Py_RETURN_NONE;
    const int64_t dims = THPVariable_Unpack(a[0]).dim();
    const at::Tensor &X = c.tensor(a[0], dims == 2 ? 2 : 3);
    const maxsim_dtype dt = c.dtype(X);
    if (!c.ok() || X.numel() == 0)
        Py_RETURN_NONE;
    const int d = c.size(X.size(-1));
    const at::Tensor codes = c.output(a[1], X.sizes(), at::kChar);
    const at::Tensor scale = c.output(a[2], X.sizes().slice(0, dims - 1), at::kFloat);
    if (!c.ok())
        Py_RETURN_NONE;
    const int rc = without_gil([&] { return entry.quantize(in(X), X.numel() / d, d, dt, at_ptr<int8_t>(codes), at_ptr<float>(scale), c.stream()); });
    return rc != 0 ? PyLong_FromLong(rc) : give2(a[1], codes, a[2], scale);
    END_HANDLE_TH_ERRORS
}

// (Q_i8, q_scale, D_i8, d_scale, scores)
PyObject *forward_i8(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    ARGUMENTS(5)
    Call c(a[0]);
    const at::Tensor &Q = c.tensor(a[0], 3), &D = c.tensor(a[2], 3);
    c.require(c.ok() && Q.scalar_type() == at::kChar && D.scalar_type() == at::kChar && D.size(2) == Q.size(2));
    if (!c.ok())
        Py_RETURN_NONE;
    const int n_q = c.size(Q.size(0)), l_q = c.size(Q.size(1)), d = c.size(Q.size(2)), l_d = c.size(D.size(1));
    const int64_t b = D.size(0);
    const at::Tensor &qs = c.tensor(a[1], {n_q, l_q}, at::kFloat), &ds = c.tensor(a[3], {b, l_d}, at::kFloat);
    const at::Tensor scores = c.output(a[4], {n_q, b}, at::kFloat);
    if (!c.ok())
        Py_RETURN_NONE;
    const int rc = without_gil([&] {
        return entry.forward_i8(at_ptr<int8_t>(Q), at_ptr<float>(qs), n_q, l_q, at_ptr<int8_t>(D), at_ptr<float>(ds), b, l_d, d, at_ptr<float>(scores), c.stream());
    });
    return rc != 0 ? PyLong_FromLong(rc) : give(a[4], scores);
    END_HANDLE_TH_ERRORS
}

// (Q_i8, q_scale, D_i8_packed, d_scale_packed, doc_offsets, scores): all rows of D_i8_packed
PyObject *forward_i8_ragged(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    ARGUMENTS(6)
    Call c(a[0]);
    const at::Tensor &Q = c.tensor(a[0], 3), &D = c.tensor(a[2], 2), &off = c.tensor(a[4], 1);
    c.require(c.ok() && Q.scalar_type() == at::kChar && D.scalar_type() == at::kChar && D.size(1) == Q.size(2) && off.scalar_type() == at::kInt && off.size(0) >= 2);
    if (!c.ok())
        Py_RETURN_NONE;
    const int n_q = c.size(Q.size(0)), l_q = c.size(Q.size(1)), d = c.size(Q.size(2));
    const int64_t b = off.size(0) - 1, tokens = D.size(0);
    const at::Tensor &qs = c.tensor(a[1], {n_q, l_q}, at::kFloat), &ds = c.tensor(a[3], {tokens}, at::kFloat);
    const at::Tensor scores = c.output(a[5], {n_q, b}, at::kFloat);
    if (!c.ok())
        Py_RETURN_NONE;
    const int rc = without_gil([&] {
        return entry.forward_i8_ragged(at_ptr<int8_t>(Q), at_ptr<float>(qs), n_q, l_q, at_ptr<int8_t>(D), at_ptr<float>(ds), at_ptr<int32_t>(off), b, tokens, d, at_ptr<float>(scores),
                                       c.stream());
    });
    return rc != 0 ? PyLong_FromLong(rc) : give(a[5], scores);
    END_HANDLE_TH_ERRORS
}

// The addresses of the entry points in the library that binding.py has loaded, in the order of Entries
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    ARGUMENTS(8)
    void *p[8];
    for (int i = 0; i < 8; ++i) {
        p[i] = PyLong_AsVoidPtr(a[i]);
        if (PyErr_Occurred())
            return nullptr;
    }
    int i = 0;
    entry.forward = reinterpret_cast<decltype(entry.forward)>(p[i++]);
    entry.forward_ragged = reinterpret_cast<decltype(entry.forward_ragged)>(p[i++]);
    entry.backward = reinterpret_cast<decltype(entry.backward)>(p[i++]);
    entry.backward_ragged = reinterpret_cast<decltype(entry.backward_ragged)>(p[i++]);
    entry.ce_grad = reinterpret_cast<decltype(entry.ce_grad)>(p[i++]);
    entry.quantize = reinterpret_cast<decltype(entry.quantize)>(p[i++]);
    entry.forward_i8 = reinterpret_cast<decltype(entry.forward_i8)>(p[i++]);
    entry.forward_i8_ragged = reinterpret_cast<decltype(entry.forward_i8_ragged)>(p[i++]);
    Py_RETURN_NONE;
}

#define METHOD(NAME) {#NAME, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(NAME)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {METHOD(bind),     METHOD(forward),    METHOD(forward_ragged),    METHOD(backward), METHOD(backward_ragged), METHOD(ce_grad),
                         METHOD(quantize), METHOD(forward_i8), METHOD(forward_i8_ragged), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

} // namespace

PyMODINIT_FUNC PyInit__marshal()
{
    PyObject *m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "BUILT_FOR", MARSHAL_ABI) < 0) { // (binding.py looks at it before anything else)
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
