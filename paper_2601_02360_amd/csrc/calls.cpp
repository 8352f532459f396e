// The calls of binding.py that launch kernels, from Python objects to the C ABI in one step: arguments converted, tensors
// checked, the current stream looked up.  In Python that took 1 to 4 us a call beside the 2.6 us of a launch, and two such
// launches of a few us each waited for it.  Every function returns the status of the call, or None where an argument is not plainly what the call
// takes: binding.py then looks at the arguments one by one, and raises what there is to raise.
#include <Python.h>

#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <climits>

#include "sparseloco.h"

namespace {

// Arguments of a call in order; ok turns false at the first that does not fit.
struct Args {
    PyObject* const* at;
    Py_ssize_t left;
    bool ok = true;

    PyObject* next() {
        if (left < 1) { ok = false; return Py_None; }
        --left;
        return *at++;
    }
    void* address() {                                         // int, or None for a null pointer
        PyObject* o = next();
        if (o == Py_None) return nullptr;
        if (!PyLong_CheckExact(o)) { ok = false; return nullptr; }
        void* p = PyLong_AsVoidPtr(o);
        if (p == nullptr && PyErr_Occurred()) { PyErr_Clear(); ok = false; }
        return p;
    }
    template <class T>
    const T* handle() { return static_cast<const T*>(address()); }
    int64_t integer(int64_t low, int64_t high) {
        PyObject* o = next();
        if (!PyLong_Check(o)) { ok = false; return 0; }
        int overflow = 0;
        const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
        if (overflow != 0 || v < low || v > high) ok = false;
        return v;
    }
    int integer() { return (int)integer(INT_MIN, INT_MAX); }
    float number() {
        PyObject* o = next();
        if (PyFloat_CheckExact(o)) return (float)PyFloat_AS_DOUBLE(o);
        ok = false;
        return 0.f;
    }
    // A contiguous GPU tensor of this type; what it is otherwise is left to Python.
    const at::Tensor* tensor(at::ScalarType type) {
        PyObject* o = next();
        if (!ok || !THPVariable_CheckExact(o)) { ok = false; return nullptr; }
        const at::Tensor& t = THPVariable_Unpack(o);
        if (t.scalar_type() != type || !t.is_cuda() || !t.is_contiguous()) { ok = false; return nullptr; }
        return &t;
    }
    void* flat(at::ScalarType type, int64_t numel) {
        const at::Tensor* t = tensor(type);
        if (!t || t->numel() != numel) { ok = false; return nullptr; }
        return t->data_ptr();
    }
    // A matrix; rows, cols < 0: whatever they are, and they are written back.
    float* matrix(int64_t& rows, int64_t& cols, at::ScalarType type = at::kFloat) {
        const at::Tensor* t = tensor(type);
        if (!t || t->dim() != 2) { ok = false; return nullptr; }
        if (rows < 0) rows = t->size(0);
        if (cols < 0) cols = t->size(1);
        if (t->size(0) != rows || t->size(1) != cols) { ok = false; return nullptr; }
        return static_cast<float*>(t->data_ptr());
    }
    bool none() {
        if (left < 1 || *at != Py_None) return false;
        next();
        return true;
    }
    void* stream() {                                          // the last argument: None for the current stream
        if (!none()) return address();
        return c10::hip::getCurrentHIPStream(c10::hip::current_device()).stream();
    }
};

// The call itself without the interpreter's lock, as ctypes does it: a launch may wait for room in the queue.
template <class Call>
PyObject* finish(const Args& a, Call call) {
    if (!a.ok || a.left != 0) Py_RETURN_NONE;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = call();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// Nothing that torch throws (tensors without storage, streams of a device that is gone) leaves a function here: Python
// meets it again on its own way through the arguments.
template <class Body>
PyObject* guarded(PyObject* const* args, Py_ssize_t n, Body body) {
    try {
        return body(Args{args, n});
    } catch (...) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

PyObject* compress(PyObject*, PyObject* const* args, Py_ssize_t n) {
    return guarded(args, n, [](Args a) {
        const auto* plan = a.handle<sparseloco_plan>();
        const int mode = a.integer();
        const auto *src_a = a.handle<sparseloco_tensors>(), *src_b = a.handle<sparseloco_tensors>(),
                   *ef = a.handle<sparseloco_tensors>();
        const int replica = a.integer();
        const float beta = a.number();
        const int64_t n_pairs = a.integer(0, INT64_MAX), n_aux = a.integer(0, INT64_MAX);
        auto* pairs = static_cast<uint16_t*>(a.flat(at::kShort, n_pairs));
        auto* aux = static_cast<float*>(a.flat(at::kFloat, n_aux));
        void* stream = a.stream();
        return finish(a, [&] { return sparseloco_compress(plan, mode, src_a, src_b, ef, replica, beta, pairs, aux, stream); });
    });
}

PyObject* aggregate(PyObject*, PyObject* const* args, Py_ssize_t n) {
    return guarded(args, n, [](Args a) {
        const auto* plan = a.handle<sparseloco_plan>();
        const auto* messages = a.handle<sparseloco_messages>();
        const auto* mean = a.handle<sparseloco_tensors>();
        void* stream = a.stream();
        return finish(a, [&] { return sparseloco_aggregate(plan, messages, mean, stream); });
    });
}

PyObject* outer_update(PyObject*, PyObject* const* args, Py_ssize_t n) {
    return guarded(args, n, [](Args a) {
        const auto* plan = a.handle<sparseloco_plan>();
        const auto *theta = a.handle<sparseloco_tensors>(), *mean = a.handle<sparseloco_tensors>();
        const float lr = a.number();
        void* stream = a.stream();
        return finish(a, [&] { return sparseloco_outer_update(plan, theta, mean, lr, stream); });
    });
}

PyObject* aggregate_update(PyObject*, PyObject* const* args, Py_ssize_t n) {
    return guarded(args, n, [](Args a) {
        const auto* plan = a.handle<sparseloco_plan>();
        const auto* messages = a.handle<sparseloco_messages>();
        const auto* theta = a.handle<sparseloco_tensors>();
        const float lr = a.number();
        const auto *mean = a.handle<sparseloco_tensors>(), *reset = a.handle<sparseloco_tensors>();
        void* stream = a.stream();
        return finish(a, [&] { return sparseloco_aggregate_update(plan, messages, theta, lr, mean, reset, stream); });
    });
}

PyObject* outer_step_batch(PyObject*, PyObject* const* args, Py_ssize_t n) {
    return guarded(args, n, [](Args a) {
        const auto* plan = a.handle<sparseloco_plan>();
        const int replicas = a.integer();
        const auto *theta = a.handle<sparseloco_tensors>(), *local = a.handle<sparseloco_tensors>(),
                   *ef = a.handle<sparseloco_tensors>();
        const float beta = a.number(), lr = a.number();
        const auto* messages = a.handle<sparseloco_messages>();
        const auto* mean = a.handle<sparseloco_tensors>();
        const int reset = a.integer();
        void* stream = a.stream();
        return finish(a, [&] {
            return sparseloco_outer_step_batch(plan, replicas, theta, local, ef, beta, lr, messages, mean, reset, stream);
        });
    });
}

// t_perp and token_ids, pos_embed: a matrix of `width` columns each, or None.
struct Tables {
    const float *t_perp = nullptr, *pos = nullptr;
    const int32_t* ids = nullptr;
    int64_t vocab = 0, seq = 0;
};
Tables tables(Args& a, int64_t rows, int64_t width) {
    Tables t;
    int64_t vocab = -1, seq = -1;
    if (a.none()) {
        if (!a.none()) a.ok = false;                          // (token ids without a table)
    } else {
        t.t_perp = a.matrix(vocab, width);
        const at::Tensor* ids = a.tensor(at::kInt);
        if (!ids || ids->dim() != 1 || ids->size(0) != rows) a.ok = false;
        else t.ids = static_cast<const int32_t*>(ids->data_ptr());
        t.vocab = vocab;
    }
    if (!a.none()) {
        t.pos = a.matrix(seq, width);
        t.seq = seq;
    }
    if (t.vocab > INT_MAX || t.seq > INT_MAX) a.ok = false;
    return t;
}

template <bool PROJECT>
PyObject* boundary(PyObject*, PyObject* const* args, Py_ssize_t n) {
    return guarded(args, n, [](Args a) {
        int64_t rows = -1, d = -1, k = -1;
        // in, u, out
        const float* in = PROJECT ? a.matrix(rows, d) : a.matrix(rows, k);
        const float* u = a.matrix(d, k);
        float* out = PROJECT ? a.matrix(rows, k) : a.matrix(rows, d);
        const Tables t = tables(a, rows, d);
        const int matmul = a.integer();
        void* stream = a.stream();
        if (d > INT_MAX || k > INT_MAX) a.ok = false;
        return finish(a, [&] {
            return (PROJECT ? sparseloco_subspace_project : sparseloco_subspace_reconstruct)(
                in, t.t_perp, t.ids, (int)t.vocab, t.pos, (int)t.seq, u, out, rows, (int)d, (int)k, matmul, stream);
        });
    });
}

PyObject* reproject(PyObject*, PyObject* const* args, Py_ssize_t n) {
    return guarded(args, n, [](Args a) {
        int64_t vocab = -1, d = -1, k = -1;
        float *t_s = a.matrix(vocab, d), *t_perp = a.matrix(vocab, d);
        const float* u = a.matrix(d, k);
        const at::Tensor* ws = a.tensor(at::kFloat);
        if (!ws || ws->numel() < vocab * k) a.ok = false;
        float* coeff = a.ok ? static_cast<float*>(ws->data_ptr()) : nullptr;
        const int matmul = a.integer();
        void* stream = a.stream();
        if (d > INT_MAX || k > INT_MAX) a.ok = false;
        return finish(a, [&] {
            return sparseloco_reproject_embedding(t_s, t_perp, u, coeff, vocab, (int)d, (int)k, matmul, stream);
        });
    });
}

using Fast = PyObject* (*)(PyObject*, PyObject* const*, Py_ssize_t);
PyCFunction method(Fast f) { return reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)); }

}  // namespace

PyMODINIT_FUNC PyInit__calls() {
    static PyMethodDef methods[] = {
        {"compress", method(compress), METH_FASTCALL, nullptr},
        {"aggregate", method(aggregate), METH_FASTCALL, nullptr},
        {"outer_update", method(outer_update), METH_FASTCALL, nullptr},
        {"aggregate_update", method(aggregate_update), METH_FASTCALL, nullptr},
        {"outer_step_batch", method(outer_step_batch), METH_FASTCALL, nullptr},
        {"project", method(boundary<true>), METH_FASTCALL, nullptr},
        {"reconstruct", method(boundary<false>), METH_FASTCALL, nullptr},
        {"reproject", method(reproject), METH_FASTCALL, nullptr},
        {nullptr, nullptr, 0, nullptr}};
    static PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};
    return PyModule_Create(&module);
}
