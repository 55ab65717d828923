// The common calls of binding.py in native code: checks, output tensors and the library call without a Python object for
// each step.  Every function here takes what its namesake in binding.py takes, outputs as None where they are to be
// allocated, and returns
//   a tuple   the outputs, as the Python code returns them;
//   an int    the status of a call that the library refused;
//   None      where anything is out of the ordinary -- another type than a plain tensor, number or bool, a layout or
//             dtype that the Python code refuses or treats apart, a torch function or dispatch mode, an allocation that
//             failed: binding.py then takes its own way, and reports what it finds.
// An exception raised in Python code that runs inside (a Python allocator, say) is passed on as it is.
// The library's functions come in as addresses (bind), so there is one copy of it in the process.  The GIL is released
// around the library call, as ctypes does.
// Host time of a call, us, ctypes and torch.empty / so: fa_fwd 8.9 / 5.9, fa_bwd 12.1 / 7.6,
// fa_fp8_quant_hadamard 8.4 / 5.6, fa_fwd_fp8 9.2 / 6.1 (the launch itself is 2.4 to 3 of it).
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/fa_mi355.h"

namespace {

struct {
    decltype(&fa_fwd_gqa) fwd;
    decltype(&fa_fwd_fp8_gqa) fwd_fp8;
    decltype(&fa_fp8_quant_hadamard) quant;
    decltype(&fa_bwd_workspace_bytes) workspace_bytes;
    decltype(&fa_bwd_gqa) bwd;
} lib;

// The arguments of a call; `ok` turns false at the first that is not as the native way takes it.
struct Arguments {
    PyObject* const* args;
    Py_ssize_t n;
    bool ok = true;

    Arguments(PyObject* const* a, Py_ssize_t count, Py_ssize_t expected) : args(a), n(count), ok(count == expected) {
        if (lib.fwd == nullptr || at::impl::torch_function_mode_enabled() || c10::impl::TorchDispatchModeTLS::any_modes_set())
            ok = false;
    }
    bool given(Py_ssize_t i) const { return ok && args[i] != Py_None; }
    // a plain contiguous device tensor
    const at::Tensor* tensor(Py_ssize_t i) {
        if (!ok || !THPVariable_CheckExact(args[i])) return fail();
        const at::Tensor& t = THPVariable_Unpack(args[i]);
        if (!t.defined() || !t.is_cuda() || !t.is_contiguous()) return fail();
        return &t;
    }
    double number(Py_ssize_t i) {
        if (ok && PyFloat_CheckExact(args[i])) return PyFloat_AS_DOUBLE(args[i]);
        ok = false;
        return 0.0;
    }
    int flag(Py_ssize_t i) {
        if (ok && PyLong_Check(args[i])) return PyObject_IsTrue(args[i]);  // a bool or an int
        ok = false;
        return 0;
    }
    // What the function args[i] says is the current stream, asked when everything else is in order.  Its failure is a case for
    // the Python code, which asks again; what is no Exception (an interrupt from the keyboard comes only once) stays set.
    void* stream(Py_ssize_t i) {
        if (!ok) return nullptr;
        PyObject* handle = PyObject_CallNoArgs(args[i]);
        void* p = handle ? PyLong_AsVoidPtr(handle) : nullptr;
        Py_XDECREF(handle);
        if (PyErr_Occurred()) {
            if (PyErr_ExceptionMatches(PyExc_Exception)) PyErr_Clear();
            ok = false;
        }
        return p;
    }

private:
    std::nullptr_t fail() {
        ok = false;
        return nullptr;
    }
};

struct Shape {
    int B, H, N, d;
};
// [B, H, N, d] of a 4-dimensional tensor
bool shape_of(const at::Tensor& t, Shape& s) {
    if (t.dim() != 4) return false;
    const auto sizes = t.sizes();
    for (int64_t x : sizes)
        if (x > 0x7fffffff) return false;
    s = {(int)sizes[0], (int)sizes[1], (int)sizes[2], (int)sizes[3]};
    return true;
}
bool dtype_code(const at::Tensor& t, int& code) {
    switch (t.scalar_type()) {
        case at::kFloat: code = FA_F32; return true;
        case at::kBFloat16: code = FA_BF16; return true;
        case at::kHalf: code = FA_F16; return true;
        default: return false;
    }
}

// The given output tensor, or a new one of these sizes on the device of `like`
at::Tensor output(Arguments& a, Py_ssize_t i, at::IntArrayRef sizes, const at::Tensor& like, at::ScalarType type) {
    if (a.given(i)) {
        const at::Tensor* t = a.tensor(i);
        return t ? *t : at::Tensor();
    }
    return a.ok ? at::empty(sizes, like.options().dtype(type)) : at::Tensor();
}
// ... with the strides of `like`
at::Tensor gradient(Arguments& a, Py_ssize_t i, const at::Tensor& like) {
    if (a.given(i)) {
        const at::Tensor* t = a.tensor(i);
        return t ? *t : at::Tensor();
    }
    return a.ok ? at::empty_strided(like.sizes(), like.strides(), like.options()) : at::Tensor();
}

template <typename Call>
int without_gil(Call&& call) {
    PyThreadState* state = PyEval_SaveThread();
    const int status = call();
    PyEval_RestoreThread(state);
    return status;
}

// A tuple of the tensors, given ones as the objects they came as, or the status
template <size_t K>
PyObject* result(int status, const Arguments& a, const Py_ssize_t (&index)[K], const at::Tensor (&tensors)[K]) {
    if (status != FA_OK) return PyLong_FromLong(status);
    PyObject* out = PyTuple_New(K);
    if (!out) return nullptr;
    for (size_t i = 0; i < K; ++i) {
        PyObject* t = a.given(index[i]) ? Py_NewRef(a.args[index[i]]) : THPVariable_Wrap(tensors[i]);
        if (!t) {
            Py_DECREF(out);
            return nullptr;
        }
        PyTuple_SET_ITEM(out, i, t);
    }
    return out;
}

// Runs `body`; an exception is a case for the Python code, but for one that Python has set already
template <typename Body>
PyObject* native(Body&& body) {
    try {
        PyObject* r = body();
        if (r) return r;
    } catch (...) {
    }
    if (PyErr_Occurred()) return nullptr;
    Py_RETURN_NONE;
}

// (q, k, v, scale, causal, o, lse, shared, stream)
PyObject* fwd(PyObject*, PyObject* const* args, Py_ssize_t n) {
    return native([&]() -> PyObject* {
        Arguments a(args, n, 9);
        const at::Tensor *q = a.tensor(0), *k = a.tensor(1), *v = a.tensor(2);
        const double scale = a.number(3);
        const int causal = a.flag(4), shared = a.flag(7);
        void* stream = a.stream(8);
        Shape s;
        int code;
        if (!a.ok || !shape_of(*q, s) || !dtype_code(*q, code) || (shared && k->dim() < 2)) return nullptr;
        const int64_t kv_heads = shared ? k->size(1) : s.H;
        if (kv_heads > 0x7fffffff) return nullptr;
        const at::Tensor o = output(a, 5, q->sizes(), *q, q->scalar_type());
        const at::Tensor lse = output(a, 6, {s.B, s.H, s.N}, *q, at::kFloat);
        if (!a.ok) return nullptr;
        const void *qp = q->data_ptr(), *kp = k->data_ptr(), *vp = v->data_ptr();
        void* op = o.data_ptr();
        float* lp = static_cast<float*>(lse.data_ptr());
        const int st = without_gil([&] {
            return lib.fwd(qp, kp, vp, op, lp, s.B, s.H, (int)kv_heads, s.N, s.d, (float)scale, causal, code, stream);
        });
        return result(st, a, {5, 6}, {o, lse});
    });
}

// (q8, k8, v8, q_scale, k_scale, v_scale, scale, causal, o, lse, shared, stream), blocks of 128 rows
PyObject* fwd_fp8(PyObject*, PyObject* const* args, Py_ssize_t n) {
    return native([&]() -> PyObject* {
        Arguments a(args, n, 12);
        const at::Tensor *q = a.tensor(0), *k = a.tensor(1), *v = a.tensor(2);
        const at::Tensor *qs = a.tensor(3), *ks = a.tensor(4), *vs = a.tensor(5);
        const double scale = a.number(6);
        const int causal = a.flag(7), shared = a.flag(10);
        void* stream = a.stream(11);
        Shape s;
        if (!a.ok || !shape_of(*q, s) || (shared && k->dim() < 2)) return nullptr;
        const int64_t kv_heads = shared ? k->size(1) : s.H;
        if (kv_heads > 0x7fffffff) return nullptr;
        const at::Tensor o = output(a, 8, q->sizes(), *q, at::kBFloat16);
        const at::Tensor lse = output(a, 9, {s.B, s.H, s.N}, *q, at::kFloat);
        if (!a.ok) return nullptr;
        const void *qp = q->data_ptr(), *kp = k->data_ptr(), *vp = v->data_ptr();
        const float *qsp = static_cast<const float*>(qs->data_ptr()), *ksp = static_cast<const float*>(ks->data_ptr()),
                    *vsp = static_cast<const float*>(vs->data_ptr());
        void* op = o.data_ptr();
        float* lp = static_cast<float*>(lse.data_ptr());
        const int st = without_gil([&] {
            return lib.fwd_fp8(qp, kp, vp, qsp, ksp, vsp, op, lp, s.B, s.H, (int)kv_heads, s.N, s.d, 128, (float)scale, causal,
                               stream);
        });
        return result(st, a, {8, 9}, {o, lse});
    });
}

// (x, signs, per_tensor, x8, scales, stream), blocks of 128 rows
PyObject* quant(PyObject*, PyObject* const* args, Py_ssize_t n) {
    return native([&]() -> PyObject* {
        Arguments a(args, n, 6);
        const at::Tensor* x = a.tensor(0);
        const at::Tensor* signs = a.given(1) ? a.tensor(1) : nullptr;
        const int per_tensor = a.flag(2);
        void* stream = a.stream(5);
        Shape s;
        int code;
        if (!a.ok || !shape_of(*x, s) || !dtype_code(*x, code)) return nullptr;
        const at::Tensor x8 = output(a, 3, x->sizes(), *x, at::kByte);
        const at::Tensor scales = output(a, 4, {s.B, s.H, (s.N + 127L) / 128}, *x, at::kFloat);
        if (!a.ok) return nullptr;
        const void* xp = x->data_ptr();
        const signed char* sp = signs ? static_cast<const signed char*>(signs->data_ptr()) : nullptr;
        void* cp = x8.data_ptr();
        float* scp = static_cast<float*>(scales.data_ptr());
        const int st =
            without_gil([&] { return lib.quant(xp, code, cp, scp, s.B, s.H, s.N, s.d, 128, sp, per_tensor, stream); });
        return result(st, a, {3, 4}, {x8, scales});
    });
}

// (q, k, v, o, lse, dout, scale, causal, dq, dk, dv, workspace, shared, stream)
PyObject* bwd(PyObject*, PyObject* const* args, Py_ssize_t n) {
    return native([&]() -> PyObject* {
        Arguments a(args, n, 14);
        const at::Tensor *q = a.tensor(0), *k = a.tensor(1), *v = a.tensor(2), *o = a.tensor(3), *lse = a.tensor(4);
        const at::Tensor* dout = a.tensor(5);
        const double scale = a.number(6);
        const int causal = a.flag(7), shared = a.flag(12);
        void* stream = a.stream(13);
        Shape s;
        int code;
        if (!a.ok || !shape_of(*q, s) || !dtype_code(*q, code) || (shared && k->dim() < 2)) return nullptr;
        const int64_t kv_heads = shared ? k->size(1) : s.H;
        if (kv_heads > 0x7fffffff) return nullptr;
        at::Tensor workspace;
        if (a.given(11)) {
            const at::Tensor* t = a.tensor(11);
            if (!t) return nullptr;
            workspace = *t;
        } else {
            const int64_t need = (int64_t)lib.workspace_bytes(s.B, s.H, s.N, s.d, code);
            workspace = at::empty({need > 16 ? need : 16}, q->options().dtype(at::kByte));
        }
        const at::Tensor dq = gradient(a, 8, *q), dk = gradient(a, 9, *k), dv = gradient(a, 10, *v);
        if (!a.ok) return nullptr;
        const void *qp = q->data_ptr(), *kp = k->data_ptr(), *vp = v->data_ptr(), *op = o->data_ptr(), *dop = dout->data_ptr();
        const float* lp = static_cast<const float*>(lse->data_ptr());
        void *dqp = dq.data_ptr(), *dkp = dk.data_ptr(), *dvp = dv.data_ptr(), *wp = workspace.data_ptr();
        const size_t bytes = (size_t)workspace.numel();
        const int st = without_gil([&] {
            return lib.bwd(qp, kp, vp, op, lp, dop, dqp, dkp, dvp, wp, bytes, s.B, s.H, (int)kv_heads, s.N, s.d, (float)scale, causal,
                           code, stream);
        });
        return result(st, a, {8, 9, 10}, {dq, dk, dv});
    });
}

// bind(address of fa_fwd_gqa, fa_fwd_fp8_gqa, fa_fp8_quant_hadamard, fa_bwd_workspace_bytes, fa_bwd_gqa)
PyObject* bind(PyObject*, PyObject* const* args, Py_ssize_t n) {
    void* p[5];
    if (n != 5) {
        PyErr_SetString(PyExc_TypeError, "bind takes five addresses");
        return nullptr;
    }
    for (int i = 0; i < 5; ++i) {
        p[i] = PyLong_AsVoidPtr(args[i]);
        if (PyErr_Occurred()) return nullptr;
    }
    lib.fwd = reinterpret_cast<decltype(lib.fwd)>(p[0]);
    lib.fwd_fp8 = reinterpret_cast<decltype(lib.fwd_fp8)>(p[1]);
    lib.quant = reinterpret_cast<decltype(lib.quant)>(p[2]);
    lib.workspace_bytes = reinterpret_cast<decltype(lib.workspace_bytes)>(p[3]);
    lib.bwd = reinterpret_cast<decltype(lib.bwd)>(p[4]);
    Py_RETURN_NONE;
}

#define FA_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FA_METHOD(bind), FA_METHOD(fwd), FA_METHOD(fwd_fp8), FA_METHOD(quant), FA_METHOD(bwd), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fa_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

// Whether the torch of this process is the one that this file was compiled against; if not, ImportError is set
bool same_torch() {
    PyObject* torch = PyImport_ImportModule("torch");
    PyObject* version = torch ? PyObject_GetAttrString(torch, "__version__") : nullptr;
    PyObject* text = version ? PyObject_Str(version) : nullptr;
    const bool same = text && PyUnicode_CompareWithASCIIString(text, FA_TORCH_VERSION) == 0;
    if (text && !same) PyErr_Format(PyExc_ImportError, "built for torch " FA_TORCH_VERSION ", not for %U", text);
    Py_XDECREF(text);
    Py_XDECREF(version);
    Py_XDECREF(torch);
    return same;
}

}  // namespace

PyMODINIT_FUNC PyInit__fa_binding() { return same_torch() ? PyModule_Create(&module) : nullptr; }
