// Argument marshalling of the hot calls for the Python binding (dfa.py), as a
// CPython extension: it checks the tensors, reads B, H, L, d from their shapes
// and calls the library's C functions, whose addresses dfa.py hands over.  A
// call whose arguments are anything but ordinary (another tensor class, type,
// layout, shape or device, an integer out of range, any exception) is not
// made: the function returns -1 and dfa.py takes its general path, which
// raises the error or handles the case.
//
// Why: in Python the checks and the ctypes conversion of a plan step cost 6.5
// to 7 us a call, as long as the kernels of short sequences run.
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>

#include <climits>
#include <cstdint>

namespace {

typedef void* stream_t;   // a hipStream_t, passed through
typedef int (*attn_fn)(const void*, const void*, const void*, void*, void*, int, int, int, int, int, stream_t);
typedef int (*plan_fn)(int, const void*, const void*, const void*, void*, void*, void*, int, int, int, int, int, stream_t);
typedef int (*qkv_fn)(const void*, const void*, const void*, void*, void*, void*, int, int, int, int, stream_t);
typedef int (*out_fn)(const void*, const void*, const void*, void*, int, int, int, int, stream_t);
typedef int (*module_fn)(int, const void*, const void*, const void*, const void*, const void*, void*, void*, void*, void*,
                         void*, void*, void*, int, int, int, int, int, stream_t);
typedef int (*mrae_fn)(const void*, const void*, size_t, void*, double*, stream_t);

struct Functions {
    attn_fn attn[3];      // full, full_and_residual, window_plus_residual
    plan_fn plan;
    qkv_fn qkv;
    out_fn out;
    module_fn module;
    mrae_fn mrae;
    PyObject* device;       // torch's current device, and
    PyObject* raw_stream;   // its current stream of a device, as integers
};

Functions g_functions;

constexpr auto BF16 = at::kBFloat16;
constexpr auto F32 = at::kFloat;

// Reads one call's arguments; `ok` turns false at the first that is not
// ordinary (declining is no error, so nothing is thrown for it).
struct Reader {
    bool ok = true;

    const at::Tensor* tensor(PyObject* o) {
        if (ok && THPVariable_CheckExact(o)) return &THPVariable_Unpack(o);
        ok = false;
        return nullptr;
    }
    // address of a contiguous GPU tensor of this type and shape (None: null)
    void* address(PyObject* o, at::ScalarType type, at::IntArrayRef shape) {
        if (!ok || o == Py_None) return nullptr;
        const at::Tensor* t = tensor(o);
        if (!t) return nullptr;
        ok = t->is_cuda() && t->scalar_type() == type && t->sizes() == shape && t->is_contiguous();
        return ok ? t->data_ptr() : nullptr;
    }
    // the same, where None is not ordinary
    void* required(PyObject* o, at::ScalarType type, at::IntArrayRef shape) {
        ok = ok && o != Py_None;
        return address(o, type, shape);
    }
    int integer(PyObject* o) {
        ok = ok && PyLong_Check(o);
        if (!ok) return 0;
        int overflow = 0;
        const long v = PyLong_AsLongAndOverflow(o, &overflow);
        ok = !overflow && v >= INT_MIN && v <= INT_MAX;
        return ok ? (int)v : 0;
    }
    // a plan code may be any integer type (an element of a numpy plan)
    int plan_code(PyObject* o) {
        if (!ok) return 0;
        PyObject* i = PyNumber_Index(o);
        if (!i) {
            PyErr_Clear();
            ok = false;
            return 0;
        }
        const int v = integer(i);
        Py_DECREF(i);
        return v;
    }
    int dim(int64_t v) {
        ok = ok && v >= 0 && v <= INT_MAX;
        return ok ? (int)v : 0;
    }
    // torch's current stream on the current device
    stream_t stream(const Functions& f) {
        if (!ok) return nullptr;
        PyObject* dev = PyObject_CallNoArgs(f.device);
        PyObject* s = dev ? PyObject_CallOneArg(f.raw_stream, dev) : nullptr;
        Py_XDECREF(dev);
        void* p = s ? PyLong_AsVoidPtr(s) : nullptr;
        Py_XDECREF(s);
        if (PyErr_Occurred()) {
            PyErr_Clear();
            ok = false;
        }
        return p;
    }
};

// B, H, L, d of a [B][H][L][d] tensor.
struct Heads {
    at::IntArrayRef shape;
    int B = 0, H = 0, L = 0, d = 0;
    Heads(Reader& r, PyObject* o) {
        const at::Tensor* t = r.tensor(o);
        if (t) shape = t->sizes();
        r.ok = r.ok && shape.size() == 4;
        if (!r.ok) return;
        B = r.dim(shape[0]);
        H = r.dim(shape[1]);
        L = r.dim(shape[2]);
        d = r.dim(shape[3]);
    }
};

// Runs `read`, which returns the library's status or leaves its Reader not ok,
// and returns the status as a Python integer, -1 for a declined call.  A tensor
// without storage throws from data_ptr().
template <class F>
PyObject* guarded(F&& read) {
    Reader r;
    int status = -1;
    try {
        status = read(r, g_functions);
    } catch (...) {
        r.ok = false;
    }
    return PyLong_FromLong(r.ok ? status : -1);
}

template <class F>
int call(const Reader& r, F&& f) {
    if (!r.ok) return -1;
    PyThreadState* st = PyEval_SaveThread();
    const int status = f();   // a C function: no exceptions
    PyEval_RestoreThread(st);
    return status;
}

// attn(which, Q, K, V, O, R, w)
PyObject* py_attn(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&](Reader& r, const Functions& f) -> int {
        r.ok = n == 7;
        if (!r.ok) return -1;
        const int which = r.integer(a[0]), w = r.integer(a[6]);
        r.ok = r.ok && which >= 0 && which <= 2;
        const Heads s(r, a[1]);
        void *Q = r.address(a[1], BF16, s.shape), *K = r.address(a[2], BF16, s.shape), *V = r.address(a[3], BF16, s.shape),
             *O = r.address(a[4], BF16, s.shape), *R = r.address(a[5], F32, s.shape);
        const stream_t st = r.stream(f);
        return call(r, [&] { return f.attn[which](Q, K, V, O, R, s.B, s.H, s.L, s.d, w, st); });
    });
}

// plan_step(code, Q, K, V, O, R, Ocache, w)
PyObject* py_plan(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&](Reader& r, const Functions& f) -> int {
        r.ok = n == 8;
        if (!r.ok) return -1;
        const int code = r.plan_code(a[0]), w = r.integer(a[7]);
        const Heads s(r, a[4]);
        void *Q = r.address(a[1], BF16, s.shape), *K = r.address(a[2], BF16, s.shape), *V = r.address(a[3], BF16, s.shape),
             *O = r.address(a[4], BF16, s.shape), *R = r.address(a[5], F32, s.shape), *C = r.address(a[6], BF16, s.shape);
        const stream_t st = r.stream(f);
        return call(r, [&] { return f.plan(code, Q, K, V, O, R, C, s.B, s.H, s.L, s.d, w, st); });
    });
}

// qkv_proj(X, Wqkv, bqkv, Q, K, V)
PyObject* py_qkv(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&](Reader& r, const Functions& f) -> int {
        r.ok = n == 6;
        if (!r.ok) return -1;
        const Heads s(r, a[3]);
        const int64_t C = (int64_t)s.H * s.d, tokens[3] = {s.B, s.L, C}, w[2] = {3 * C, C}, b[1] = {3 * C};
        void *X = r.required(a[0], BF16, tokens), *W = r.address(a[1], BF16, w), *bias = r.address(a[2], F32, b),
             *Q = r.required(a[3], BF16, s.shape), *K = r.required(a[4], BF16, s.shape), *V = r.required(a[5], BF16, s.shape);
        const stream_t st = r.stream(f);
        return call(r, [&] { return f.qkv(X, W, bias, Q, K, V, s.B, s.H, s.L, s.d, st); });
    });
}

// out_proj(O, Wo, bo, Y)
PyObject* py_out(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&](Reader& r, const Functions& f) -> int {
        r.ok = n == 4;
        if (!r.ok) return -1;
        const Heads s(r, a[0]);
        const int64_t C = (int64_t)s.H * s.d, tokens[3] = {s.B, s.L, C}, w[2] = {C, C}, b[1] = {C};
        void *O = r.required(a[0], BF16, s.shape), *W = r.address(a[1], BF16, w), *bias = r.address(a[2], F32, b),
             *Y = r.required(a[3], BF16, tokens);
        const stream_t st = r.stream(f);
        return call(r, [&] { return f.out(O, W, bias, Y, s.B, s.H, s.L, s.d, st); });
    });
}

// module_step(code, X, Wqkv, bqkv, Wo, bo, Q, K, V, O, R, Y, Ycache, w, H)
PyObject* py_module(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&](Reader& r, const Functions& f) -> int {
        r.ok = n == 15;
        if (!r.ok) return -1;
        const int code = r.plan_code(a[0]), w = r.integer(a[13]), H = r.integer(a[14]);
        const at::Tensor* y = r.tensor(a[11]);
        r.ok = r.ok && H > 0 && y->sizes().size() == 3 && y->sizes()[2] % H == 0;
        if (!r.ok) return -1;
        const at::IntArrayRef tokens = y->sizes();
        const int B = r.dim(tokens[0]), L = r.dim(tokens[1]), C = r.dim(tokens[2]), d = C / H;
        const int64_t C3 = 3 * (int64_t)C, heads[4] = {B, H, L, d}, wq[2] = {C3, C}, bq[1] = {C3}, wo[2] = {C, C}, bo[1] = {C};
        void *X = r.address(a[1], BF16, tokens), *Wq = r.address(a[2], BF16, wq), *bqkv = r.address(a[3], F32, bq),
             *Wo = r.address(a[4], BF16, wo), *bout = r.address(a[5], F32, bo), *Q = r.address(a[6], BF16, heads),
             *K = r.address(a[7], BF16, heads), *V = r.address(a[8], BF16, heads), *O = r.address(a[9], BF16, heads),
             *R = r.address(a[10], F32, heads), *Y = r.required(a[11], BF16, tokens), *Yc = r.address(a[12], BF16, tokens);
        const stream_t st = r.stream(f);
        return call(r, [&] { return f.module(code, X, Wq, bqkv, Wo, bout, Q, K, V, O, R, Y, Yc, B, H, L, d, w, st); });
    });
}

// mrae(A, B, workspace, result)
PyObject* py_mrae(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&](Reader& r, const Functions& f) -> int {
        r.ok = n == 4;
        if (!r.ok) return -1;
        const at::Tensor *A = r.tensor(a[0]), *B = r.tensor(a[1]), *ws = r.tensor(a[2]), *res = r.tensor(a[3]);
        r.ok = r.ok && A->numel() == B->numel() && ws->numel() * (int64_t)ws->element_size() >= 8192 && res->numel() >= 1;
        if (!r.ok) return -1;
        void *pa = r.address(a[0], BF16, A->sizes()), *pb = r.address(a[1], BF16, B->sizes()),
             *pw = r.address(a[2], ws->scalar_type(), ws->sizes()), *pr = r.address(a[3], at::kDouble, res->sizes());
        const size_t count = (size_t)A->numel();
        const stream_t st = r.stream(f);
        return call(r, [&] { return f.mrae(pa, pb, count, pw, (double*)pr, st); });
    });
}

// init(device, raw_stream, full, full_and_residual, window, plan, qkv, out, module, mrae): the functions' addresses
PyObject* py_init(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 10) {
        PyErr_SetString(PyExc_TypeError, "init takes 10 arguments");
        return nullptr;
    }
    void* p[8];
    for (int i = 0; i < 8; ++i) {
        p[i] = PyLong_AsVoidPtr(a[i + 2]);
        if (!p[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null function address");
            return nullptr;
        }
    }
    for (int i = 0; i < 3; ++i) g_functions.attn[i] = (attn_fn)p[i];
    g_functions.plan = (plan_fn)p[3];
    g_functions.qkv = (qkv_fn)p[4];
    g_functions.out = (out_fn)p[5];
    g_functions.module = (module_fn)p[6];
    g_functions.mrae = (mrae_fn)p[7];
    Py_INCREF(a[0]);
    Py_INCREF(a[1]);
    Py_XDECREF(g_functions.device);
    Py_XDECREF(g_functions.raw_stream);
    g_functions.device = a[0];
    g_functions.raw_stream = a[1];
    Py_RETURN_NONE;
}

#define DFA_METHOD(name, fn) {name, (PyCFunction)(void (*)(void))fn, METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {
    DFA_METHOD("init", py_init), DFA_METHOD("attn", py_attn),     DFA_METHOD("plan_step", py_plan),
    DFA_METHOD("qkv_proj", py_qkv), DFA_METHOD("out_proj", py_out), DFA_METHOD("module_step", py_module),
    DFA_METHOD("mrae", py_mrae), {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_dfa_binding", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__dfa_binding() { return PyModule_Create(&g_module); }
