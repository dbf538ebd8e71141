// marshal.cpp -- the binding's per-call work in native code: tensors' shapes,
// types and placement checked, their pointers taken, and the C entry point
// called.  A call of the attention's smaller kernels lasts 4 to 6 us
// on the GPU; marshalling it through Python and ctypes takes 10, here 3.
//
// Each function takes the entry point's address and the Python function's
// arguments, and returns its status, or None for a call that it does not take:
// anything but plain strided GPU tensors of the expected shapes and types.  The
// Python function then goes its own way, which raises the error (or takes what
// is left, tensor subclasses for one).  No tensor, pointer or result is kept
// between calls.
#include <torch/csrc/autograd/python_variable.h>

#include <climits>
#include <initializer_list>

namespace {

// torch's functions for the current device, and for a device's current stream
PyObject* current_device = nullptr;
PyObject* current_stream = nullptr;

struct Args {
    PyObject* const* v;
    Py_ssize_t n;
    bool ok = true;
    void* fn() { return PyLong_AsVoidPtr(v[0]); }
    // tensor i, or null and ok = false
    const at::Tensor* tensor(Py_ssize_t i) {
        if (!ok || i >= n || !THPVariable_CheckExact(v[i])) return fail();
        const at::Tensor& t = THPVariable_Unpack(v[i]);
        if (!t.defined() || !t.has_storage() || t.layout() != c10::kStrided || !t.is_cuda() || !t.is_contiguous())
            return fail();
        return &t;
    }
    const at::Tensor* tensor(Py_ssize_t i, at::IntArrayRef shape, c10::ScalarType type) {
        const at::Tensor* t = tensor(i);
        if (t && (t->sizes() != shape || t->scalar_type() != type)) return fail();
        return t;
    }
    // a tensor or None (then null, with ok as it was)
    const at::Tensor* maybe(Py_ssize_t i, at::IntArrayRef shape, c10::ScalarType type) {
        return ok && i < n && v[i] == Py_None ? nullptr : tensor(i, shape, type);
    }
    long long integer(Py_ssize_t i) {
        if (!ok || i >= n || !PyLong_CheckExact(v[i])) return fail(), 0;
        int over = 0;
        const long long r = PyLong_AsLongLongAndOverflow(v[i], &over);
        if (over || r < INT_MIN || r > INT_MAX) fail();
        return r;
    }
    float real(Py_ssize_t i) {
        if (!ok || i >= n || !PyFloat_CheckExact(v[i])) return fail(), 0.0f;
        return (float)PyFloat_AS_DOUBLE(v[i]);
    }
    // the stream argument: None for the current stream of the current device
    void* stream(Py_ssize_t i) {
        if (!ok || i >= n) return fail();
        PyObject* h = nullptr;
        if (v[i] != Py_None) {
            h = PyObject_GetAttrString(v[i], "cuda_stream");
        } else if (PyObject* dev = current_device ? PyObject_CallNoArgs(current_device) : nullptr) {
            h = PyObject_CallOneArg(current_stream, dev);
            Py_DECREF(dev);
        }
        void* s = h && PyLong_Check(h) ? PyLong_AsVoidPtr(h) : fail();
        Py_XDECREF(h);
        if (PyErr_Occurred()) fail();
        return s;
    }
    std::nullptr_t fail() {
        ok = false;
        return nullptr;
    }
};

// the C ABI's element types; -1 for another
int type_code(const at::Tensor& t) {
    switch (t.scalar_type()) {
        case c10::kHalf: return 0;
        case c10::kBFloat16: return 1;
        case c10::kFloat: return 2;
        default: return -1;
    }
}
void* ptr(const at::Tensor* t) { return t ? t->data_ptr() : nullptr; }
bool fits(std::initializer_list<int64_t> sizes) {
    for (int64_t s : sizes)
        if (s > INT_MAX) return false;
    return true;
}

// Call the entry point without the interpreter lock, as ctypes does.
template <typename... A>
PyObject* call(void* fn, A... a) {
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = reinterpret_cast<int (*)(A...)>(fn)(a...);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

// A C++ exception (a tensor without storage, a device without a runtime) leaves
// the call to the Python function.
template <PyObject* (*F)(Args&)>
PyObject* entry(PyObject*, PyObject* const* v, Py_ssize_t n) {
    try {
        Args a{v, n};
        PyObject* r = n > 0 ? F(a) : nullptr;
        if (r) return r;
    } catch (...) {
    }
    if (PyErr_Occurred()) PyErr_Clear();
    Py_RETURN_NONE;
}

// fn, q, k, v, out, scale, stream
PyObject* forward(Args& a) {
    const at::Tensor* q = a.tensor(1);
    const at::Tensor* k = a.tensor(2);
    if (!q || !k || q->dim() != 4 || k->dim() != 4 || q->scalar_type() != c10::kHalf) return nullptr;
    const int64_t B = q->size(0), H = q->size(1), Lq = q->size(2), D = q->size(3), Lk = k->size(2);
    const int64_t kv[] = {B, H, Lk, D};
    a.tensor(2, kv, c10::kHalf);
    const at::Tensor *v = a.tensor(3, kv, c10::kHalf), *out = a.tensor(4, q->sizes(), c10::kHalf);
    const float scale = a.real(5);
    void* s = a.stream(6);
    if (!a.ok || !fits({B, H, Lq, Lk, D})) return nullptr;
    return call(a.fn(), ptr(q), ptr(k), ptr(v), ptr(out), (int)B, (int)H, (int)Lq, (int)Lk, (int)D, scale, s);
}

// fn, q, k, v, out, ls, scale, stream
PyObject* forward_ex(Args& a) {
    const at::Tensor* q = a.tensor(1);
    if (!q || q->dim() != 4) return nullptr;
    const auto type = q->scalar_type();
    const int64_t B = q->size(0), H = q->size(1), Lq = q->size(2), D = q->size(3);
    const at::Tensor* k = a.tensor(2);
    if (!k || k->dim() != 4) return nullptr;
    const int64_t Lk = k->size(2);
    const int64_t kv[] = {B, H, Lk, D}, st[] = {B, H, Lq, 2};
    a.tensor(2, kv, type);
    const at::Tensor* v = a.tensor(3, kv, type);
    const at::Tensor* out = a.tensor(4, q->sizes(), type);
    const at::Tensor* ls = a.maybe(5, st, c10::kFloat);
    const float scale = a.real(6);
    void* s = a.stream(7);
    const int code = type_code(*q);
    if (!a.ok || code < 0 || !fits({B, H, Lq, Lk, D})) return nullptr;
    return call(a.fn(), ptr(q), ptr(k), ptr(v), ptr(out), ptr(ls), (int)B, (int)H, (int)Lq, (int)Lk, (int)D, scale, code, s);
}

// fn, a, ls, p, scale, stream
PyObject* softmax_rows(Args& a) {
    const at::Tensor* x = a.tensor(1);
    if (!x || x->dim() != 2) return nullptr;
    const at::Tensor* ls = a.tensor(2);
    const at::Tensor* p = a.maybe(3, x->sizes(), x->scalar_type());
    const float scale = a.real(4);
    void* s = a.stream(5);
    const int code = type_code(*x);
    if (!a.ok || code < 0 || ls->scalar_type() != c10::kFloat || ls->numel() != 2 * x->size(0)) return nullptr;
    return call(a.fn(), ptr(x), ptr(ls), ptr(p), (long long)x->size(0), (long long)x->size(1), scale, code, s);
}

// fn, q, k, a, scale, stream
PyObject* logits(Args& a) {
    const at::Tensor* q = a.tensor(1);
    const at::Tensor* k = a.tensor(2);
    if (!q || !k || q->dim() != 4 || k->dim() != 4) return nullptr;
    const int64_t B = q->size(0), H = q->size(1), Lq = q->size(2), D = q->size(3), Lk = k->size(2);
    const int64_t ks[] = {B, H, Lk, D}, as[] = {B, H, Lq, Lk};
    a.tensor(2, ks, q->scalar_type());
    const at::Tensor* x = a.tensor(3);
    const float scale = a.real(4);
    void* s = a.stream(5);
    if (!a.ok || x->sizes() != at::IntArrayRef(as) || !fits({B, H, Lq, Lk, D})) return nullptr;
    const int code = type_code(*q), acode = type_code(*x);
    if (code < 0 || acode < 0) return nullptr;
    return call(a.fn(), ptr(q), ptr(k), ptr(x), (int)B, (int)H, (int)Lq, (int)Lk, (int)D, scale, code, acode, s);
}

// fn, a, ls, v, out, stream
PyObject* softmax_pv(Args& a) {
    const at::Tensor* x = a.tensor(1);
    const at::Tensor* ls = a.tensor(2);
    const at::Tensor* v = a.tensor(3);
    if (!x || !ls || !v || x->dim() != 4 || v->dim() != 4) return nullptr;
    const int64_t B = x->size(0), H = x->size(1), Lq = x->size(2), Lk = x->size(3), D = v->size(3);
    const int64_t vs[] = {B, H, Lk, D}, os[] = {B, H, Lq, D};
    a.tensor(3, vs, v->scalar_type());
    const at::Tensor* out = a.tensor(4, os, v->scalar_type());
    void* s = a.stream(5);
    const int code = type_code(*v), acode = type_code(*x);
    if (!a.ok || code < 0 || acode < 0 || ls->scalar_type() != c10::kFloat || ls->numel() != 2 * B * H * Lq ||
        !fits({B, H, Lq, Lk, D}))
        return nullptr;
    return call(a.fn(), ptr(x), ptr(ls), ptr(v), ptr(out), (int)B, (int)H, (int)Lq, (int)Lk, (int)D, acode, code, s);
}

// fn, x, ctx, wq, wk, wv, wo, bo, out, workspace, heads, scale, stream
PyObject* attention_block(Args& a) {
    const at::Tensor* x = a.tensor(1);
    const at::Tensor* ctx = a.tensor(2);
    if (!x || !ctx || x->dim() != 3 || ctx->dim() != 3) return nullptr;
    const auto type = x->scalar_type();
    const int64_t B = x->size(0), Lq = x->size(1), C = x->size(2), Lk = ctx->size(1), Cc = ctx->size(2);
    const int64_t cs[] = {B, Lk, Cc}, cc[] = {C, C}, ccc[] = {C, Cc}, c1[] = {C};
    a.tensor(2, cs, type);
    const at::Tensor *wq = a.tensor(3, cc, type), *wk = a.tensor(4, ccc, type), *wv = a.tensor(5, ccc, type),
                     *wo = a.tensor(6, cc, type), *bo = a.maybe(7, c1, type), *out = a.tensor(8, x->sizes(), type),
                     *ws = a.tensor(9);
    const int heads = (int)a.integer(10);
    const float scale = a.real(11);
    void* s = a.stream(12);
    const int code = type_code(*x);
    if (!a.ok || code < 0 || !fits({B, Lq, Lk, C, Cc})) return nullptr;
    return call(a.fn(), ptr(x), ptr(ctx), ptr(wq), ptr(wk), ptr(wv), ptr(wo), ptr(bo), ptr(out), ptr(ws),
                (long long)(ws->numel() * ws->element_size()), (int)B, (int)Lq, (int)Lk, (int)C, (int)Cc, heads, scale,
                code, s);
}

// fn, x, wq, k, v, wo, bo, out, workspace, scale, stream
PyObject* attention_block_kv(Args& a) {
    const at::Tensor* x = a.tensor(1);
    const at::Tensor* k = a.tensor(3);
    if (!x || !k || x->dim() != 3 || k->dim() != 4) return nullptr;
    const auto type = x->scalar_type();
    const int64_t B = x->size(0), Lq = x->size(1), C = x->size(2), H = k->size(1), Lk = k->size(2);
    if (H < 1) return nullptr;
    const int64_t ks[] = {B, H, Lk, C / H}, cc[] = {C, C}, c1[] = {C};
    a.tensor(3, ks, type);
    const at::Tensor *wq = a.tensor(2, cc, type), *v = a.tensor(4, ks, type), *wo = a.tensor(5, cc, type),
                     *bo = a.maybe(6, c1, type), *out = a.tensor(7, x->sizes(), type), *ws = a.tensor(8);
    const float scale = a.real(9);
    void* s = a.stream(10);
    const int code = type_code(*x);
    if (!a.ok || code < 0 || !fits({B, Lq, Lk, C, H})) return nullptr;
    return call(a.fn(), ptr(x), ptr(wq), ptr(k), ptr(v), ptr(wo), ptr(bo), ptr(out), ptr(ws),
                (long long)(ws->numel() * ws->element_size()), (int)B, (int)Lq, (int)Lk, (int)C, (int)H, scale, code, s);
}

// fn, x, groups, y, gamma, beta, eps, stream
PyObject* group_norm(Args& a) {
    const at::Tensor* x = a.tensor(1);
    if (!x || x->dim() < 2) return nullptr;
    const auto type = x->scalar_type();
    const int64_t B = x->size(0), C = x->size(1), c1[] = {C};
    int64_t HW = 1;
    for (int64_t i = 2; i < x->dim(); ++i) HW *= x->size(i);
    const int groups = (int)a.integer(2);
    const at::Tensor *y = a.tensor(3, x->sizes(), type), *gamma = a.maybe(4, c1, type), *beta = a.maybe(5, c1, type);
    const float eps = a.real(6);
    void* s = a.stream(7);
    const int code = type_code(*x);
    if (!a.ok || code < 0 || !fits({B, C})) return nullptr;
    return call(a.fn(), ptr(x), ptr(gamma), ptr(beta), ptr(y), (int)B, (int)C, (long long)HW, groups, eps, code, s);
}

// fn, h, out, stream
PyObject* geglu(Args& a) {
    const at::Tensor* h = a.tensor(1);
    if (!h || h->dim() < 1 || h->numel() == 0) return nullptr;
    const int64_t F2 = h->size(-1);
    if (F2 % 2) return nullptr;
    const at::Tensor* out = a.tensor(2);
    void* s = a.stream(3);
    const int code = type_code(*h);
    if (!a.ok || code < 0 || out->scalar_type() != h->scalar_type() || out->dim() != h->dim() ||
        out->sizes().slice(0, out->dim() - 1) != h->sizes().slice(0, h->dim() - 1) || out->size(-1) != F2 / 2 ||
        !fits({F2 / 2}))
        return nullptr;
    return call(a.fn(), ptr(h), ptr(out), (long long)(h->numel() / F2), (int)(F2 / 2), code, s);
}

// fn, x, u, y, workspace, bias, stream
PyObject* conv3x3(Args& a) {
    const at::Tensor* x = a.tensor(1);
    const at::Tensor* u = a.tensor(2);
    if (!x || !u || x->dim() != 4 || u->dim() != 3) return nullptr;
    const auto type = x->scalar_type();
    const int64_t B = x->size(0), Ci = x->size(1), H = x->size(2), W = x->size(3), Co = u->size(1);
    const int64_t us[] = {36, Co, Ci}, ys[] = {B, Co, H, W}, c1[] = {Co};
    a.tensor(2, us, type);
    const at::Tensor *y = a.tensor(3, ys, type), *ws = a.tensor(4), *bias = a.maybe(5, c1, type);
    void* s = a.stream(6);
    const int code = type_code(*x);
    if (!a.ok || code < 0 || !fits({B, Ci, Co, H, W})) return nullptr;
    return call(a.fn(), ptr(x), ptr(u), ptr(bias), ptr(y), ptr(ws), (long long)(ws->numel() * ws->element_size()),
                (int)B, (int)Ci, (int)Co, (int)H, (int)W, code, s);
}

PyObject* use_streams(PyObject*, PyObject* const* v, Py_ssize_t n) {
    if (n == 2) {
        Py_INCREF(v[0]);
        Py_INCREF(v[1]);
        current_device = v[0];
        current_stream = v[1];
    }
    Py_RETURN_NONE;
}

#define FAST(f) {#f, (PyCFunction)(void (*)(void))entry<f>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {{"use_streams", (PyCFunction)(void (*)(void))use_streams, METH_FASTCALL, nullptr},
                         FAST(forward), FAST(forward_ex), FAST(softmax_rows), FAST(logits), FAST(softmax_pv), FAST(attention_block),
                         FAST(attention_block_kv), FAST(group_norm), FAST(geglu), FAST(conv3x3),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

extern "C" __attribute__((visibility("default"))) PyObject* PyInit__marshal(void) { return PyModule_Create(&module); }
