// The Python binding's argument handling in native code: checks tensors, allocates what the
// caller did not bring, and calls the C ABI (include/esc_convattn.h).  binding.py keeps the
// signatures and hands its arguments on by position.
//
// Why native: a forward of a small feature map lasts 9 us on the GPU, and a Python and ctypes
// call in front of it took 11.5 us (tensor attributes one by one, fifteen ctypes conversions,
// the stream and allocator asked for through Python), so that the host set the pace.  No
// torch type crosses the C ABI; this module is the only translation unit that knows both.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/core/LegacyTypeDispatch.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <string>
#include <vector>

#include "esc_convattn.h"

namespace {

// A Python exception is already set (or the C++ one below describes it).
struct PyError {};

[[noreturn]] void fail(PyObject *type, const std::string &msg)
{
    PyErr_SetString(type, msg.c_str());
    throw PyError{};
}

[[noreturn]] void fail_status(int st)
{
    PyObject *mod = PyImport_ImportModule("paper_2503_06671_amd.binding");
    PyObject *cls = mod != nullptr ? PyObject_GetAttrString(mod, "EscError") : nullptr;
    PyObject *exc = cls != nullptr ? PyObject_CallFunction(cls, "is", st, esc_status_string((esc_status)st)) : nullptr;
    if (exc != nullptr) PyErr_SetObject(cls, exc);
    Py_XDECREF(exc);
    Py_XDECREF(cls);
    Py_XDECREF(mod);
    throw PyError{};
}

void check(esc_status st)
{
    if (st != ESC_OK) fail_status((int)st);
}

bool given(PyObject *o) { return o != nullptr && o != Py_None; }

const at::Tensor &tensor(PyObject *o, const char *name)
{
    if (!THPVariable_Check(o)) fail(PyExc_TypeError, std::string(name) + " must be a tensor");
    return THPVariable_Unpack(o);
}

// whatever int() takes, as the callers may pass numpy integers or floats
long whole_number(PyObject *o)
{
    const long v = PyLong_AsLong(o);
    if (v != -1 || !PyErr_Occurred()) return v;
    PyErr_Clear();
    PyObject *i = PyNumber_Long(o);
    if (i == nullptr) throw PyError{};
    const long w = PyLong_AsLong(i);
    Py_DECREF(i);
    if (w == -1 && PyErr_Occurred()) throw PyError{};
    return w;
}

int integer(PyObject *o)
{
    const long v = whole_number(o);
    if (v != (long)(int)v) fail(PyExc_OverflowError, "integer argument out of range");
    return (int)v;
}

// An optional contiguous fp32 device tensor: nullptr when None.
const at::Tensor *dev_f32(PyObject *o, const char *name)
{
    if (!given(o)) return nullptr;
    if (THPVariable_Check(o)) {
        const at::Tensor &t = THPVariable_Unpack(o);
        if (t.is_cuda() && t.scalar_type() == at::kFloat && t.is_contiguous()) return &t;
    }
    fail(PyExc_TypeError, std::string(name) + " must be a contiguous float32 device tensor");
}

const at::Tensor &dev_f32_required(PyObject *o, const char *name)
{
    const at::Tensor *t = dev_f32(o, name);
    if (t == nullptr) fail(PyExc_TypeError, std::string(name) + " must be a contiguous float32 device tensor");
    return *t;
}

const float *ptr(const at::Tensor *t) { return t != nullptr ? static_cast<const float *>(t->data_ptr()) : nullptr; }

struct Shape {
    esc_dtype dt;
    int N, C, H, W;
};

Shape x_checked(const at::Tensor &x)
{
    if (!x.is_cuda() || x.dim() != 4 || !x.is_contiguous()) fail(PyExc_TypeError, "x must be a contiguous [N,C,H,W] device tensor");
    Shape s;
    if (x.scalar_type() == at::kFloat) s.dt = ESC_F32;
    else if (x.scalar_type() == at::kBFloat16) s.dt = ESC_BF16;
    else fail(PyExc_TypeError, std::string("x must be float32 or bfloat16, got ") + c10::toString(x.scalar_type()));
    int *const d[4] = {&s.N, &s.C, &s.H, &s.W};
    for (int i = 0; i < 4; ++i) {
        const int64_t v = x.size(i);
        if (v != (int64_t)(int)v) fail(PyExc_ValueError, "x is too large");
        *d[i] = (int)v;
    }
    return s;
}

bool like(const at::Tensor &t, const at::Tensor &x)
{
    return t.scalar_type() == x.scalar_type() && t.sizes() == x.sizes() && t.is_contiguous();
}

at::Tensor out_or_new(PyObject *o, const at::Tensor &x, const char *what = "out must match x in dtype and shape and be contiguous")
{
    if (!given(o)) return at::empty(x.sizes(), x.options());
    const at::Tensor &t = tensor(o, "out");
    if (!like(t, x)) fail(PyExc_TypeError, what);
    return t;
}

// The stream to enqueue on: the caller's (an object with `cuda_stream`), or the current one of the current device.
void *stream_of(PyObject *o)
{
    if (!given(o)) return c10::hip::getCurrentHIPStream().stream();
    static PyObject *const attr = PyUnicode_InternFromString("cuda_stream");
    PyObject *h = PyObject_GetAttr(o, attr);
    if (h == nullptr) throw PyError{};
    void *p = PyLong_AsVoidPtr(h);
    Py_DECREF(h);
    if (p == nullptr && PyErr_Occurred()) throw PyError{};
    return p;
}

struct Ws {
    void *ptr;
    size_t bytes;
};

Ws workspace(PyObject *o)
{
    const at::Tensor &t = tensor(o, "workspace");
    return Ws{t.data_ptr(), (size_t)t.numel() * (size_t)t.element_size()};
}

// ---- the estimator's weights: a capsule made once per binding.GenParams ----
struct Gen {
    esc_gen_params p;
    int64_t n_w_down, n_b_down, n_w_up, n_b_up;  // elements, -1 where there is no tensor
    std::vector<int64_t> sizes[4];               // in that order
};
constexpr const char *kGenCapsule = "esc_gen";

const Gen *gen_of(PyObject *o, int Ca)
{
    if (!given(o)) return nullptr;
    static PyObject *const attr = PyUnicode_InternFromString("handle");
    PyObject *h = PyObject_GetAttr(o, attr);
    if (h == nullptr) throw PyError{};
    const Gen *g = static_cast<const Gen *>(PyCapsule_GetPointer(h, kGenCapsule));
    Py_DECREF(h);  // (the GenParams object, which the caller holds, keeps it)
    if (g == nullptr) throw PyError{};
    // the library reads these buffers by the sizes C_a and hidden imply: refuse others
    const int64_t hidden = g->p.hidden, K = hidden > 0 ? hidden : Ca;
    auto want = [&](const char *name, int64_t has, int64_t need) {
        if (has >= 0 && has != need)
            fail(PyExc_ValueError, std::string(name) + " has " + std::to_string(has) + " elements, C_a = " + std::to_string(Ca) +
                                       " and hidden = " + std::to_string(hidden) + " need " + std::to_string(need));
    };
    if (hidden > 0 && g->n_w_down < 0) fail(PyExc_ValueError, "hidden > 0 needs w_down");
    want("w_up", g->n_w_up, 9 * (int64_t)Ca * K);
    want("b_up", g->n_b_up, 9 * (int64_t)Ca);
    if (hidden > 0) {
        want("w_down", g->n_w_down, hidden * Ca);
        want("b_down", g->n_b_down, hidden);
    }
    return g;
}

// ---- the large kernel: [Ca,Ks,Ks] (one filter per channel), [Ks,Ks] (one for all), or a flat
// buffer read with an explicit Ks and channel stride ----
struct Lk {
    const float *ptr;
    int Ks;
    long stride;
};

Lk lk_checked(PyObject *o, int Ca, PyObject *ks = nullptr, PyObject *stride = nullptr)
{
    const at::Tensor &t = dev_f32_required(o, "lk");
    const float *p = ptr(&t);
    if (given(ks) || given(stride)) {
        if (!given(ks) || !given(stride)) fail(PyExc_ValueError, "give ks and lk_channel_stride together");
        const int k = integer(ks);
        const long st = whole_number(stride);
        // (128 bits: the product of any two such numbers, which must not wrap round to a small one)
        const __int128 need = ((st != 0 && Ca > 0) ? (__int128)(Ca - 1) * st : 0) + (__int128)k * k;
        if (t.numel() < need)
            fail(PyExc_ValueError, "lk holds " + std::to_string(t.numel()) + " values, Ks = " + std::to_string(k) +
                                       " with channel stride " + std::to_string(st) + " reads more");
        return Lk{p, k, st};
    }
    if (t.dim() == 2 && t.size(0) == t.size(1)) return Lk{p, (int)t.size(0), 0};
    if (t.dim() == 3 && t.size(1) == t.size(2) && (t.size(0) == Ca || Ca == 0))
        return Lk{p, (int)t.size(1), (long)(t.size(1) * t.size(2))};
    std::string shape;
    for (int64_t i = 0; i < t.dim(); ++i) shape += (i > 0 ? ", " : "") + std::to_string(t.size(i));
    fail(PyExc_ValueError, "lk must be [Ca,Ks,Ks] with Ca = " + std::to_string(Ca) + ", or [Ks,Ks]; got (" + shape + ")");
}

const at::Tensor *dk_checked(PyObject *o, const Shape &s, int Ca)
{
    const at::Tensor *t = dev_f32(o, "dk_in");
    if (t != nullptr && t->numel() != (int64_t)s.N * Ca * 9) fail(PyExc_ValueError, "dk_in must hold [N, Ca, 3, 3] values");
    return t;
}

PyObject *wrap(const at::Tensor &t) { return THPVariable_Wrap(t); }

// The buffer the caller gave as `out`, or the new tensor.
PyObject *result(PyObject *given_out, const at::Tensor &t)
{
    if (given(given_out)) {
        Py_INCREF(given_out);
        return given_out;
    }
    return wrap(t);
}

void want_args(Py_ssize_t n, Py_ssize_t want)
{
    if (n != want) fail(PyExc_TypeError, "expected " + std::to_string(want) + " arguments, got " + std::to_string(n));
}

// Runs a C ABI call without the interpreter's lock.
template <typename F>
esc_status unlocked(F &&f)
{
    PyThreadState *ts = PyEval_SaveThread();
    const esc_status st = f();
    PyEval_RestoreThread(ts);
    return st;
}

// ---- ConvFFN's weights ----
struct Ffn {
    int Ch;
    const float *w1, *b1, *k, *bk, *w2, *b2;
};

Ffn ffn_checked(int C, PyObject *w1o, PyObject *ko, PyObject *w2o, PyObject *b1o, PyObject *bko, PyObject *b2o)
{
    const at::Tensor &w1 = dev_f32_required(w1o, "w1"), &k = dev_f32_required(ko, "k_dw"), &w2 = dev_f32_required(w2o, "w2");
    const at::Tensor *b1 = dev_f32(b1o, "b1"), *bk = dev_f32(bko, "b_dw"), *b2 = dev_f32(b2o, "b2");
    if (w1.dim() != 2 || w1.size(1) != C)
        fail(PyExc_ValueError, "w1 must be [Ch, C] with C = " + std::to_string(C));
    const int64_t Ch = w1.size(0);
    if (k.dim() != 3 || k.size(0) != Ch || k.size(1) != 3 || k.size(2) != 3 || w2.dim() != 2 || w2.size(0) != C || w2.size(1) != Ch)
        fail(PyExc_ValueError, "k_dw must be [Ch, 3, 3] and w2 [C, Ch]");
    if ((b1 != nullptr && b1->numel() != Ch) || (bk != nullptr && bk->numel() != Ch) || (b2 != nullptr && b2->numel() != C))
        fail(PyExc_ValueError, "b1 and b_dw must hold Ch values, b2 C values");
    return Ffn{(int)Ch, ptr(&w1), ptr(b1), ptr(&k), ptr(bk), ptr(&w2), ptr(b2)};
}

// ---- entry points (positional arguments, in binding.py's order) ----

PyObject *gen_handle(PyObject *const *a, Py_ssize_t n)
{
    want_args(n, 5);  // hidden, w_down, b_down, w_up, b_up
    const at::Tensor *t[4];
    const char *const names[4] = {"w_down", "b_down", "w_up", "b_up"};
    for (int i = 0; i < 4; ++i) t[i] = dev_f32(a[1 + i], names[i]);
    auto count = [](const at::Tensor *p) { return p != nullptr ? p->numel() : (int64_t)-1; };
    Gen *g = new Gen{{integer(a[0]), ptr(t[0]), ptr(t[1]), ptr(t[2]), ptr(t[3])}, count(t[0]), count(t[1]), count(t[2]), count(t[3]), {}};
    for (int i = 0; i < 4; ++i)
        if (t[i] != nullptr) g->sizes[i] = t[i]->sizes().vec();
    PyObject *cap = PyCapsule_New(g, kGenCapsule, [](PyObject *c) { delete static_cast<Gen *>(PyCapsule_GetPointer(c, kGenCapsule)); });
    if (cap == nullptr) {
        delete g;
        throw PyError{};
    }
    return cap;
}

PyObject *dynkernel_gen(PyObject *const *a, Py_ssize_t n)
{
    want_args(n, 6);  // x, Ca, gen, workspace, dk_out, stream
    const at::Tensor &x = tensor(a[0], "x");
    const Shape s = x_checked(x);
    const int Ca = integer(a[1]);
    const Gen *g = gen_of(a[2], Ca);
    const Ws ws = workspace(a[3]);
    at::Tensor dk = given(a[4]) ? dev_f32_required(a[4], "dk_out") : at::empty({s.N, Ca, 3, 3}, x.options().dtype(at::kFloat));
    if (dk.numel() != (int64_t)s.N * Ca * 9) fail(PyExc_ValueError, "dk_out must hold [N, Ca, 3, 3] values");
    void *st = stream_of(a[5]);
    float *dkp = static_cast<float *>(dk.data_ptr());
    const void *xp = x.data_ptr();
    check(unlocked([&] { return esc_dynkernel_gen(xp, s.dt, s.N, s.C, s.H, s.W, Ca, g != nullptr ? &g->p : nullptr, dkp, ws.ptr, ws.bytes, st); }));
    return result(a[4], dk);
}

PyObject *convattn_forward(PyObject *const *a, Py_ssize_t n)
{
    want_args(n, 10);  // x, Ca, lk, workspace, gen, dk_in, out, stream, ks, lk_channel_stride
    const at::Tensor &x = tensor(a[0], "x");
    const Shape s = x_checked(x);
    const int Ca = integer(a[1]);
    const Lk lk = lk_checked(a[2], Ca, a[8], a[9]);
    const Gen *g = gen_of(a[4], Ca);
    const at::Tensor out = out_or_new(a[6], x);
    const float *dk = ptr(dk_checked(a[5], s, Ca));
    void *st = stream_of(a[7]);
    const esc_gen_params *gp = g != nullptr ? &g->p : nullptr;
    const void *xp = x.data_ptr();
    void *op = out.data_ptr();
    if (!given(a[3])) {  // the entry point that allocates nothing: the library's own scratch
        check(unlocked([&] { return esc_convattn_forward_noalloc(xp, s.dt, s.N, s.C, s.H, s.W, Ca, lk.ptr, lk.Ks, lk.stride, gp, dk, op, st); }));
    } else {
        const Ws ws = workspace(a[3]);
        check(unlocked([&] {
            return esc_convattn_forward(xp, s.dt, s.N, s.C, s.H, s.W, Ca, lk.ptr, lk.Ks, lk.stride, gp, dk, op, ws.ptr, ws.bytes, st);
        }));
    }
    return result(a[6], out);
}

// Conv_fuse's and LK^c's weights, for the fused call and the residual step
struct Fuse {
    const float *w, *b, *lkc;
};

Fuse fuse_checked(int C, int Ca, PyObject *w, PyObject *b, PyObject *lkc)
{
    const at::Tensor &wf = dev_f32_required(w, "w_fuse");
    const at::Tensor *bf = dev_f32(b, "b_fuse"), *lc = dev_f32(lkc, "lk_c");
    if (wf.numel() != (int64_t)C * C || (bf != nullptr && bf->numel() != C)) fail(PyExc_ValueError, "w_fuse must be [C, C] and b_fuse [C]");
    if (lc != nullptr && lc->numel() != (int64_t)Ca * Ca) fail(PyExc_ValueError, "lk_c must be [Ca, Ca]");
    return Fuse{ptr(&wf), ptr(bf), ptr(lc)};
}

PyObject *convattn_fused_forward(PyObject *const *a, Py_ssize_t n)
{
    want_args(n, 12);  // x, Ca, lk, w_fuse, workspace, b_fuse, lk_c, residual, gen, dk_in, out, stream
    const at::Tensor &x = tensor(a[0], "x");
    const Shape s = x_checked(x);
    const int Ca = integer(a[1]);
    const Lk lk = lk_checked(a[2], Ca);
    const Gen *g = gen_of(a[8], Ca);
    const Fuse f = fuse_checked(s.C, Ca, a[3], a[5], a[6]);
    const float *dk = ptr(dk_checked(a[9], s, Ca));
    const void *res = nullptr;
    if (given(a[7])) {
        const at::Tensor &r = tensor(a[7], "residual");
        if (!like(r, x) || !r.is_cuda())
            fail(PyExc_TypeError, "residual must match x in dtype and shape and be a contiguous device tensor");
        res = r.data_ptr();
    }
    const at::Tensor out = out_or_new(a[10], x);
    const Ws ws = workspace(a[4]);
    void *st = stream_of(a[11]);
    const void *xp = x.data_ptr();
    void *op = out.data_ptr();
    check(unlocked([&] {
        return esc_convattn_fused_forward(xp, s.dt, s.N, s.C, s.H, s.W, Ca, f.lkc, lk.ptr, lk.Ks, lk.stride, g != nullptr ? &g->p : nullptr,
                                          dk, f.w, f.b, res, op, ws.ptr, ws.bytes, st);
    }));
    return result(a[10], out);
}

PyObject *convffn_forward(PyObject *const *a, Py_ssize_t n)
{
    want_args(n, 10);  // x, w1, k_dw, w2, workspace, b1, b_dw, b2, out, stream
    const at::Tensor &x = tensor(a[0], "x");
    const Shape s = x_checked(x);
    const Ffn f = ffn_checked(s.C, a[1], a[2], a[3], a[5], a[6], a[7]);
    const at::Tensor out = out_or_new(a[8], x);
    const Ws ws = workspace(a[4]);
    void *st = stream_of(a[9]);
    const void *xp = x.data_ptr();
    void *op = out.data_ptr();
    check(unlocked([&] {
        return esc_convffn_forward(xp, s.dt, s.N, s.C, s.H, s.W, f.Ch, f.w1, f.b1, f.k, f.bk, f.w2, f.b2, op, ws.ptr, ws.bytes, st);
    }));
    return result(a[8], out);
}

PyObject *residual_step_forward(PyObject *const *a, Py_ssize_t n)
{
    // f_in, w1, k_dw, w2, Ca, lk, w_fuse, workspace, b1, b_dw, b2, lk_c, gen, b_fuse, out, stream
    want_args(n, 16);
    const at::Tensor &x = tensor(a[0], "x");
    const Shape s = x_checked(x);
    const Ffn f = ffn_checked(s.C, a[1], a[2], a[3], a[8], a[9], a[10]);
    const int Ca = integer(a[4]);
    const Lk lk = lk_checked(a[5], Ca);
    const Gen *g = gen_of(a[12], Ca);
    const Fuse fu = fuse_checked(s.C, Ca, a[6], a[13], a[11]);
    const at::Tensor out = out_or_new(a[14], x, "out must match f_in in dtype and shape and be contiguous");
    const Ws ws = workspace(a[7]);
    void *st = stream_of(a[15]);
    const void *xp = x.data_ptr();
    void *op = out.data_ptr();
    check(unlocked([&] {
        return esc_residual_step_forward(xp, s.dt, s.N, s.C, s.H, s.W, f.Ch, f.w1, f.b1, f.k, f.bk, f.w2, f.b2, Ca, fu.lkc, lk.ptr, lk.Ks,
                                         lk.stride, g != nullptr ? &g->p : nullptr, fu.w, fu.b, op, ws.ptr, ws.bytes, st);
    }));
    return result(a[14], out);
}

PyObject *convattn_dense_forward(PyObject *const *a, Py_ssize_t n)
{
    want_args(n, 8);  // x, Ca, lk_dense, workspace, gen, dk_in, out, stream
    const at::Tensor &x = tensor(a[0], "x");
    const Shape s = x_checked(x);
    const int Ca = integer(a[1]);
    const at::Tensor &lk = dev_f32_required(a[2], "lk_dense");
    if (lk.dim() != 4 || lk.size(0) != Ca || lk.size(1) != Ca || lk.size(2) != lk.size(3))
        fail(PyExc_ValueError, "lk_dense must be [Ca, Ca, Ks, Ks] with Ca = " + std::to_string(Ca));
    const int Ks = (int)lk.size(2);
    const Gen *g = gen_of(a[4], Ca);
    const float *dk = ptr(dk_checked(a[5], s, Ca));
    const at::Tensor out = out_or_new(a[6], x);
    const Ws ws = workspace(a[3]);
    void *st = stream_of(a[7]);
    const float *lp = ptr(&lk);
    const void *xp = x.data_ptr();
    void *op = out.data_ptr();
    check(unlocked([&] {
        return esc_convattn_dense_forward(xp, s.dt, s.N, s.C, s.H, s.W, Ca, lp, Ks, g != nullptr ? &g->p : nullptr, dk, op, ws.ptr, ws.bytes, st);
    }));
    return result(a[6], out);
}

// A dict's value by name (borrowed), or nullptr where there is none.
PyObject *item(PyObject *d, const char *key)
{
    PyObject *v = PyDict_GetItemString(d, key);
    return given(v) ? v : nullptr;
}

PyObject *convattn_backward(PyObject *const *a, Py_ssize_t n)
{
    want_args(n, 10);  // x, grad_out, Ca, lk, workspace, gen, dk_in, accumulate, grads, stream
    const at::Tensor &x = tensor(a[0], "x");
    const Shape s = x_checked(x);
    const at::Tensor &go = tensor(a[1], "grad_out");
    if (!like(go, x) || !go.is_cuda()) fail(PyExc_TypeError, "grad_out must match x in dtype and shape and be a contiguous device tensor");
    const int Ca = integer(a[2]);
    const Lk lk = lk_checked(a[3], Ca);
    const at::Tensor &lk_t = THPVariable_Unpack(a[3]);
    const Gen *g = gen_of(a[5], Ca);
    const float *dk = ptr(dk_checked(a[6], s, Ca));
    const int acc = PyObject_IsTrue(a[7]);
    if (acc < 0) throw PyError{};
    struct Dict {
        PyObject *d;
        ~Dict() { Py_XDECREF(d); }
    } grads{nullptr};
    const int brought_any = given(a[8]) ? PyObject_IsTrue(a[8]) : 0;
    if (brought_any < 0) throw PyError{};
    // (whatever dict() takes: a mapping, or pairs)
    grads.d = brought_any != 0 ? PyObject_CallFunctionObjArgs((PyObject *)&PyDict_Type, a[8], nullptr) : PyDict_New();
    if (grads.d == nullptr) throw PyError{};
    // Buffers the caller did not bring.  A call writes every element of the parameter gradients, so
    // they need no zeros first - unless it adds to them, or has no attention channels to write any.
    const bool zero = acc != 0 || Ca == 0;
    const auto f32 = x.options().dtype(at::kFloat);
    auto need = [&](const char *name, at::IntArrayRef sizes, bool zeroed) -> float * {
        PyObject *v = item(grads.d, name);
        if (v != nullptr) return static_cast<float *>(dev_f32_required(v, name).data_ptr());
        const at::Tensor t = zeroed ? at::zeros(sizes, f32) : at::empty(sizes, f32);
        PyObject *o = wrap(t);
        const int rc = o != nullptr ? PyDict_SetItemString(grads.d, name, o) : -1;
        Py_XDECREF(o);
        if (rc != 0) throw PyError{};
        return static_cast<float *>(t.data_ptr());
    };
    void *gxp;
    if (PyObject *v = item(grads.d, "grad_x")) {
        const at::Tensor &t = tensor(v, "grad_x");
        // (a buffer to write into, as a pool of bytes may hold it: its own type and shape are the caller's business)
        if (!t.is_cuda() || t.nbytes() < x.nbytes() || !t.is_contiguous())
            fail(PyExc_TypeError, "grad_x must be a contiguous device tensor with room for x's gradient");
        gxp = t.data_ptr();
    } else {
        const at::Tensor t = at::empty(x.sizes(), x.options());
        PyObject *o = wrap(t);
        const int rc = o != nullptr ? PyDict_SetItemString(grads.d, "grad_x", o) : -1;
        Py_XDECREF(o);
        if (rc != 0) throw PyError{};
        gxp = t.data_ptr();
    }
    float *glk = need("grad_lk", lk_t.sizes(), zero);
    float *gdk = need("grad_dk", {s.N, Ca, 3, 3}, false);
    esc_gen_grads gg{};
    if (g != nullptr) {
        auto brought = [&](const char *name) -> float * {  // (the gradient of a bias that is not there)
            PyObject *v = item(grads.d, name);
            return v != nullptr ? static_cast<float *>(dev_f32_required(v, name).data_ptr()) : nullptr;
        };
        // (shaped like the weights; an estimator without w_up is the library's to refuse, but has no shape to allocate)
        if (g->n_w_up < 0 && item(grads.d, "grad_w_up") == nullptr) fail(PyExc_TypeError, "the estimator needs w_up");
        gg.w_up = need("grad_w_up", g->sizes[2], zero);
        gg.b_up = g->n_b_up >= 0 ? need("grad_b_up", g->sizes[3], zero) : brought("grad_b_up");
        if (g->p.hidden > 0) {
            gg.w_down = need("grad_w_down", g->sizes[0], zero);
            gg.b_down = g->n_b_down >= 0 ? need("grad_b_down", g->sizes[1], zero) : brought("grad_b_down");
        }
    }
    // every other buffer the caller put into the dict is held to the same rule
    PyObject *key, *val;
    for (Py_ssize_t pos = 0; PyDict_Next(grads.d, &pos, &key, &val);)
        if (PyUnicode_Check(key) && PyUnicode_CompareWithASCIIString(key, "grad_x") != 0) {
            const char *name = PyUnicode_AsUTF8(key);
            if (name == nullptr) throw PyError{};
            dev_f32(val, name);
        }
    const Ws ws = workspace(a[4]);
    void *st = stream_of(a[9]);
    const void *xp = x.data_ptr(), *gop = go.data_ptr();
    check(unlocked([&] {
        return esc_convattn_backward(xp, gop, s.dt, s.N, s.C, s.H, s.W, Ca, lk.ptr, lk.Ks, lk.stride, g != nullptr ? &g->p : nullptr, dk, gxp,
                                     glk, g != nullptr ? &gg : nullptr, gdk, acc, ws.ptr, ws.bytes, st);
    }));
    PyObject *r = grads.d;
    grads.d = nullptr;
    return r;
}

// Runs an entry point and turns what it throws into the Python exception.
template <PyObject *(*F)(PyObject *const *, Py_ssize_t)>
PyObject *entry(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    try {
        at::AutoDispatchBelowADInplaceOrView below;  // buffers are allocated without a look at autograd
        return F(args, n);
    } catch (const PyError &) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, "esc_native: unknown error");
    } catch (const c10::OutOfMemoryError &e) {
        PyObject *mod = PyImport_ImportModule("torch");
        PyObject *cls = mod != nullptr ? PyObject_GetAttrString(mod, "OutOfMemoryError") : nullptr;
        PyErr_SetString(cls != nullptr ? cls : PyExc_MemoryError, e.what_without_backtrace());
        Py_XDECREF(cls);
        Py_XDECREF(mod);
    } catch (const c10::Error &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what_without_backtrace());
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
    }
    return nullptr;
}

#define ESC_ENTRY(name) {#name, (PyCFunction)(void (*)(void))entry<name>, METH_FASTCALL, nullptr}
PyMethodDef kMethods[] = {ESC_ENTRY(gen_handle),         ESC_ENTRY(dynkernel_gen),    ESC_ENTRY(convattn_forward),
                          ESC_ENTRY(convattn_fused_forward), ESC_ENTRY(convffn_forward), ESC_ENTRY(residual_step_forward),
                          ESC_ENTRY(convattn_dense_forward), ESC_ENTRY(convattn_backward), {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_native", "Argument handling of the binding over the C ABI.", -1, kMethods,
                       nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() { return PyModule_Create(&kModule); }
