// The hot calls' argument handling between torch tensors and the C ABI, in native code.
//
// A layer's pair of calls on a few hundred rows keeps the GPU busy for 12-16 us; checking the
// tensors, sizing and allocating the outputs and finding the stream took 23 us per pair as Python
// with ctypes, so the host set the pace of every small layer.  Each function below does one
// call's checks (the same errors with the same texts), allocates what the caller did not pass
// through torch's allocator on the current stream, and enqueues with the interpreter lock
// released (a launch may wait for room in the queue).  It keeps no state between calls.
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "dgq.h"

namespace {

struct Raised {};  // a Python exception is set

PyObject *g_error = nullptr;  // the package's DgqError
PyObject *s_handle = nullptr, *s_out_channels = nullptr, *s_cuda_stream = nullptr;

[[noreturn]] void raise(PyObject *type, const char *text) {
    PyErr_SetString(type, text);
    throw Raised();
}
[[noreturn]] void raise_value(const char *text) { raise(PyExc_ValueError, text); }

const char *dtype_name(at::ScalarType t) {
    switch (t) {
        case at::kFloat: return "torch.float32";
        case at::kChar: return "torch.int8";
        case at::kByte: return "torch.uint8";
        default: return "torch.int32";
    }
}

bool given(PyObject *o) { return o != Py_None; }

const at::Tensor &tensor(PyObject *o, at::ScalarType t, const char *name) {
    if (THPVariable_Check(o)) {
        const at::Tensor &v = THPVariable_Unpack(o);
        if (v.is_cuda() && v.scalar_type() == t && v.is_contiguous()) return v;
    }
    PyErr_Format(PyExc_TypeError, "%s must be a contiguous CUDA tensor of dtype %s", name, dtype_name(t));
    throw Raised();
}

// data pointer of an optional tensor
template <class T>
T *pointer(const at::Tensor &v) { return static_cast<T *>(v.data_ptr()); }

template <class T>
T *optional(PyObject *o, at::ScalarType t, const char *name) {
    return given(o) ? pointer<T>(tensor(o, t, name)) : nullptr;
}

void *handle_of(PyObject *o) {  // None: a handle that was freed (the C call reports the null)
    PyObject *h = PyObject_GetAttr(o, s_handle);
    if (!h) throw Raised();
    void *p = given(h) ? PyLong_AsVoidPtr(h) : nullptr;
    Py_DECREF(h);
    if (!p && PyErr_Occurred()) throw Raised();
    return p;
}
const dgq_groups_t *groups_of(PyObject *o) { return static_cast<const dgq_groups_t *>(handle_of(o)); }
const dgq_weight_t *weight_of(PyObject *o) { return static_cast<const dgq_weight_t *>(handle_of(o)); }

int64_t integer(PyObject *o) {
    const int64_t v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw Raised();
    return v;
}
// sizes of the C ABI are 32 bits wide; what does not fit is reported by the call as an empty tensor
int32_t integer32(PyObject *o) {
    const int64_t v = integer(o);
    return v >= INT32_MIN && v <= INT32_MAX ? (int32_t)v : -1;
}

int64_t out_channels_of(PyObject *weight) {
    PyObject *o = PyObject_GetAttr(weight, s_out_channels);
    if (!o) throw Raised();
    const int64_t v = PyLong_AsLongLong(o);
    Py_DECREF(o);
    if (v == -1 && PyErr_Occurred()) throw Raised();
    return v;
}

void *stream_of(PyObject *o) {
    if (!given(o)) return c10::hip::getCurrentHIPStream().stream();
    PyObject *s = PyObject_GetAttr(o, s_cuda_stream);
    if (!s) throw Raised();
    void *p = PyLong_AsVoidPtr(s);
    Py_DECREF(s);
    if (!p && PyErr_Occurred()) throw Raised();
    return p;
}

at::Tensor empty(at::IntArrayRef sizes, at::ScalarType t, const at::Tensor &like) {
    at::AutoDispatchBelowADInplaceOrView below;  // no gradients here
    return at::empty(sizes, like.options().dtype(t).requires_grad(false));
}

dgq_groups_info_t info_of(const dgq_groups_t *g) {
    dgq_groups_info_t i{};
    if (g) dgq_groups_info(g, &i);
    return i;
}

// Shape of the block-tiled code buffer: [row blocks, chunks, 1024].
struct CodesShape {
    int64_t n[3];
    CodesShape(const dgq_groups_t *g, int64_t rows) {
        const int64_t chunks = info_of(g).k_padded / DGQ_K_GRANULE;
        n[0] = chunks ? (int64_t)dgq_codes_bytes(g, rows) / (chunks * 1024) : 0;
        n[1] = chunks;
        n[2] = 1024;
    }
    at::IntArrayRef sizes() const { return at::IntArrayRef(n, 3); }
    bool is(const at::Tensor &t) const { return t.sizes() == sizes(); }
};

bool shape_is(const at::Tensor &t, std::initializer_list<int64_t> s) {
    return t.sizes() == at::IntArrayRef(s.begin(), s.size());
}

// The C ABI sees no sizes: a tensor it would read or write past the end of is refused here.
void holds(const at::Tensor &t, int64_t n, const char *name) {
    if (t.numel() >= n) return;
    PyErr_Format(PyExc_ValueError, "%s has %lld elements, the call needs %lld", name, (long long)t.numel(), (long long)n);
    throw Raised();
}
void holds_if_given(PyObject *o, int64_t n, const char *name) {
    if (given(o)) holds(THPVariable_Unpack(o), n, name);
}

template <class F>
void enqueue(F &&call) {
    int rc;
    Py_BEGIN_ALLOW_THREADS;
    rc = call();
    Py_END_ALLOW_THREADS;
    if (rc == 0) return;
    if (PyObject *e = PyObject_CallFunction(g_error, "is", rc, dgq_last_error())) {
        PyErr_SetObject(g_error, e);
        Py_DECREF(e);
    }
    throw Raised();
}

PyObject *wrap(const at::Tensor &t) {
    PyObject *o = THPVariable_Wrap(t);
    if (!o) throw Raised();
    return o;
}
// (the caller's object where one was passed, else the new tensor), as a pair
PyObject *pair(PyObject *a_given, const at::Tensor &a, PyObject *b_given, const at::Tensor &b) {
    PyObject *t = PyTuple_New(2);
    if (!t) throw Raised();
    try {
        PyTuple_SET_ITEM(t, 0, given(a_given) ? (Py_INCREF(a_given), a_given) : wrap(a));
        PyTuple_SET_ITEM(t, 1, given(b_given) ? (Py_INCREF(b_given), b_given) : wrap(b));
    } catch (...) {
        Py_DECREF(t);
        throw;
    }
    return t;
}
PyObject *one(PyObject *a_given, const at::Tensor &a) {
    if (!given(a_given)) return wrap(a);
    Py_INCREF(a_given);
    return a_given;
}

using Args = PyObject *const *;

// (groups, x, codes, row_class, stream)
PyObject *quantize_act(Args a) {
    const dgq_groups_t *g = groups_of(a[0]);
    const at::Tensor &x = tensor(a[1], at::kFloat, "x");
    if (x.dim() != 2) raise_value("x must be [rows, channels]");
    const int64_t rows = x.size(0);
    const dgq_groups_info_t info = info_of(g);
    if (g && x.size(1) != info.channels) {
        PyErr_Format(PyExc_ValueError, "x has %lld channels, the groups have %d", (long long)x.size(1), info.channels);
        throw Raised();
    }
    const CodesShape shape(g, rows);
    const at::Tensor codes = given(a[2]) ? tensor(a[2], at::kChar, "codes") : empty(shape.sizes(), at::kChar, x);
    const at::Tensor cls = given(a[3]) ? tensor(a[3], at::kByte, "row_class") : empty({rows}, at::kByte, x);
    if (!shape.is(codes) || cls.numel() != rows) raise_value("codes / row_class have the wrong shape");
    void *st = stream_of(a[4]);
    const float *xp = pointer<float>(x);
    int8_t *cp = pointer<int8_t>(codes);
    uint8_t *rp = pointer<uint8_t>(cls);
    enqueue([&] { return dgq_quantize_act(g, xp, rows, cp, rp, st); });
    return pair(a[2], codes, a[3], cls);
}

struct LinearIn {
    const dgq_groups_t *g;
    const dgq_weight_t *w;
    const at::Tensor &codes, &cls;
    int64_t rows;
    LinearIn(PyObject *groups, PyObject *weight, PyObject *c, PyObject *r)
        : g(groups_of(groups)), w(weight_of(weight)), codes(tensor(c, at::kChar, "codes")),
          cls(tensor(r, at::kByte, "row_class")), rows(cls.numel()) {
        if (!CodesShape(g, rows).is(codes)) raise_value("codes / row_class have the wrong shape");
    }
};

// (groups, weight, codes, row_class, y, acc_dump, stream, workspace)
PyObject *linear(Args a) {
    const LinearIn in(a[0], a[1], a[2], a[3]);
    const int64_t O = out_channels_of(a[1]);
    const at::Tensor y = given(a[4]) ? tensor(a[4], at::kFloat, "y") : empty({in.rows, O}, at::kFloat, in.codes);
    if (!shape_is(y, {in.rows, O})) raise_value("y has the wrong shape");
    int32_t *dump = nullptr;
    if (given(a[5])) {
        const at::Tensor &d = tensor(a[5], at::kInt, "acc_dump");
        if (!shape_is(d, {in.rows, O, info_of(in.g).n_groups})) raise_value("acc_dump has the wrong shape");
        dump = pointer<int32_t>(d);
    }
    void *ws = nullptr;
    size_t ws_bytes = 0;
    if (given(a[7])) {
        const at::Tensor &t = tensor(a[7], at::kByte, "workspace");
        ws = t.data_ptr();
        ws_bytes = (size_t)t.numel();
    }
    void *st = stream_of(a[6]);
    const int8_t *cp = pointer<int8_t>(in.codes);
    const uint8_t *rp = pointer<uint8_t>(in.cls);
    float *yp = pointer<float>(y);
    enqueue([&] { return dgq_linear(in.g, in.w, cp, rp, in.rows, yp, dump, ws, ws_bytes, st); });
    return one(a[4], y);
}

// (groups, weight, codes, row_class, y, stream)
PyObject *linear_geglu(Args a) {
    const LinearIn in(a[0], a[1], a[2], a[3]);
    const int64_t oh = out_channels_of(a[1]) / 2;
    const at::Tensor y = given(a[4]) ? tensor(a[4], at::kFloat, "y") : empty({in.rows, oh}, at::kFloat, in.codes);
    if (!shape_is(y, {in.rows, oh})) raise_value("y has the wrong shape");
    void *st = stream_of(a[5]);
    const int8_t *cp = pointer<int8_t>(in.codes);
    const uint8_t *rp = pointer<uint8_t>(in.cls);
    float *yp = pointer<float>(y);
    enqueue([&] { return dgq_linear_geglu(in.g, in.w, cp, rp, in.rows, yp, st); });
    return one(a[4], y);
}

// (groups, weight, codes, row_class, next_groups, codes_next, row_class_next, stream)
PyObject *linear_geglu_requant(Args a) {
    const LinearIn in(a[0], a[1], a[2], a[3]);
    const CodesShape shape(groups_of(a[4]), in.rows);
    const at::Tensor codes2 = given(a[5]) ? tensor(a[5], at::kChar, "codes_next") : empty(shape.sizes(), at::kChar, in.codes);
    const at::Tensor cls2 = given(a[6]) ? tensor(a[6], at::kByte, "row_class_next") : empty({in.rows}, at::kByte, in.codes);
    if (!shape.is(codes2) || cls2.numel() != in.rows) raise_value("codes_next / row_class_next have the wrong shape");
    void *st = stream_of(a[7]);
    const int8_t *cp = pointer<int8_t>(in.codes);
    const uint8_t *rp = pointer<uint8_t>(in.cls);
    int8_t *c2 = pointer<int8_t>(codes2);
    uint8_t *r2 = pointer<uint8_t>(cls2);
    enqueue([&] { return dgq_linear_geglu_requant(in.g, in.w, cp, rp, in.rows, c2, r2, st); });
    return pair(a[5], codes2, a[6], cls2);
}

// (groups9, codes, B, H, W, codes9, stream)
PyObject *conv3x3_codes(Args a) {
    const dgq_groups_t *g9 = groups_of(a[0]);
    const at::Tensor &codes = tensor(a[1], at::kChar, "codes");
    const int32_t B = integer32(a[2]), H = integer32(a[3]), W = integer32(a[4]);
    const CodesShape shape(g9, (int64_t)B * H * W);
    if (codes.numel() * 9 != shape.n[0] * shape.n[1] * shape.n[2])
        raise_value("codes do not belong to a [B*H*W, C] map of this layer");
    const at::Tensor out = given(a[5]) ? tensor(a[5], at::kChar, "codes9") : empty(shape.sizes(), at::kChar, codes);
    if (!shape.is(out)) raise_value("codes9 has the wrong shape");
    void *st = stream_of(a[6]);
    const int8_t *cp = pointer<int8_t>(codes);
    int8_t *op = pointer<int8_t>(out);
    enqueue([&] { return dgq_conv3x3_codes(g9, cp, B, H, W, op, st); });
    return one(a[5], out);
}

// (groups, groups9, x, B, H, W, codes3, row_class, stream)
PyObject *quantize_act_conv3x3(Args a) {
    const dgq_groups_t *g = groups_of(a[0]), *g9 = groups_of(a[1]);
    const at::Tensor &x = tensor(a[2], at::kFloat, "x");
    const int32_t B = integer32(a[3]), H = integer32(a[4]), W = integer32(a[5]);
    const int64_t rows = (int64_t)B * H * W;
    if (g && !shape_is(x, {rows, info_of(g).channels})) raise_value("x must be [B*H*W, C]");
    const int64_t nbytes = (int64_t)dgq_conv3x3_codes3_bytes(g9, B, H, W);
    const at::Tensor codes3 = given(a[6]) ? tensor(a[6], at::kChar, "codes3") : empty({nbytes}, at::kChar, x);
    const at::Tensor cls = given(a[7]) ? tensor(a[7], at::kByte, "row_class") : empty({rows}, at::kByte, x);
    if (codes3.numel() != nbytes || cls.numel() != rows) raise_value("codes3 / row_class have the wrong size");
    void *st = stream_of(a[8]);
    const float *xp = pointer<float>(x);
    int8_t *cp = pointer<int8_t>(codes3);
    uint8_t *rp = pointer<uint8_t>(cls);
    enqueue([&] { return dgq_quantize_act_conv3x3(g, g9, xp, B, H, W, cp, rp, st); });
    return pair(a[6], codes3, a[7], cls);
}

// (groups9, weight, codes3, row_class, B, H, W, y, stream)
PyObject *linear_conv3x3(Args a) {
    const dgq_groups_t *g9 = groups_of(a[0]);
    const dgq_weight_t *w = weight_of(a[1]);
    const at::Tensor &codes3 = tensor(a[2], at::kChar, "codes3"), &cls = tensor(a[3], at::kByte, "row_class");
    const int32_t B = integer32(a[4]), H = integer32(a[5]), W = integer32(a[6]);
    const int64_t rows = (int64_t)B * H * W, O = out_channels_of(a[1]);
    holds(codes3, (int64_t)dgq_conv3x3_codes3_bytes(g9, B, H, W), "codes3");
    holds(cls, rows, "row_class");
    const at::Tensor y = given(a[7]) ? tensor(a[7], at::kFloat, "y") : empty({rows, O}, at::kFloat, codes3);
    if (!shape_is(y, {rows, O})) raise_value("y has the wrong shape");
    void *st = stream_of(a[8]);
    const int8_t *cp = pointer<int8_t>(codes3);
    const uint8_t *rp = pointer<uint8_t>(cls);
    float *yp = pointer<float>(y);
    enqueue([&] { return dgq_linear_conv3x3(g9, w, cp, rp, B, H, W, yp, st); });
    return one(a[7], y);
}

// The sizes of an attention call's queries.
struct AttnShape {
    int64_t B, N, H, d;
    explicit AttnShape(const at::Tensor &q) {
        if (q.dim() != 4) raise_value("q must be [B, N, H, d]");
        B = q.size(0), N = q.size(1), H = q.size(2), d = q.size(3);
        if (B > INT32_MAX || N > INT32_MAX || H > INT32_MAX || d > INT32_MAX) raise_value("q is too large");
    }
};

// (q, k, v, key_bias, attn_bits, out, scale_out, codes_dump, workspace, stream)
PyObject *xattn_logq(Args a) {
    const at::Tensor &q = tensor(a[0], at::kFloat, "q"), &k = tensor(a[1], at::kFloat, "k"), &v = tensor(a[2], at::kFloat, "v");
    const float *kb = optional<float>(a[3], at::kFloat, "key_bias");
    const AttnShape s(q);
    const int64_t nk = k.dim() > 1 ? k.size(1) : 0;
    if (nk > INT32_MAX || !shape_is(k, {s.B, nk, s.H, s.d}) || !shape_is(v, {s.B, nk, s.H, s.d}))
        raise_value("k / v have the wrong shape");
    if (kb && THPVariable_Unpack(a[3]).numel() != nk) raise_value("key_bias has the wrong shape");
    const int32_t bits = integer32(a[4]);
    const at::Tensor out = given(a[5]) ? tensor(a[5], at::kFloat, "out") : empty(q.sizes(), at::kFloat, q);
    holds(out, q.numel(), "out");
    const at::Tensor scale = given(a[6]) ? tensor(a[6], at::kFloat, "scale_out") : empty({s.B}, at::kFloat, q);
    holds(scale, s.B, "scale_out");
    uint8_t *dump = optional<uint8_t>(a[7], at::kByte, "codes_dump");
    if (dump && !shape_is(THPVariable_Unpack(a[7]), {s.B, s.H, s.N, nk - 1})) raise_value("codes_dump has the wrong shape");
    at::Tensor ws;
    if (given(a[8])) {
        if (!THPVariable_Check(a[8])) raise(PyExc_TypeError, "workspace must be a tensor");
        ws = THPVariable_Unpack(a[8]);
    } else if (const size_t need = dgq_xattn_workspace_bytes((int32_t)s.B, (int32_t)s.N, (int32_t)s.H, (int32_t)s.d, (int32_t)nk)) {
        ws = empty({(int64_t)need}, at::kByte, q);
    }
    void *wp = ws.defined() ? ws.data_ptr() : nullptr;
    const size_t wb = ws.defined() ? (size_t)ws.numel() * ws.element_size() : 0;
    void *st = stream_of(a[9]);
    const float *qp = pointer<float>(q), *kp = pointer<float>(k), *vp = pointer<float>(v);
    float *op = pointer<float>(out), *sp = pointer<float>(scale);
    enqueue([&] {
        return dgq_xattn_logq(qp, kp, vp, kb, (int32_t)s.B, (int32_t)s.N, (int32_t)s.H, (int32_t)s.d, (int32_t)nk, bits, op,
                              sp, dump, wp, wb, st);
    });
    return pair(a[5], out, a[6], scale);
}

// (q, k, v, key_bias, attn_bits, scale_in, out, scale_out, codes_dump, stream); scale_out None stays None
PyObject *xattn_logq_static(Args a) {
    const at::Tensor &q = tensor(a[0], at::kFloat, "q"), &k = tensor(a[1], at::kFloat, "k"), &v = tensor(a[2], at::kFloat, "v");
    const at::Tensor &sin = tensor(a[5], at::kFloat, "scale_in");
    const AttnShape s(q);
    const int64_t nk = k.dim() > 1 ? k.size(1) : 0;
    if (nk > INT32_MAX || k.numel() != s.B * nk * s.H * s.d || v.numel() != k.numel())
        raise_value("k / v have the wrong size");
    const float *kb = optional<float>(a[3], at::kFloat, "key_bias");
    holds_if_given(a[3], nk, "key_bias");
    holds(sin, s.B, "scale_in");
    const int32_t bits = integer32(a[4]);
    const at::Tensor out = given(a[6]) ? tensor(a[6], at::kFloat, "out") : empty(q.sizes(), at::kFloat, q);
    holds(out, q.numel(), "out");
    float *so = optional<float>(a[7], at::kFloat, "scale_out");
    holds_if_given(a[7], s.B, "scale_out");
    uint8_t *dump = optional<uint8_t>(a[8], at::kByte, "codes_dump");
    holds_if_given(a[8], s.B * s.H * s.N * (nk - 1), "codes_dump");
    void *st = stream_of(a[9]);
    const float *qp = pointer<float>(q), *kp = pointer<float>(k), *vp = pointer<float>(v), *ip = pointer<float>(sin);
    float *op = pointer<float>(out);
    enqueue([&] {
        return dgq_xattn_logq_static(qp, kp, vp, kb, (int32_t)s.B, (int32_t)s.N, (int32_t)s.H, (int32_t)s.d, (int32_t)nk,
                                     bits, ip, op, so, dump, st);
    });
    PyObject *o = one(a[6], out);
    PyObject *t = PyTuple_Pack(2, o, a[7]);
    Py_DECREF(o);
    if (!t) throw Raised();
    return t;
}

// (q, k, v, attn_bits, scale_in, out, scale_out, codes_dump, workspace, stream)
PyObject *selfattn_logq(Args a) {
    const at::Tensor &q = tensor(a[0], at::kFloat, "q"), &k = tensor(a[1], at::kFloat, "k"), &v = tensor(a[2], at::kFloat, "v");
    const at::Tensor &sin = tensor(a[4], at::kFloat, "scale_in");
    const AttnShape s(q);
    if (k.sizes() != q.sizes() || v.sizes() != q.sizes() || sin.numel() != s.B)
        raise_value("q, k, v must share one shape [B,N,H,d] and scale_in have B entries");
    const int32_t bits = integer32(a[3]);
    const at::Tensor out = given(a[5]) ? tensor(a[5], at::kFloat, "out") : empty(q.sizes(), at::kFloat, q);
    holds(out, q.numel(), "out");
    float *so = optional<float>(a[6], at::kFloat, "scale_out");
    holds_if_given(a[6], s.B, "scale_out");
    uint8_t *dump = optional<uint8_t>(a[7], at::kByte, "codes_dump");
    if (dump && !shape_is(THPVariable_Unpack(a[7]), {s.B, s.H, s.N, s.N})) raise_value("codes_dump must be [B,H,N,N]");
    at::Tensor ws;
    if (given(a[8])) {
        if (!THPVariable_Check(a[8])) raise(PyExc_TypeError, "workspace must be a tensor");
        ws = THPVariable_Unpack(a[8]);
    } else {
        const size_t need = dgq_selfattn_workspace_bytes((int32_t)s.B, (int32_t)s.N, (int32_t)s.H, (int32_t)s.d);
        ws = empty({(int64_t)(need > 16 ? need : 16)}, at::kByte, q);
    }
    void *wp = ws.data_ptr(), *st = stream_of(a[9]);
    const size_t wb = (size_t)ws.numel();
    const float *qp = pointer<float>(q), *kp = pointer<float>(k), *vp = pointer<float>(v), *ip = pointer<float>(sin);
    float *op = pointer<float>(out);
    enqueue([&] {
        return dgq_selfattn_logq(qp, kp, vp, (int32_t)s.B, (int32_t)s.N, (int32_t)s.H, (int32_t)s.d, bits, ip, op, so, dump,
                                 wp, wb, st);
    });
    return one(a[5], out);
}

template <PyObject *(*F)(Args), int NARGS>
PyObject *call(PyObject *, Args a, Py_ssize_t n) {
    if (n != NARGS) {
        PyErr_Format(PyExc_TypeError, "expected %d arguments, got %zd", NARGS, n);
        return nullptr;
    }
    HANDLE_TH_ERRORS  // torch's own errors (out of memory and the like) as its Python calls report them
    try {
        return F(a);
    } catch (const Raised &) {
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}

PyObject *set_error_class(PyObject *, PyObject *cls) {
    Py_INCREF(cls);
    Py_XSETREF(g_error, cls);
    Py_RETURN_NONE;
}

#define DGQ_METHOD(NAME, NARGS) {#NAME, (PyCFunction)(void (*)(void))call<NAME, NARGS>, METH_FASTCALL, nullptr}
PyMethodDef kMethods[] = {
    DGQ_METHOD(quantize_act, 5),
    DGQ_METHOD(linear, 8),
    DGQ_METHOD(linear_geglu, 6),
    DGQ_METHOD(linear_geglu_requant, 8),
    DGQ_METHOD(conv3x3_codes, 7),
    DGQ_METHOD(quantize_act_conv3x3, 9),
    DGQ_METHOD(linear_conv3x3, 9),
    DGQ_METHOD(xattn_logq, 10),
    DGQ_METHOD(xattn_logq_static, 10),
    DGQ_METHOD(selfattn_logq, 10),
    {"set_error_class", set_error_class, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_hot", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

extern "C" __attribute__((visibility("default"))) PyObject *PyInit__hot(void) {
    s_handle = PyUnicode_InternFromString("handle");
    s_out_channels = PyUnicode_InternFromString("out_channels");
    s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    if (!s_handle || !s_out_channels || !s_cuda_stream) return nullptr;
    return PyModule_Create(&kModule);
}
