// The binding's calls in native code: what binding.py does for them in Python, for the plain case.
//
// What a call costs on the host decides the smallest problems: kernels of 5 us, launched in 2.3 us each, behind 1 to 1.5 us per
// torch.empty, 1.5 to 2 us of ctypes and as much again of attribute look-ups.  A forward of 256 x 1024 -> 1024 (two calls,
// six allocations, two launches) takes 20.6 us through the Python code and 12 through this.
//
// Every function returns None for anything but the plain case (an argument that is not exactly a torch.Tensor with storage on
// a GPU, a dict or number of another type, a shape or type that the Python code refuses, torch function or dispatch modes):
// binding.py then runs its own code, which says what is wrong or does what the mode asks for.  The kernels are the same
// either way; the addresses of the library's functions come from the library that binding.py has loaded.
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/ops/empty.h>
#include <ATen/ops/empty_strided.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>

#include "moss.h"
#include "moss_producer.h"

namespace {

struct Library {
    decltype(&moss_quant_workspace_bytes) quant_workspace_bytes;
    decltype(&moss_quant_act_2level) quant_act_2level;
    decltype(&moss_quant_act_2level_given_max) quant_act_2level_given_max;
    decltype(&moss_gemm_fp8_mx) gemm_fp8_mx;
    decltype(&moss_weight_workspace_bytes) weight_workspace_bytes;
    decltype(&moss_weight_autoscale_cast) weight_autoscale_cast;
    decltype(&moss_internal_swiglu_bf16) swiglu_bf16;
    decltype(&moss_internal_swiglu_bf16_backward) swiglu_bf16_backward;
    decltype(&moss_internal_add_rmsnorm_bf16) add_rmsnorm_bf16;
    decltype(&moss_internal_rmsnorm_bf16_backward) rmsnorm_bf16_backward;
};

Library lib;
PyObject *check = nullptr, *adamw_type = nullptr, *get_device = nullptr, *get_stream = nullptr;
PyObject *k_q_row, *k_e_row, *k_q_col, *k_e_col, *k_s;

bool plain_state() { return !at::impl::torch_function_mode_enabled() && !c10::impl::dispatch_mode_enabled(); }

// the tensor of a plain argument, nullptr otherwise
const at::Tensor *plain(PyObject *o)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || !t.has_storage() || t.numel() == 0) return nullptr;
    return &t;
}

// an optional tensor: false if it is there and not plain
bool optional(PyObject *o, const at::Tensor *&t)
{
    t = nullptr;
    return o == Py_None || (t = plain(o)) != nullptr;
}

void *ptr(const at::Tensor *t) { return t ? t->data_ptr() : nullptr; }
uint8_t *bytes(const at::Tensor *t) { return static_cast<uint8_t *>(ptr(t)); }

at::Tensor make(at::IntArrayRef shape, at::ScalarType type, const at::Tensor &like)
{
    return at::empty(shape, at::TensorOptions().dtype(type).device(like.device()));
}

at::Tensor make_rows(const at::Tensor &like)
{
    return at::empty_strided({like.size(0), like.size(1)}, {like.stride(0), 1}, at::TensorOptions().dtype(at::kBFloat16).device(like.device()));
}

// an argument that the call allocates if it is absent: the Python object to return (a new reference) and the tensor
struct Output {
    at::Tensor t;
    PyObject *o = nullptr;
    ~Output() { Py_XDECREF(o); }
    void take(PyObject *given, const at::Tensor *tensor)
    {
        t = *tensor;
        Py_INCREF(given);
        o = given;
    }
    void set(at::Tensor made)
    {
        t = std::move(made);
        o = THPVariable_Wrap(t);
    }
    PyObject *release()
    {
        PyObject *r = o;
        o = nullptr;
        return r;
    }
};

// the current stream of the current device, as binding.py asks for it; false with an exception set
bool current_stream(void *&stream)
{
    PyObject *device = PyObject_CallNoArgs(get_device);
    if (!device) return false;
    PyObject *handle = PyObject_CallOneArg(get_stream, device);
    Py_DECREF(device);
    if (!handle) return false;
    stream = PyLong_AsVoidPtr(handle);
    Py_DECREF(handle);
    return !(stream == nullptr && PyErr_Occurred());
}

// false with the exception set that binding.py raises for the status
bool checked(int rc, const char *what)
{
    if (rc == MOSS_OK) return true;
    PyObject *r = PyObject_CallFunction(check, "is", rc, what);
    if (r) {
        Py_DECREF(r);
        PyErr_SetString(PyExc_RuntimeError, what);
    }
    return false;
}

bool rows_bf16(const at::Tensor &t) { return t.dim() == 2 && t.scalar_type() == at::kBFloat16 && t.stride(1) == 1; }
bool same_rows(const at::Tensor *t, const at::Tensor &like)
{
    return !t || (rows_bf16(*t) && t->size(0) == like.size(0) && t->size(1) == like.size(1) && t->stride(0) == like.stride(0));
}

// An exception of torch (out of memory, say) must not cross into C: it becomes the Python exception it is there.
template <typename F>
PyObject *guarded(F f)
{
    HANDLE_TH_ERRORS
    return f();
    END_HANDLE_TH_ERRORS
}

#define PLAIN_OR_NONE(cond) \
    do {                    \
        if (!(cond)) Py_RETURN_NONE; \
    } while (0)

template <typename F>
int without_gil(F f)
{
    PyThreadState *save = PyEval_SaveThread();
    const int rc = f();
    PyEval_RestoreThread(save);
    return rc;
}

struct QuantOutputs {
    Output q_row, e_row, q_col, e_col, s;

    // out[key] of a dict or None: false if it is there and not plain
    static bool get(PyObject *out, PyObject *key, PyObject *&o, const at::Tensor *&t)
    {
        o = out == Py_None ? nullptr : PyDict_GetItem(out, key);
        t = nullptr;
        if (!o || o == Py_None) {
            o = nullptr;
            return true;
        }
        return (t = plain(o)) != nullptr;
    }

    static bool group(PyObject *out, bool want, PyObject *kq, PyObject *ke, Output &q, Output &e, int64_t n, int64_t inner, const at::Tensor &x)
    {
        if (!want) return true;
        PyObject *oq, *oe;
        const at::Tensor *tq, *te;
        if (!get(out, kq, oq, tq) || !get(out, ke, oe, te)) return false;
        if (tq) {
            if (!te) return false;
            q.take(oq, tq);
            e.take(oe, te);
        } else {
            q.set(make({n, inner}, at::kByte, x));
            e.set(make({n, inner / 32}, at::kByte, x));
        }
        return true;
    }

    bool fill(PyObject *out, unsigned flags, const at::Tensor &x)
    {
        if (out != Py_None && !PyDict_CheckExact(out)) return false;
        PyObject *os;
        const at::Tensor *ts;
        const int64_t rows = x.size(0), cols = x.size(1);
        if (!get(out, k_s, os, ts)) return false;
        if (!group(out, flags & MOSS_Q_ROW, k_q_row, k_e_row, q_row, e_row, rows, cols, x)) return false;
        if (!group(out, flags & MOSS_Q_COL, k_q_col, k_e_col, q_col, e_col, cols, rows, x)) return false;
        if (ts) s.take(os, ts);
        else s.set(make({1}, at::kFloat, x));
        return true;
    }

    static uint8_t *at(const Output &o) { return o.o ? bytes(&o.t) : nullptr; }

    PyObject *dict() const
    {
        PyObject *d = PyDict_New();
        if (!d) return nullptr;
        const std::pair<PyObject *, const Output *> items[5] = {{k_q_row, &q_row}, {k_e_row, &e_row}, {k_q_col, &q_col}, {k_e_col, &e_col}, {k_s, &s}};
        for (const auto &[key, value] : items)
            if (PyDict_SetItem(d, key, value->o ? value->o : Py_None) < 0) {
                Py_DECREF(d);
                return nullptr;
            }
        return d;
    }
};

bool flags_of(PyObject *o, unsigned &flags)
{
    if (!PyLong_CheckExact(o)) return false;
    int overflow;
    const long v = PyLong_AsLongAndOverflow(o, &overflow);
    if (overflow || v < 0 || v > 0xFF) return false;
    flags = (unsigned)v;
    return true;
}

// (x, flags, out, workspace)
PyObject *quant_act_2level(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject * {
        unsigned flags;
        const at::Tensor *x, *ws;
        PLAIN_OR_NONE(n == 4 && plain_state() && (x = plain(a[0])) && rows_bf16(*x) && flags_of(a[1], flags) && optional(a[3], ws));
        QuantOutputs out;
        PLAIN_OR_NONE(out.fill(a[2], flags, *x));
        const int64_t rows = x->size(0), cols = x->size(1);
        at::Tensor own;
        if (!ws) {
            own = make({std::max<int64_t>((int64_t)lib.quant_workspace_bytes(rows, cols, flags), 16)}, at::kByte, *x);
            ws = &own;
        }
        void *stream;
        if (!current_stream(stream)) return nullptr;
        void *px = ptr(x), *pw = ptr(ws);
        uint8_t *qr = out.at(out.q_row), *er = out.at(out.e_row), *qc = out.at(out.q_col), *ec = out.at(out.e_col);
        float *s = reinterpret_cast<float *>(out.at(out.s));
        const int64_t ld = x->stride(0);
        const size_t wn = (size_t)ws->numel();
        const int rc = without_gil([&] { return lib.quant_act_2level(px, rows, cols, ld, flags, qr, er, qc, ec, s, pw, wn, stream); });
        return checked(rc, "moss_quant_act_2level") ? out.dict() : nullptr;
    });
}

// (x, absmax_bits, flags, out)
PyObject *quant_act_2level_given_max(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject * {
        unsigned flags;
        const at::Tensor *x, *top;
        PLAIN_OR_NONE(n == 4 && plain_state() && (x = plain(a[0])) && rows_bf16(*x) && (top = plain(a[1])) && top->scalar_type() == at::kInt &&
                      top->numel() == 1 && flags_of(a[2], flags));
        QuantOutputs out;
        PLAIN_OR_NONE(out.fill(a[3], flags, *x));
        void *stream;
        if (!current_stream(stream)) return nullptr;
        const int64_t rows = x->size(0), cols = x->size(1), ld = x->stride(0);
        void *px = ptr(x);
        const uint32_t *word = static_cast<const uint32_t *>(ptr(top));
        uint8_t *qr = out.at(out.q_row), *er = out.at(out.e_row), *qc = out.at(out.q_col), *ec = out.at(out.e_col);
        float *s = reinterpret_cast<float *>(out.at(out.s));
        const int rc = without_gil([&] { return lib.quant_act_2level_given_max(px, rows, cols, ld, flags, word, qr, er, qc, ec, s, stream); });
        return checked(rc, "moss_quant_act_2level_given_max") ? out.dict() : nullptr;
    });
}

// 0 BF16, 1 FP32, -1 neither
int dtype_of(const at::Tensor &t)
{
    return t.scalar_type() == at::kFloat ? MOSS_DT_F32 : t.scalar_type() == at::kBFloat16 ? MOSS_DT_BF16 : -1;
}

// (a_q, a_e, a_s, b_q, b_e, b_s, out, accumulate); without `out` the result is BF16
PyObject *gemm_fp8_mx(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject * {
        const at::Tensor *aq, *ae, *as, *bq, *be, *bs, *given;
        PLAIN_OR_NONE(n == 8 && plain_state() && (aq = plain(a[0])) && optional(a[1], ae) && optional(a[2], as) && (bq = plain(a[3])) &&
                      optional(a[4], be) && optional(a[5], bs) && optional(a[6], given) && PyBool_Check(a[7]));
        PLAIN_OR_NONE(aq->dim() == 2 && bq->dim() == 2 && aq->size(1) == bq->size(1) && aq->is_contiguous() && bq->is_contiguous());
        const int64_t M = aq->size(0), N = bq->size(0), K = aq->size(1);
        Output out;
        if (given) {
            PLAIN_OR_NONE(given->dim() >= 1 && dtype_of(*given) >= 0);
            out.take(a[6], given);
        } else {
            out.set(make({M, N}, at::kBFloat16, *aq));
        }
        void *stream;
        if (!current_stream(stream)) return nullptr;
        const uint8_t *pa = bytes(aq), *pae = bytes(ae), *pb = bytes(bq), *pbe = bytes(be);
        const float *sa = static_cast<const float *>(ptr(as)), *sb = static_cast<const float *>(ptr(bs));
        void *po = ptr(&out.t);
        const int dt = dtype_of(out.t), acc = a[7] == Py_True;
        const int64_t ld = out.t.stride(0);
        const int rc = without_gil([&] { return lib.gemm_fp8_mx(M, N, K, pa, pae, sa, pb, pbe, sb, po, dt, ld, acc, nullptr, 0, stream); });
        return checked(rc, "moss_gemm_fp8_mx") ? out.release() : nullptr;
    });
}

// (w, m, v, g, args, state, wq, wq_t, want_transpose, workspace)
PyObject *weight_autoscale_cast(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject * {
        const at::Tensor *t[3], *g, *state, *wq, *wq_t, *ws;
        PLAIN_OR_NONE(n == 10 && plain_state());
        for (int i = 0; i < 3; i++) PLAIN_OR_NONE((t[i] = plain(a[i])) && t[i]->is_contiguous() && t[i]->scalar_type() == at::kFloat);
        PLAIN_OR_NONE((g = plain(a[3])) && g->is_contiguous() && dtype_of(*g) >= 0 && t[0]->dim() == 2);
        PLAIN_OR_NONE((PyObject *)Py_TYPE(a[4]) == adamw_type && (state = plain(a[5])) && optional(a[6], wq) && optional(a[7], wq_t) &&
                      PyBool_Check(a[8]) && optional(a[9], ws));
        moss_adamw_args args;
        {
            Py_buffer view;
            if (PyObject_GetBuffer(a[4], &view, PyBUF_SIMPLE) < 0) return nullptr;
            const bool fits = view.len == (Py_ssize_t)sizeof(args);
            if (fits) memcpy(&args, view.buf, sizeof(args));
            PyBuffer_Release(&view);
            PLAIN_OR_NONE(fits);
        }
        const int64_t rows = t[0]->size(0), cols = t[0]->size(1);
        Output q, q_t;
        if (wq) q.take(a[6], wq);
        else q.set(make({rows, cols}, at::kByte, *t[0]));
        if (wq_t) q_t.take(a[7], wq_t);
        else if (a[8] == Py_True) q_t.set(make({cols, rows}, at::kByte, *t[0]));
        at::Tensor own;
        if (!ws) {
            own = make({std::max<int64_t>((int64_t)lib.weight_workspace_bytes(rows, cols), 16)}, at::kByte, *t[0]);
            ws = &own;
        }
        void *stream;
        if (!current_stream(stream)) return nullptr;
        float *w = static_cast<float *>(ptr(t[0])), *m = static_cast<float *>(ptr(t[1])), *v = static_cast<float *>(ptr(t[2]));
        void *pg = ptr(g), *pw = ptr(ws);
        auto *st = static_cast<moss_wscale_state *>(ptr(state));
        uint8_t *pq = bytes(&q.t), *pq_t = q_t.o ? bytes(&q_t.t) : nullptr;
        const int dt = dtype_of(*g);
        const size_t wn = (size_t)ws->numel();
        const int rc = without_gil([&] { return lib.weight_autoscale_cast(w, m, v, pg, dt, rows, cols, &args, st, pq, pq_t, pw, wn, stream); });
        if (!checked(rc, "moss_weight_autoscale_cast")) return nullptr;
        return PyTuple_Pack(2, q.o, q_t.o ? q_t.o : Py_None);
    });
}

// a one-element int32 tensor: the caller's, or a new one
bool word(PyObject *o, Output &out, const at::Tensor &like)
{
    const at::Tensor *t;
    if (!optional(o, t)) return false;
    if (t) out.take(o, t);
    else out.set(make({1}, at::kInt, like));
    return true;
}

// BF16 rows of the stride of `like`: the caller's (`check_stride`: of this very stride, columns neighbours), or new ones
bool rows_out(PyObject *o, Output &out, const at::Tensor &like, bool check_stride)
{
    const at::Tensor *t;
    if (!optional(o, t)) return false;
    if (t) {
        if (t->dim() != 2 || (check_stride && (t->stride(0) != like.stride(0) || t->stride(1) != 1))) return false;
        out.take(o, t);
    } else {
        out.set(make_rows(like));
    }
    return true;
}

// scratch of a producer: any contents, the call's own until it has run (the allocator hands it out again in stream order)
at::Tensor producer_workspace(const at::Tensor &like) { return make({(int64_t)kProducerWorkspaceBytes}, at::kByte, like); }

uint32_t *word_ptr(const Output &o) { return static_cast<uint32_t *>(ptr(&o.t)); }

// (gate, up, h, absmax_bits)
PyObject *swiglu_bf16(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject * {
        const at::Tensor *gate, *up;
        PLAIN_OR_NONE(n == 4 && plain_state() && (gate = plain(a[0])) && rows_bf16(*gate) && (up = plain(a[1])) && same_rows(up, *gate));
        Output h, top;
        PLAIN_OR_NONE(rows_out(a[2], h, *gate, true) && word(a[3], top, *gate));
        void *stream;
        if (!current_stream(stream)) return nullptr;
        const int64_t rows = gate->size(0), cols = gate->size(1), ld = gate->stride(0);
        void *pg = ptr(gate), *pu = ptr(up), *ph = ptr(&h.t);
        uint32_t *w = word_ptr(top);
        const at::Tensor ws = producer_workspace(*gate);
        void *pw = ws.data_ptr();
        const int rc = without_gil([&] { return lib.swiglu_bf16(pg, pu, rows, cols, ld, ph, w, pw, kProducerWorkspaceBytes, stream); });
        return checked(rc, "moss_swiglu_bf16") ? PyTuple_Pack(2, h.o, top.o) : nullptr;
    });
}

// (gate, up, dh, d_gate, d_up, d_gate_absmax_bits, d_up_absmax_bits)
PyObject *swiglu_bf16_backward(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject * {
        const at::Tensor *gate, *up, *dh;
        PLAIN_OR_NONE(n == 7 && plain_state() && (gate = plain(a[0])) && rows_bf16(*gate) && (up = plain(a[1])) && same_rows(up, *gate) &&
                      (dh = plain(a[2])) && same_rows(dh, *gate));
        Output dg, du, tg, tu;
        PLAIN_OR_NONE(rows_out(a[3], dg, *gate, true) && rows_out(a[4], du, *gate, true) && word(a[5], tg, *gate) && word(a[6], tu, *gate));
        void *stream;
        if (!current_stream(stream)) return nullptr;
        const int64_t rows = gate->size(0), cols = gate->size(1), ld = gate->stride(0);
        void *pg = ptr(gate), *pu = ptr(up), *pd = ptr(dh), *og = ptr(&dg.t), *ou = ptr(&du.t);
        uint32_t *wg = word_ptr(tg), *wu = word_ptr(tu);
        const at::Tensor ws = producer_workspace(*gate);
        void *pw = ws.data_ptr();
        const int rc = without_gil([&] { return lib.swiglu_bf16_backward(pg, pu, pd, rows, cols, ld, og, ou, wg, wu, pw, kProducerWorkspaceBytes, stream); });
        return checked(rc, "moss_swiglu_bf16_backward") ? PyTuple_Pack(4, dg.o, du.o, tg.o, tu.o) : nullptr;
    });
}

bool gamma_ok(const at::Tensor *g, const at::Tensor &x)
{
    return g && g->scalar_type() == at::kBFloat16 && g->is_contiguous() && g->dim() == 1 && g->size(0) == x.size(1);
}

// (x, gamma, eps, delta, h, y, absmax_bits)
PyObject *add_rmsnorm_bf16(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject * {
        const at::Tensor *x, *delta;
        PLAIN_OR_NONE(n == 7 && plain_state() && (x = plain(a[0])) && rows_bf16(*x) && gamma_ok(plain(a[1]), *x) && PyFloat_CheckExact(a[2]) &&
                      optional(a[3], delta) && same_rows(delta, *x));
        const at::Tensor *gamma = plain(a[1]);
        Output h, y, top;
        if (delta) PLAIN_OR_NONE(rows_out(a[4], h, *x, false));
        PLAIN_OR_NONE(rows_out(a[5], y, *x, false) && word(a[6], top, *x));
        void *stream;
        if (!current_stream(stream)) return nullptr;
        const float eps = (float)PyFloat_AS_DOUBLE(a[2]);
        const int64_t rows = x->size(0), cols = x->size(1), ld = x->stride(0);
        void *px = ptr(x), *pd = ptr(delta), *pg = ptr(gamma), *ph = delta ? ptr(&h.t) : nullptr, *py = ptr(&y.t);
        uint32_t *w = word_ptr(top);
        const at::Tensor ws = producer_workspace(*x);
        void *pw = ws.data_ptr();
        const int rc = without_gil([&] { return lib.add_rmsnorm_bf16(px, pd, pg, eps, rows, cols, ld, ph, py, w, pw, kProducerWorkspaceBytes, stream); });
        return checked(rc, "moss_add_rmsnorm_bf16") ? PyTuple_Pack(3, delta ? h.o : a[0], y.o, top.o) : nullptr;
    });
}

// (h, gamma, dy, eps, d_res, d_h, absmax_bits)
PyObject *rmsnorm_bf16_backward(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject * {
        const at::Tensor *h, *dy, *d_res;
        PLAIN_OR_NONE(n == 7 && plain_state() && (h = plain(a[0])) && rows_bf16(*h) && gamma_ok(plain(a[1]), *h) && (dy = plain(a[2])) &&
                      same_rows(dy, *h) && PyFloat_CheckExact(a[3]) && optional(a[4], d_res) && same_rows(d_res, *h));
        const at::Tensor *gamma = plain(a[1]);
        Output d_h, top;
        PLAIN_OR_NONE(rows_out(a[5], d_h, *h, false) && word(a[6], top, *h));
        void *stream;
        if (!current_stream(stream)) return nullptr;
        const float eps = (float)PyFloat_AS_DOUBLE(a[3]);
        const int64_t rows = h->size(0), cols = h->size(1), ld = h->stride(0);
        void *ph = ptr(h), *pg = ptr(gamma), *py = ptr(dy), *pr = ptr(d_res), *po = ptr(&d_h.t);
        uint32_t *w = word_ptr(top);
        const at::Tensor ws = producer_workspace(*h);
        void *pw = ws.data_ptr();
        const int rc = without_gil([&] { return lib.rmsnorm_bf16_backward(ph, pg, py, pr, eps, rows, cols, ld, po, w, pw, kProducerWorkspaceBytes, stream); });
        return checked(rc, "moss_rmsnorm_bf16_backward") ? PyTuple_Pack(2, d_h.o, top.o) : nullptr;
    });
}

// (addresses of the library's functions in the order of Library, _check, AdamWArgs, torch's current device and raw stream)
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 5 || !PyTuple_Check(a[0]) || PyTuple_GET_SIZE(a[0]) != (Py_ssize_t)(sizeof(lib) / sizeof(void *))) {
        PyErr_SetString(PyExc_TypeError, "bind(addresses, check, AdamWArgs, get_device, get_stream)");
        return nullptr;
    }
    void *at[sizeof(lib) / sizeof(void *)];
    for (Py_ssize_t i = 0; i < PyTuple_GET_SIZE(a[0]); i++) {
        at[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(a[0], i));
        if (!at[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "no address");
            return nullptr;
        }
    }
    memcpy(&lib, at, sizeof(lib));
    PyObject **const kept[4] = {&check, &adamw_type, &get_device, &get_stream};
    for (int i = 0; i < 4; i++) {
        Py_INCREF(a[i + 1]);
        Py_XSETREF(*kept[i], a[i + 1]);
    }
    Py_RETURN_NONE;
}

#define CALL(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {CALL(bind), CALL(quant_act_2level), CALL(quant_act_2level_given_max), CALL(gemm_fp8_mx), CALL(weight_autoscale_cast),
                         CALL(swiglu_bf16), CALL(swiglu_bf16_backward), CALL(add_rmsnorm_bf16), CALL(rmsnorm_bf16_backward),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_moss_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__moss_calls()
{
    k_q_row = PyUnicode_InternFromString("q_row");
    k_e_row = PyUnicode_InternFromString("e_row");
    k_q_col = PyUnicode_InternFromString("q_col");
    k_e_col = PyUnicode_InternFromString("e_col");
    k_s = PyUnicode_InternFromString("s");
    if (!k_q_row || !k_e_row || !k_q_col || !k_e_col || !k_s) return nullptr;
    PyObject *m = PyModule_Create(&module);
    // what this was compiled for: binding.py compares it with the torch and the library that it has before it binds anything
    if (m && (PyModule_AddStringConstant(m, "torch_version", MOSS_TORCH_VERSION) < 0 ||
              PyModule_AddObject(m, "interface", PyLong_FromUnsignedLong(MOSS_INTERFACE)) < 0)) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
