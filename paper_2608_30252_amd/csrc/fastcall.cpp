// fastcall.cpp -- the Python binding's argument marshalling in native code.
//
// A call through ctypes spends 12 - 16 us on the host (attribute reads, checks,
// two stream objects, sixteen argument conversions), more than most of the
// library's kernels run.  These functions read the same arguments, make the
// same checks and call the same C entry points in 2 - 3 us.  They handle the
// ordinary call only: on anything else -- a failed check, a tensor subclass,
// lengths that are not a list or tuple of ints, a workspace still to be
// allocated -- they return None without having enqueued anything, and the
// caller takes its Python path, which does the work or raises the error.  An
// int result is the C entry point's return code.  Nothing is kept between
// calls but the C functions' addresses.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <ATen/core/Tensor.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cmath>
#include <cstring>
#include <initializer_list>

#include "mad.h"

namespace {

struct Entry {
    decltype(&mad_draft_decode_attn) decode;
    decltype(&mad_draft_step_attn) step;
    decltype(&mad_memory_update) update;
    decltype(&mad_verify_attn) verify;
    decltype(&mad_verify_attn_vt) verify_vt;
    decltype(&mad_accept_greedy) greedy;
    decltype(&mad_accept_stochastic) stoch;
    decltype(&mad_rmsnorm_qkv_rope) qkv;
    decltype(&mad_linear_residual) linear;
    decltype(&mad_rmsnorm_swiglu) swiglu;
    decltype(&mad_workspace_bytes) ws_bytes;
} g;
PyObject *g_kv, *g_ws, *g_stream;   // class KV, the default workspaces' dict, the raw-stream getter
PyObject *s_k, *s_v, *s_length, *s_start, *s_buf;

struct Unhandled {};   // thrown for every call the Python path has to take
void need(bool ok) {
    if (!ok) throw Unhandled();
}

// an owned reference
struct Ref {
    PyObject *p;
    explicit Ref(PyObject *o) : p(o) { need(o != nullptr); }
    ~Ref() { Py_DECREF(p); }
    Ref(const Ref &) = delete;
};

const at::Tensor &tensor(PyObject *o) {
    need(THPVariable_CheckExact(o));
    return THPVariable_Unpack(o);
}
// a contiguous tensor on the call's device
const at::Tensor &dense(PyObject *o, const at::Device &dev) {
    const at::Tensor &t = tensor(o);
    need(t.is_contiguous() && t.device() == dev);
    return t;
}
const at::Tensor &first(PyObject *o) {
    const at::Tensor &t = tensor(o);
    need(t.is_contiguous() && t.is_cuda() && t.layout() == at::kStrided);
    return t;
}
bool shape(const at::Tensor &t, std::initializer_list<int64_t> want) { return t.sizes() == at::IntArrayRef(want); }
int dtype_code(const at::Tensor &t) {
    if (t.scalar_type() == at::kBFloat16) return MAD_BF16;
    need(t.scalar_type() == at::kFloat);
    return MAD_F32;
}
int small(int64_t v) {
    need(v >= 0 && v <= 0x7fffffff);
    return (int)v;
}
int as_int(PyObject *o) {
    need(PyLong_CheckExact(o));
    int over = 0;
    const long v = PyLong_AsLongAndOverflow(o, &over);
    need(!over && v >= INT32_MIN && v <= INT32_MAX);
    return (int)v;
}
double as_double(PyObject *o) {
    const double v = PyFloat_AsDouble(o);
    need(v != -1.0 || !PyErr_Occurred());
    return v;
}
// the n ints of a list or tuple
template <typename I> void ints(PyObject *o, int64_t n, I *out) {
    need((PyList_CheckExact(o) || PyTuple_CheckExact(o)) && PySequence_Fast_GET_SIZE(o) == n);
    PyObject **items = PySequence_Fast_ITEMS(o);
    for (int64_t i = 0; i < n; ++i) {
        const int v = as_int(items[i]);
        need(sizeof(I) == 4 || (v >= 0 && v <= 255));
        out[i] = (I)v;
    }
}

// What the types of the arguments alone say, looked at before anything is read: a call that is not an ordinary one
// for them goes back at once (0.2 us; an exception on the way costs 3, a fifth of the call on the Python path).
bool plain_ints(PyObject *o) {
    const Py_ssize_t n = PyList_CheckExact(o) || PyTuple_CheckExact(o) ? PySequence_Fast_GET_SIZE(o) : 0;
    return n > 0 && PyLong_CheckExact(PySequence_Fast_GET_ITEM(o, 0)) && PyLong_CheckExact(PySequence_Fast_GET_ITEM(o, n - 1));
}
bool plain_rows(PyObject *o) {   // [B][n] ints
    const Py_ssize_t n = PyList_CheckExact(o) || PyTuple_CheckExact(o) ? PySequence_Fast_GET_SIZE(o) : 0;
    return n > 0 && plain_ints(PySequence_Fast_GET_ITEM(o, 0));
}
bool plain_flags(PyObject *o) {   // ints or bools, or None
    if (o == Py_None) return true;
    const Py_ssize_t n = PyList_CheckExact(o) || PyTuple_CheckExact(o) ? PySequence_Fast_GET_SIZE(o) : 0;
    return n > 0 && (PyBool_Check(PySequence_Fast_GET_ITEM(o, 0)) || PyLong_CheckExact(PySequence_Fast_GET_ITEM(o, 0)));
}
bool plain_real(PyObject *o) { return PyFloat_CheckExact(o) || PyLong_CheckExact(o); }
bool plain_attr(PyObject *o, PyObject *name, bool none) {
    PyObject *v = PyObject_GetAttr(o, name);
    const bool ok = v && (v == Py_None ? none : plain_ints(v));
    Py_XDECREF(v);
    PyErr_Clear();
    return ok;
}
bool plain_kv(PyObject *o) {
    return Py_TYPE(o) == (PyTypeObject *)g_kv && plain_attr(o, s_length, false) && plain_attr(o, s_start, true);
}
bool plain_tensors(PyObject *const *a, std::initializer_list<int> at) {
    for (int i : at)
        if (!THPVariable_CheckExact(a[i])) return false;
    return true;
}
#define ORDINARY(n_args, cond) \
    if (n != (n_args) || !(cond)) Py_RETURN_NONE

struct View {
    mad_kv_view c;
    int32_t len[MAD_MAX_BATCH], start[MAD_MAX_BATCH];
    // KV `o` for B rows of [Hkv, cap, d] (Hkv < 0: any, returned in Hkv)
    mad_kv_view *read(PyObject *o, int B, int64_t *Hkv, int64_t d, const at::Tensor &like) {
        need(Py_TYPE(o) == (PyTypeObject *)g_kv && B <= MAD_MAX_BATCH);
        Ref ko(PyObject_GetAttr(o, s_k)), vo(PyObject_GetAttr(o, s_v)), lo(PyObject_GetAttr(o, s_length)),
            so(PyObject_GetAttr(o, s_start));
        const at::Tensor &k = tensor(ko.p), &v = tensor(vo.p);
        need(k.dim() == 4 && k.sizes() == v.sizes() && k.strides() == v.strides());
        need(k.stride(3) == 1 && k.stride(2) == k.size(3));
        need(k.size(0) == 1 || k.size(0) == B);
        if (*Hkv < 0) *Hkv = k.size(1);
        need(k.size(1) == *Hkv && k.size(3) == d);
        need(k.scalar_type() == like.scalar_type() && v.scalar_type() == like.scalar_type());
        need(k.device() == like.device() && v.device() == like.device());
        ints(lo.p, B, len);
        if (so.p != Py_None) ints(so.p, B, start);
        c.k = k.data_ptr();
        c.v = v.data_ptr();
        c.seq_stride = k.size(0) > 1 ? k.stride(0) : 0;
        c.head_stride = k.stride(1);
        c.cap = small(k.size(2));
        c.start = so.p != Py_None ? start : nullptr;
        c.len = len;
        return &c;
    }
};

void *stream_of(const at::Device &dev) {
    Ref index(PyLong_FromLong(dev.index()));
    Ref s(PyObject_CallOneArg(g_stream, index.p));
    void *p = PyLong_AsVoidPtr(s.p);
    need(!PyErr_Occurred());
    return p;
}

// the caller's workspace, or the one kept for (device, stream) if it is large enough.  It is held until the C entry
// point has returned: without the interpreter lock another thread may put a larger one in the kept one's place, and
// memory given back before this call's kernels are enqueued could be another tensor's by the time they run.
struct Scratch {
    const Ref held;
    void *p;
    size_t n;
    Scratch(PyObject *ws, const at::Device &dev, void *stream, size_t bytes) : held(of(ws, dev, stream)) {
        const at::Tensor &t = tensor(held.p);
        need((size_t)t.numel() >= bytes);
        p = t.data_ptr();
        n = (size_t)t.numel();
    }
    static PyObject *of(PyObject *ws, const at::Device &dev, void *stream) {   // an owned reference
        if (ws != Py_None) {
            Py_INCREF(ws);
            return ws;
        }
        Ref key(Py_BuildValue("(iN)", (int)dev.index(), PyLong_FromVoidPtr(stream)));
        PyObject *w = PyDict_GetItemWithError(g_ws, key.p);
        need(w != nullptr);
        return PyObject_GetAttr(w, s_buf);
    }
};

template <typename F> PyObject *guarded(F f) {
    try {
        return PyLong_FromLong(f());
    } catch (...) {   // Unhandled, or a C++ error of a tensor accessor
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}
#define RELEASED(call)         \
    int rc;                    \
    Py_BEGIN_ALLOW_THREADS     \
    rc = (call);               \
    Py_END_ALLOW_THREADS       \
    return rc

float scale_of(PyObject *o, int64_t d) { return o == Py_None ? (float)std::pow((double)d, -0.5) : (float)as_double(o); }

// attn(q, mem, win, k_new, v_new, out, lse, scale, ws, modes | None)
PyObject *attn(PyObject *, PyObject *const *a, Py_ssize_t n) {
    ORDINARY(10, plain_tensors(a, {0, 5, 6}) && (a[1] == Py_None || plain_kv(a[1])) && (a[2] == Py_None || plain_kv(a[2])) &&
                     (a[1] != Py_None || a[2] != Py_None) && (a[7] == Py_None || plain_real(a[7])) &&
                     (a[9] == Py_None || plain_ints(a[9])));
    return guarded([&]() -> int {
        const at::Tensor &q = first(a[0]);
        const at::Device dev = q.device();
        need(q.dim() == 3);
        const int B = small(q.size(0)), Hq = small(q.size(1)), d = small(q.size(2));
        int64_t Hkv = -1;
        View mem, win;
        mad_kv_view *mv = a[1] != Py_None ? mem.read(a[1], B, &Hkv, d, q) : nullptr;
        mad_kv_view *wv = a[2] != Py_None ? win.read(a[2], B, &Hkv, d, q) : nullptr;
        need(Hkv >= 1 && Hq % Hkv == 0);
        const at::Tensor &out = dense(a[5], dev), &lse = dense(a[6], dev);
        need(out.sizes() == q.sizes() && out.scalar_type() == q.scalar_type());
        need(shape(lse, {B, Hq}) && lse.scalar_type() == at::kFloat);
        need((a[3] == Py_None) == (a[4] == Py_None));
        void *kn = nullptr, *vn = nullptr;
        if (a[3] != Py_None) {
            const at::Tensor &k = dense(a[3], dev), &v = dense(a[4], dev);
            need(shape(k, {B, Hkv, d}) && shape(v, {B, Hkv, d}) && k.scalar_type() == q.scalar_type() &&
                 v.scalar_type() == q.scalar_type());
            kn = k.data_ptr();
            vn = v.data_ptr();
        }
        const float scale = scale_of(a[7], d);
        uint8_t modes[MAD_MAX_BATCH];
        const bool step = a[9] != Py_None;
        if (step) ints(a[9], B, modes);
        void *st = stream_of(dev);
        const Scratch ws(a[8], dev, st, g.ws_bytes(MAD_OP_DECODE, B, Hq, (int)Hkv, d, 1, 0));
        const int dt = dtype_code(q);
        void *qp = q.data_ptr(), *op = out.data_ptr();
        float *lp = (float *)lse.data_ptr();
        if (step) {
            RELEASED(g.step(qp, B, Hq, (int)Hkv, d, dt, scale, mv, wv, kn, vn, modes, op, lp, ws.p, ws.n, st));
        }
        RELEASED(g.decode(qp, B, Hq, (int)Hkv, d, dt, scale, mv, wv, kn, vn, op, lp, ws.p, ws.n, st));
    });
}

// update(x, w_kv, pos, mem, fire | None, rope_base)
PyObject *update(PyObject *, PyObject *const *a, Py_ssize_t n) {
    ORDINARY(6, plain_tensors(a, {0, 1}) && plain_rows(a[2]) && plain_kv(a[3]) && plain_flags(a[4]) && plain_real(a[5]));
    return guarded([&]() -> int {
        const at::Tensor &x = first(a[0]);
        const at::Tensor &w = dense(a[1], x.device());
        need(x.dim() == 3);
        const int B = small(x.size(0)), nn = small(x.size(1)), D = small(x.size(2));
        need(B <= MAD_MAX_BATCH && (int64_t)B * nn <= MAD_MAX_UPDATE_ROWS && w.dim() == 2 && w.size(1) == D &&
             w.scalar_type() == x.scalar_type());
        Ref ko(PyObject_GetAttr(a[3], s_k));
        const at::Tensor &k = tensor(ko.p);
        need(k.dim() == 4);
        int64_t Hkv = k.size(1);
        const int d = small(k.size(3));
        need(w.size(0) == 2 * Hkv * d);
        View mem;
        mad_kv_view *mv = mem.read(a[3], B, &Hkv, d, x);
        need((PyList_CheckExact(a[2]) || PyTuple_CheckExact(a[2])) && PySequence_Fast_GET_SIZE(a[2]) == B);
        int32_t pos[MAD_MAX_UPDATE_ROWS];
        for (int b = 0; b < B; ++b) ints(PySequence_Fast_ITEMS(a[2])[b], nn, pos + (size_t)b * nn);
        uint8_t fire[MAD_MAX_BATCH];
        if (a[4] != Py_None) {
            need((PyList_CheckExact(a[4]) || PyTuple_CheckExact(a[4])) && PySequence_Fast_GET_SIZE(a[4]) == B);
            for (int b = 0; b < B; ++b) {
                PyObject *f = PySequence_Fast_ITEMS(a[4])[b];
                need(PyBool_Check(f) || PyLong_CheckExact(f));
                fire[b] = PyObject_IsTrue(f) ? 1 : 0;
            }
        }
        const double base = as_double(a[5]);
        const int dt = dtype_code(x);
        void *st = stream_of(x.device()), *xp = x.data_ptr(), *wp = w.data_ptr();
        const uint8_t *fp = a[4] != Py_None ? fire : nullptr;
        RELEASED(g.update(xp, wp, pos, fp, B, nn, D, (int)Hkv, d, dt, base, mv, st));
    });
}

// verify(q, kv, out, lse, scale, ws)
PyObject *verify(PyObject *, PyObject *const *a, Py_ssize_t n) {
    ORDINARY(6, plain_tensors(a, {0, 2, 3}) && plain_kv(a[1]) && (a[4] == Py_None || plain_real(a[4])));
    return guarded([&]() -> int {
        const at::Tensor &q = first(a[0]);
        const at::Device dev = q.device();
        need(q.dim() == 4);
        const int B = small(q.size(0)), T = small(q.size(1)), Hq = small(q.size(2)), d = small(q.size(3));
        int64_t Hkv = -1;
        View kv;
        mad_kv_view *v = kv.read(a[1], B, &Hkv, d, q);
        need(v->start == nullptr && Hkv >= 1);
        const at::Tensor &out = dense(a[2], dev), &lse = dense(a[3], dev);
        need(out.sizes() == q.sizes() && out.scalar_type() == q.scalar_type());
        need(shape(lse, {B, T, Hq}) && lse.scalar_type() == at::kFloat);
        const float scale = scale_of(a[4], d);
        void *st = stream_of(dev);
        const Scratch ws(a[5], dev, st, g.ws_bytes(MAD_OP_VERIFY, B, Hq, (int)Hkv, d, T, 0));
        const int dt = dtype_code(q);
        void *qp = q.data_ptr(), *op = out.data_ptr();
        float *lp = (float *)lse.data_ptr();
        RELEASED(g.verify(qp, B, T, Hq, (int)Hkv, d, dt, scale, v, op, lp, ws.p, ws.n, st));
    });
}

// verify_vt(q, k, vt, length, out, lse, scale, ws)
PyObject *verify_vt(PyObject *, PyObject *const *a, Py_ssize_t n) {
    ORDINARY(8, plain_tensors(a, {0, 1, 2, 4, 5}) && plain_ints(a[3]) && (a[6] == Py_None || plain_real(a[6])));
    return guarded([&]() -> int {
        const at::Tensor &q = first(a[0]);
        const at::Device dev = q.device();
        const at::Tensor &k = tensor(a[1]), &vt = tensor(a[2]);
        need(q.dim() == 4 && k.dim() == 4 && vt.dim() == 4);
        const int B = small(q.size(0)), T = small(q.size(1)), Hq = small(q.size(2)), d = small(q.size(3));
        const int Hkv = small(k.size(1)), cap = small(k.size(2));
        need(B <= MAD_MAX_BATCH && shape(vt, {B, Hkv, d, cap}) && shape(k, {B, Hkv, cap, d}));
        need(k.stride(3) == 1 && k.stride(2) == d && vt.stride(3) == 1 && vt.stride(2) == cap);
        need(k.stride(0) == vt.stride(0) && k.stride(1) == vt.stride(1));
        need(k.scalar_type() == q.scalar_type() && vt.scalar_type() == q.scalar_type() && k.device() == dev && vt.device() == dev);
        int32_t len[MAD_MAX_BATCH];
        ints(a[3], B, len);
        const at::Tensor &out = dense(a[4], dev), &lse = dense(a[5], dev);
        need(out.sizes() == q.sizes() && out.scalar_type() == q.scalar_type());
        need(shape(lse, {B, T, Hq}) && lse.scalar_type() == at::kFloat);
        const float scale = scale_of(a[6], d);
        void *st = stream_of(dev);
        const Scratch ws(a[7], dev, st, g.ws_bytes(MAD_OP_VERIFY, B, Hq, Hkv, d, T, 0));
        const int dt = dtype_code(q);
        void *qp = q.data_ptr(), *op = out.data_ptr(), *kp = k.data_ptr(), *vp = vt.data_ptr();
        float *lp = (float *)lse.data_ptr();
        const int64_t seq = B > 1 ? k.stride(0) : 0, head = k.stride(1);
        RELEASED(g.verify_vt(qp, B, T, Hq, Hkv, d, dt, scale, kp, vp, seq, head, cap, len, op, lp, ws.p, ws.n, st));
    });
}

const at::Tensor &i32(PyObject *o, const at::Device &dev, std::initializer_list<int64_t> want) {
    const at::Tensor &t = dense(o, dev);
    need(t.scalar_type() == at::kInt && shape(t, want));
    return t;
}

// greedy(logits, draft | None, n_accept, next_tok, ws)
PyObject *greedy(PyObject *, PyObject *const *a, Py_ssize_t n) {
    ORDINARY(5, plain_tensors(a, {0, 2, 3}) && (a[1] == Py_None || THPVariable_CheckExact(a[1])));
    return guarded([&]() -> int {
        const at::Tensor &x = first(a[0]);
        const at::Device dev = x.device();
        need(x.dim() == 3);
        const int B = small(x.size(0)), T = small(x.size(1)), V = small(x.size(2));
        int32_t *draft = T > 1 ? (int32_t *)i32(a[1], dev, {B, T - 1}).data_ptr() : nullptr;
        need(T > 1 || a[1] == Py_None);
        int32_t *na = (int32_t *)i32(a[2], dev, {B}).data_ptr(), *nt = (int32_t *)i32(a[3], dev, {B}).data_ptr();
        void *st = stream_of(dev);
        const Scratch ws(a[4], dev, st, g.ws_bytes(MAD_OP_ACCEPT, B, 1, 1, 64, T, V));
        const int dt = dtype_code(x);
        void *xp = x.data_ptr();
        RELEASED(g.greedy(xp, dt, draft, B, T, V, na, nt, ws.p, ws.n, st));
    });
}

// stoch(p, q, draft, u, n_accept, next_tok, ws)
PyObject *stoch(PyObject *, PyObject *const *a, Py_ssize_t n) {
    ORDINARY(7, plain_tensors(a, {0, 1, 2, 3, 4, 5}));
    return guarded([&]() -> int {
        const at::Tensor &p = first(a[0]);
        const at::Device dev = p.device();
        need(p.dim() == 3 && p.scalar_type() == at::kFloat);
        const int B = small(p.size(0)), T = small(p.size(1)), V = small(p.size(2));
        need(T > 1);
        const at::Tensor &q = dense(a[1], dev), &u = dense(a[3], dev);
        need(shape(q, {B, T - 1, V}) && q.scalar_type() == at::kFloat && shape(u, {B, T}) && u.scalar_type() == at::kFloat);
        int32_t *draft = (int32_t *)i32(a[2], dev, {B, T - 1}).data_ptr();
        int32_t *na = (int32_t *)i32(a[4], dev, {B}).data_ptr(), *nt = (int32_t *)i32(a[5], dev, {B}).data_ptr();
        void *st = stream_of(dev);
        const Scratch ws(a[6], dev, st, g.ws_bytes(MAD_OP_ACCEPT_STOCH, B, 1, 1, 64, T, V));
        const float *pp = (const float *)p.data_ptr(), *qp = (const float *)q.data_ptr(), *up = (const float *)u.data_ptr();
        RELEASED(g.stoch(pp, qp, draft, up, B, T, V, na, nt, ws.p, ws.n, st));
    });
}

// qkv(x, gamma, w, pos, Hq, Hkv, d, q, k, v, xn | None, eps, rope_base, kv_from_row0)
PyObject *qkv(PyObject *, PyObject *const *a, Py_ssize_t n) {
    ORDINARY(14, plain_tensors(a, {0, 1, 2, 7, 8, 9}) && plain_ints(a[3]) && plain_real(a[11]) && plain_real(a[12]) &&
                     PyBool_Check(a[13]));
    return guarded([&]() -> int {
        const at::Tensor &x = first(a[0]);
        const at::Device dev = x.device();
        need(x.dim() == 2 && x.scalar_type() == at::kBFloat16);
        const int R = small(x.size(0)), D = small(x.size(1)), Hq = as_int(a[4]), Hkv = as_int(a[5]), d = as_int(a[6]);
        need(R <= MAD_MAX_LAYER_ROWS);
        const at::Tensor &gm = dense(a[1], dev), &w = dense(a[2], dev), &q = dense(a[7], dev), &k = dense(a[8], dev),
                         &v = dense(a[9], dev);
        need(shape(gm, {D}) && shape(w, {((int64_t)Hq + 2 * Hkv) * d, D}) && shape(q, {R, Hq, d}) && shape(k, {R, Hkv, d}) &&
             shape(v, {R, Hkv, d}));
        void *xn = nullptr;
        if (a[10] != Py_None) {
            const at::Tensor &t = dense(a[10], dev);
            need(shape(t, {R, D}));
            xn = t.data_ptr();
        }
        int32_t pos[MAD_MAX_LAYER_ROWS];
        ints(a[3], R, pos);
        const float eps = (float)as_double(a[11]);
        const double base = as_double(a[12]);
        const int row0 = a[13] == Py_True;
        void *st = stream_of(dev), *xp = x.data_ptr(), *gp = gm.data_ptr(), *wp = w.data_ptr(), *qp = q.data_ptr(),
             *kp = k.data_ptr(), *vp = v.data_ptr();
        RELEASED(g.qkv(xp, gp, eps, wp, pos, R, D, Hq, Hkv, d, base, row0, qp, kp, vp, xn, st));
    });
}

// linear(x, w, res, out)
PyObject *linear(PyObject *, PyObject *const *a, Py_ssize_t n) {
    ORDINARY(4, plain_tensors(a, {0, 1, 2, 3}));
    return guarded([&]() -> int {
        const at::Tensor &x = first(a[0]);
        const at::Device dev = x.device();
        const at::Tensor &w = dense(a[1], dev), &res = dense(a[2], dev), &out = dense(a[3], dev);
        need(x.dim() == 2 && w.dim() == 2 && x.scalar_type() == at::kBFloat16);
        const int R = small(x.size(0)), D = small(x.size(1)), N = small(w.size(0));
        need(shape(w, {N, D}) && shape(res, {R, N}) && shape(out, {R, N}));
        void *st = stream_of(dev), *xp = x.data_ptr(), *wp = w.data_ptr(), *rp = res.data_ptr(), *op = out.data_ptr();
        RELEASED(g.linear(xp, wp, rp, R, D, N, op, st));
    });
}

// swiglu(x, gamma, w_gate_up, out, eps)
PyObject *swiglu(PyObject *, PyObject *const *a, Py_ssize_t n) {
    ORDINARY(5, plain_tensors(a, {0, 1, 2, 3}) && plain_real(a[4]));
    return guarded([&]() -> int {
        const at::Tensor &x = first(a[0]);
        const at::Device dev = x.device();
        const at::Tensor &gm = dense(a[1], dev), &w = dense(a[2], dev), &out = dense(a[3], dev);
        need(x.dim() == 2 && w.dim() == 2 && x.scalar_type() == at::kBFloat16);
        const int R = small(x.size(0)), D = small(x.size(1)), F = small(w.size(0) / 2);
        need(shape(gm, {D}) && shape(w, {2 * (int64_t)F, D}) && shape(out, {R, F}));
        const float eps = (float)as_double(a[4]);
        void *st = stream_of(dev), *xp = x.data_ptr(), *gp = gm.data_ptr(), *wp = w.data_ptr(), *op = out.data_ptr();
        RELEASED(g.swiglu(xp, gp, eps, wp, R, D, F, op, st));
    });
}

// bind(addresses of the C entry points in Entry's order, KV, the default workspaces, the raw-stream getter)
PyObject *bind(PyObject *, PyObject *args) {
    PyObject *addr, *kv, *ws, *st;
    if (!PyArg_ParseTuple(args, "O!OO!O", &PyTuple_Type, &addr, &kv, &PyDict_Type, &ws, &st)) return nullptr;
    void *f[sizeof(Entry) / sizeof(void *)];
    const Py_ssize_t n = sizeof(f) / sizeof(f[0]);
    if (PyTuple_GET_SIZE(addr) != n) {
        PyErr_SetString(PyExc_ValueError, "bind: wrong number of entry points");
        return nullptr;
    }
    for (Py_ssize_t i = 0; i < n; ++i) {
        f[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(addr, i));
        if (PyErr_Occurred()) return nullptr;
    }
    memcpy(&g, f, sizeof(g));
    Py_INCREF(kv);
    Py_INCREF(ws);
    Py_INCREF(st);
    Py_XSETREF(g_kv, kv);
    Py_XSETREF(g_ws, ws);
    Py_XSETREF(g_stream, st);
    Py_RETURN_NONE;
}

#define FAST(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {{"bind", bind, METH_VARARGS, nullptr}, FAST(attn), FAST(update), FAST(verify), FAST(verify_vt),
                         FAST(greedy), FAST(stoch), FAST(qkv), FAST(linear), FAST(swiglu), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall(void) {
    s_k = PyUnicode_InternFromString("k");
    s_v = PyUnicode_InternFromString("v");
    s_length = PyUnicode_InternFromString("length");
    s_start = PyUnicode_InternFromString("start");
    s_buf = PyUnicode_InternFromString("buf");
    return PyModule_Create(&module);
}
