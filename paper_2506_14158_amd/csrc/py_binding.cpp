// Python side of the hot calls: argument marshalling of libs4c's entry points straight from torch tensors.
//
// A verification step at batch 1 is a few kernels of a few microseconds each, and marshalling through ctypes (tensor
// properties read one Python attribute at a time, sixteen arguments converted one by one) cost 4-6 us a call, more than
// the launch itself.  Each function here takes the positional arguments of its namesake in binding.py, checks what
// binding.py checks, and calls the C ABI on the current stream.  It returns the library's status code, or kNotMine if
// anything is not as it has to be (a wrong type, shape or device): binding.py then runs its own checks on the same
// arguments and raises.  Nothing is decided here that binding.py would decide differently.
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/core/Tensor.h>
#include <c10/hip/HIPStream.h>

#include "s4c.h"

namespace {

constexpr long kNotMine = 1;
using at::ScalarType;
using at::Tensor;

// Collects arguments; `ok` turns false at the first one that is not as it has to be.
struct Args {
    PyObject* const* v;
    bool ok;
    Args(PyObject* const* args, Py_ssize_t n, Py_ssize_t want) : v(args), ok(n == want) {}
    // argument i as a contiguous device tensor; null if it is not one
    const Tensor* tensor(int i) {
        if (!ok || !THPVariable_Check(v[i])) { ok = false; return nullptr; }
        const Tensor* t = &THPVariable_Unpack(v[i]);
        if (!t->is_cuda() || !t->is_contiguous()) { ok = false; return nullptr; }
        return t;
    }
    const Tensor* tensor(int i, ScalarType type) {
        const Tensor* t = tensor(i);
        if (ok && t->scalar_type() != type) ok = false;
        return t;
    }
    // null for None
    const Tensor* maybe(int i) { return ok && v[i] == Py_None ? nullptr : tensor(i); }
    const Tensor* maybe(int i, ScalarType type) { return ok && v[i] == Py_None ? nullptr : tensor(i, type); }
    long integer(int i) {
        if (!ok) return 0;
        const long x = PyLong_AsLong(v[i]);
        if (x == -1 && PyErr_Occurred()) { PyErr_Clear(); ok = false; }
        if (x != (int32_t)x) ok = false;
        return x;
    }
    float real(int i) {
        if (!ok) return 0.f;
        const double x = PyFloat_AsDouble(v[i]);
        if (x == -1.0 && PyErr_Occurred()) { PyErr_Clear(); ok = false; }
        return (float)x;
    }
    void need(bool c) { ok = ok && c; }
    void shape(const Tensor* t, std::initializer_list<int64_t> s) {
        if (ok) ok = t->sizes().equals(at::IntArrayRef(s.begin(), s.size()));
    }
    void same(const Tensor* t, const Tensor* u) {
        if (ok) ok = t->sizes().equals(u->sizes()) && t->scalar_type() == u->scalar_type();
    }
};

void* ptr(const Tensor* t) { return t ? t->data_ptr() : nullptr; }
size_t bytes(const Tensor* t) { return t ? t->nbytes() : 0; }
void* stream() { return (void*)c10::hip::getCurrentHIPStream().stream(); }
PyObject* answer(long code) { return PyLong_FromLong(code); }
// The launch itself runs without the interpreter lock: it may have to wait for room in a full queue.  Its arguments are
// evaluated by the caller, with the lock: a data pointer or the stream can throw (a tensor without storage, an error of
// the device), which `guarded` catches.
template <class... P, class... A>
PyObject* launch(s4c_status (*entry)(P...), A... args) {
    long code;
    Py_BEGIN_ALLOW_THREADS
    code = entry(args...);
    Py_END_ALLOW_THREADS
    return answer(code);
}
// A C++ exception must not leave a function that the interpreter calls.  Nothing has been launched when one arises, so
// the call is left to binding.py, where the same access raises it as the Python error that it is.
template <PyObject* (*call)(PyObject*, PyObject* const*, Py_ssize_t)>
PyObject* guarded(PyObject* self, PyObject* const* v, Py_ssize_t n) {
    try {
        return call(self, v, n);
    } catch (...) {
        PyErr_Clear();
        return answer(kNotMine);
    }
}

// s4c_dtype of a tensor; -1 (with ok = false) if it has none
int dtype(Args& a, const Tensor* t) {
    if (!a.ok) return -1;
    switch (t->scalar_type()) {
        case ScalarType::Float: return S4C_F32;
        case ScalarType::BFloat16: return S4C_BF16;
        case ScalarType::Half: return S4C_F16;
        default: a.ok = false; return -1;
    }
}

constexpr ScalarType I32 = ScalarType::Int, F32 = ScalarType::Float;

// q [B][N][Hq][D], trees [B][N][Hkv][D], caches / pools of four dimensions
struct AttnTensors {
    const Tensor *q, *kt, *vt, *kc, *vc, *out;
    s4c_attn_shape s;
};
AttnTensors attn_tensors(Args& a, int q, int kt, int kc, int out) {
    AttnTensors t{a.tensor(q), a.tensor(kt), a.tensor(kt + 1), a.tensor(kc), a.tensor(kc + 1), a.tensor(out), {}};
    if (!a.ok || t.q->dim() != 4 || t.kt->dim() != 4 || t.kc->dim() != 4) { a.ok = false; return t; }
    t.s = {(int32_t)t.q->size(0), (int32_t)t.q->size(2), (int32_t)t.kt->size(2), (int32_t)t.q->size(3), (int32_t)t.q->size(1), 0, dtype(a, t.q)};
    a.shape(t.kt, {t.s.B, t.s.N, t.s.Hkv, t.s.D});
    a.same(t.vt, t.kt);
    a.same(t.vc, t.kc);
    a.same(t.out, t.q);
    a.need(a.ok && t.kt->scalar_type() == t.q->scalar_type() && t.kc->scalar_type() == t.q->scalar_type());
    return t;
}

// (q, k_tree, v_tree, k_cache, v_cache, cache_len, parent, max_cache_len, out, scale, status, workspace)
PyObject* tree_attn(PyObject*, PyObject* const* v, Py_ssize_t n) {
    Args a(v, n, 12);
    AttnTensors t = attn_tensors(a, 0, 1, 3, 8);
    const Tensor *len = a.tensor(5, I32), *par = a.tensor(6, I32), *status = a.maybe(10), *ws = a.maybe(11);
    const long mcl = a.integer(7);
    const float scale = a.real(9);
    if (a.ok) {
        t.s.S_cap = (int32_t)t.kc->size(2);
        a.shape(t.kc, {t.s.B, t.s.Hkv, t.s.S_cap, t.s.D});
        a.shape(par, {t.s.B, t.s.N});
    }
    if (!a.ok) return answer(kNotMine);
    return launch(s4c_tree_attn, &t.s, ptr(t.q), ptr(t.kt), ptr(t.vt), ptr(t.kc), ptr(t.vc), (int32_t*)ptr(len), (int32_t*)ptr(par),
                  (int32_t)mcl, scale, ptr(t.out), (int32_t*)ptr(status), ptr(ws), bytes(ws), stream());
}

// (q, k_tree, v_tree, k_pool, v_pool, block_table, cache_len, parent, max_cache_len, out, scale, status, workspace)
PyObject* tree_attn_paged(PyObject*, PyObject* const* v, Py_ssize_t n) {
    Args a(v, n, 13);
    AttnTensors t = attn_tensors(a, 0, 1, 3, 9);
    const Tensor *bt = a.tensor(5, I32), *len = a.tensor(6, I32), *par = a.tensor(7, I32), *status = a.maybe(11), *ws = a.maybe(12);
    const long mcl = a.integer(8);
    const float scale = a.real(10);
    int32_t pages = 0, page = 0, blocks = 0;
    if (a.ok && bt->dim() == 2) {
        pages = (int32_t)t.kc->size(0); page = (int32_t)t.kc->size(2); blocks = (int32_t)bt->size(1);
        t.s.S_cap = blocks * page;
        a.need((int64_t)blocks * page == t.s.S_cap);
        a.shape(t.kc, {pages, t.s.Hkv, page, t.s.D});
        a.shape(bt, {t.s.B, blocks});
    } else a.ok = false;
    if (!a.ok) return answer(kNotMine);
    return launch(s4c_tree_attn_paged, &t.s, ptr(t.q), ptr(t.kt), ptr(t.vt), ptr(t.kc), ptr(t.vc), (int32_t*)ptr(bt), blocks, page, pages,
                  (int32_t*)ptr(len), (int32_t*)ptr(par), (int32_t)mcl, scale, ptr(t.out), (int32_t*)ptr(status),
                  ptr(ws), bytes(ws), stream());
}

// the tensors that both acceptance entry points take
struct AcceptTensors {
    const Tensor *logits, *par, *tok, *path, *len, *acc, *bonus, *pd, *u, *status;
    int32_t B, N, V, dt;
    long mode, max_path;
    float temperature;
};
// (logits, parent, tokens, mode, max_path, path, accept_len, accepted_tokens, bonus_token, p_draft, uniforms, temperature, status)
AcceptTensors accept_tensors(Args& a) {
    AcceptTensors t{a.tensor(0), a.tensor(1, I32), a.tensor(2, I32), a.tensor(5, I32), a.tensor(6, I32), a.tensor(7, I32), a.tensor(8, I32),
                    a.maybe(9, F32), a.maybe(10, F32), a.maybe(12), 0, 0, 0, 0, a.integer(3), a.integer(4), a.real(11)};
    t.dt = dtype(a, t.logits);
    if (!a.ok || t.logits->dim() != 3) { a.ok = false; return t; }
    t.B = (int32_t)t.logits->size(0); t.N = (int32_t)t.logits->size(1); t.V = (int32_t)t.logits->size(2);
    a.shape(t.par, {t.B, t.N});
    a.shape(t.tok, {t.B, t.N});
    a.shape(t.path, {t.B, t.max_path});
    a.shape(t.acc, {t.B, t.max_path});
    if (t.pd) a.shape(t.pd, {t.B, t.N});
    if (t.u) a.shape(t.u, {t.B, t.N});
    return t;
}

// (..., workspace)
PyObject* accept_path(PyObject*, PyObject* const* v, Py_ssize_t n) {
    Args a(v, n, 14);
    const AcceptTensors t = accept_tensors(a);
    const Tensor* ws = a.maybe(13);
    if (!a.ok) return answer(kNotMine);
    return launch(s4c_accept_path, t.B, t.N, t.V, t.dt, (int32_t)t.mode, t.temperature, ptr(t.logits), (int32_t*)ptr(t.par), (int32_t*)ptr(t.tok),
                  (float*)ptr(t.pd), (float*)ptr(t.u), (int32_t)t.max_path, (int32_t*)ptr(t.path), (int32_t*)ptr(t.len),
                  (int32_t*)ptr(t.acc), (int32_t*)ptr(t.bonus), (int32_t*)ptr(t.status), ptr(ws), bytes(ws), stream());
}

PyObject* accept_path_static(PyObject*, PyObject* const* v, Py_ssize_t n) {
    Args a(v, n, 13);
    const AcceptTensors t = accept_tensors(a);
    if (!a.ok) return answer(kNotMine);
    return launch(s4c_accept_path_static, t.B, t.N, t.V, t.dt, (int32_t)t.mode, t.temperature, ptr(t.logits), (int32_t*)ptr(t.par),
                  (int32_t*)ptr(t.tok), (float*)ptr(t.pd), (float*)ptr(t.u), (int32_t)t.max_path,
                  (int32_t*)ptr(t.path), (int32_t*)ptr(t.len), (int32_t*)ptr(t.acc), (int32_t*)ptr(t.bonus),
                  (int32_t*)ptr(t.status), stream());
}

// (logits, draft_probs, parent, tokens, uniforms, u_resample, max_path, path, accept_len, accepted_tokens, bonus_token, workspace,
//  temperature, status)
PyObject* accept_resample(PyObject*, PyObject* const* v, Py_ssize_t n) {
    Args a(v, n, 14);
    const Tensor *lg = a.tensor(0), *dp = a.tensor(1, F32), *par = a.tensor(2, I32), *tok = a.tensor(3, I32), *u = a.tensor(4, F32),
                 *ur = a.tensor(5, F32), *path = a.tensor(7, I32), *len = a.tensor(8, I32), *acc = a.tensor(9, I32), *bonus = a.tensor(10, I32),
                 *ws = a.maybe(11), *status = a.maybe(13);
    const long mp = a.integer(6);
    const float temperature = a.real(12);
    const int dt = dtype(a, lg);
    if (!a.ok || lg->dim() != 3) return answer(kNotMine);
    const int64_t B = lg->size(0), N = lg->size(1), V = lg->size(2);
    a.shape(dp, {B, N, V});
    a.shape(par, {B, N});
    a.shape(tok, {B, N});
    a.shape(u, {B, N});
    a.shape(ur, {B});
    a.shape(path, {B, mp});
    a.shape(acc, {B, mp});
    if (!a.ok) return answer(kNotMine);
    return launch(s4c_accept_resample, (int32_t)B, (int32_t)N, (int32_t)V, dt, temperature, ptr(lg), (float*)ptr(dp), (int32_t*)ptr(par),
                  (int32_t*)ptr(tok), (float*)ptr(u), (float*)ptr(ur), (int32_t)mp, (int32_t*)ptr(path), (int32_t*)ptr(len),
                  (int32_t*)ptr(acc), (int32_t*)ptr(bonus), (int32_t*)ptr(status), ptr(ws), bytes(ws), stream());
}

// (k_tree, v_tree, k_cache, v_cache, cache_len, path, accept_len, dst_index, status)
PyObject* kv_compact(PyObject*, PyObject* const* v, Py_ssize_t n) {
    Args a(v, n, 9);
    const Tensor *kt = a.tensor(0), *vt = a.tensor(1), *kc = a.tensor(2), *vc = a.tensor(3), *len = a.tensor(4, I32), *path = a.tensor(5, I32),
                 *alen = a.tensor(6, I32), *dst = a.maybe(7), *status = a.maybe(8);
    const int dt = dtype(a, kt);
    if (!a.ok || kt->dim() != 4 || kc->dim() != 4 || path->dim() != 2) return answer(kNotMine);
    const s4c_attn_shape s = {(int32_t)kt->size(0), (int32_t)kt->size(2), (int32_t)kt->size(2), (int32_t)kt->size(3), (int32_t)kt->size(1),
                              (int32_t)kc->size(2), dt};
    a.shape(kc, {s.B, s.Hkv, s.S_cap, s.D});
    a.same(vt, kt);
    a.same(vc, kc);
    a.need(kc->scalar_type() == kt->scalar_type());
    if (!a.ok) return answer(kNotMine);
    return launch(s4c_kv_compact, &s, ptr(kt), ptr(vt), ptr(kc), ptr(vc), (int32_t*)ptr(len), (int32_t*)ptr(path), (int32_t*)ptr(alen),
                  (int32_t)path->size(1), (int32_t*)ptr(dst), (int32_t*)ptr(status), stream());
}

// (k_tree, v_tree, k_pool, v_pool, block_table, cache_len, path, accept_len, dst_index, status)
PyObject* kv_compact_paged(PyObject*, PyObject* const* v, Py_ssize_t n) {
    Args a(v, n, 10);
    const Tensor *kt = a.tensor(0), *vt = a.tensor(1), *kc = a.tensor(2), *vc = a.tensor(3), *bt = a.tensor(4, I32), *len = a.tensor(5, I32),
                 *path = a.tensor(6, I32), *alen = a.tensor(7, I32), *dst = a.maybe(8), *status = a.maybe(9);
    const int dt = dtype(a, kt);
    if (!a.ok || kt->dim() != 4 || kc->dim() != 4 || bt->dim() != 2 || path->dim() != 2) return answer(kNotMine);
    const int32_t pages = (int32_t)kc->size(0), page = (int32_t)kc->size(2), blocks = (int32_t)bt->size(1);
    const s4c_attn_shape s = {(int32_t)kt->size(0), (int32_t)kt->size(2), (int32_t)kt->size(2), (int32_t)kt->size(3), (int32_t)kt->size(1),
                              blocks * page, dt};
    a.need((int64_t)blocks * page == s.S_cap);
    a.shape(kc, {pages, s.Hkv, page, s.D});
    a.shape(bt, {s.B, blocks});
    a.same(vt, kt);
    a.same(vc, kc);
    a.need(kc->scalar_type() == kt->scalar_type());
    if (!a.ok) return answer(kNotMine);
    return launch(s4c_kv_compact_paged, &s, ptr(kt), ptr(vt), ptr(kc), ptr(vc), (int32_t*)ptr(bt), blocks, page, pages, (int32_t*)ptr(len),
                  (int32_t*)ptr(path), (int32_t*)ptr(alen), (int32_t)path->size(1), (int32_t*)ptr(dst),
                  (int32_t*)ptr(status), stream());
}

// bytes of a feature row; features [B][N][...] and features_out [B][max_path][...] go together
int64_t feature_bytes(Args& a, const Tensor* f, const Tensor* fo, int64_t B, int64_t N, int64_t mp) {
    if (!a.ok || (!f && !fo)) return 0;
    if (!f || !fo || f->scalar_type() != fo->scalar_type() || f->dim() < 2 || fo->dim() != f->dim() || f->size(0) != B || f->size(1) != N ||
        fo->size(0) != B || fo->size(1) != mp || !f->sizes().slice(2).equals(fo->sizes().slice(2)) || B == 0 || N == 0) {
        a.ok = false;
        return 0;
    }
    const int64_t n = f->nbytes() / (B * N);
    a.need(n == (int32_t)n);
    return n;
}

// (k_tree, v_tree, k_cache, v_cache, cache_len, path, accept_len, features, features_out, dst_index, status)
PyObject* commit_path(PyObject*, PyObject* const* v, Py_ssize_t n) {
    Args a(v, n, 11);
    const Tensor *kt = a.tensor(0), *vt = a.tensor(1), *kc = a.tensor(2), *vc = a.tensor(3), *len = a.tensor(4, I32), *path = a.tensor(5, I32),
                 *alen = a.tensor(6, I32), *f = a.maybe(7), *fo = a.maybe(8), *dst = a.maybe(9), *status = a.maybe(10);
    const int dt = dtype(a, kt);
    if (!a.ok || kt->dim() != 5 || kc->dim() != 5 || path->dim() != 2) return answer(kNotMine);
    const s4c_attn_shape s = {(int32_t)kt->size(1), (int32_t)kt->size(3), (int32_t)kt->size(3), (int32_t)kt->size(4), (int32_t)kt->size(2),
                              (int32_t)kc->size(3), dt};
    a.shape(kc, {kt->size(0), s.B, s.Hkv, s.S_cap, s.D});
    a.same(vt, kt);
    a.same(vc, kc);
    a.need(kc->scalar_type() == kt->scalar_type());
    const int64_t fb = feature_bytes(a, f, fo, s.B, s.N, path->size(1));
    if (!a.ok) return answer(kNotMine);
    return launch(s4c_commit_path, &s, (int32_t)kt->size(0), ptr(kt), ptr(vt), ptr(kc), ptr(vc), (int32_t*)ptr(len), (int32_t*)ptr(path),
                  (int32_t*)ptr(alen), (int32_t)path->size(1), ptr(f), (int32_t)fb, ptr(fo), (int32_t*)ptr(dst),
                  (int32_t*)ptr(status), stream());
}

// (k_tree, v_tree, k_pool, v_pool, block_table, cache_len, path, accept_len, features, features_out, dst_index, status)
PyObject* commit_path_paged(PyObject*, PyObject* const* v, Py_ssize_t n) {
    Args a(v, n, 12);
    const Tensor *kt = a.tensor(0), *vt = a.tensor(1), *kc = a.tensor(2), *vc = a.tensor(3), *bt = a.tensor(4, I32), *len = a.tensor(5, I32),
                 *path = a.tensor(6, I32), *alen = a.tensor(7, I32), *f = a.maybe(8), *fo = a.maybe(9), *dst = a.maybe(10), *status = a.maybe(11);
    const int dt = dtype(a, kt);
    if (!a.ok || kt->dim() != 5 || kc->dim() != 5 || bt->dim() != 2 || path->dim() != 2) return answer(kNotMine);
    const int32_t pages = (int32_t)kc->size(1), page = (int32_t)kc->size(3), blocks = (int32_t)bt->size(1);
    const s4c_attn_shape s = {(int32_t)kt->size(1), (int32_t)kt->size(3), (int32_t)kt->size(3), (int32_t)kt->size(4), (int32_t)kt->size(2),
                              blocks * page, dt};
    a.need((int64_t)blocks * page == s.S_cap);
    a.shape(kc, {kt->size(0), pages, s.Hkv, page, s.D});
    a.shape(bt, {s.B, blocks});
    a.same(vt, kt);
    a.same(vc, kc);
    a.need(kc->scalar_type() == kt->scalar_type());
    const int64_t fb = feature_bytes(a, f, fo, s.B, s.N, path->size(1));
    if (!a.ok) return answer(kNotMine);
    return launch(s4c_commit_path_paged, &s, (int32_t)kt->size(0), ptr(kt), ptr(vt), ptr(kc), ptr(vc), (int32_t*)ptr(bt), blocks, page, pages,
                  (int32_t*)ptr(len), (int32_t*)ptr(path), (int32_t*)ptr(alen), (int32_t)path->size(1), ptr(f),
                  (int32_t)fb, ptr(fo), (int32_t*)ptr(dst), (int32_t*)ptr(status), stream());
}

// (draft_logits, nchild, root_token, kmax, parent, tokens, p_draft, workspace, temperature, level, status)
PyObject* build_tree(PyObject*, PyObject* const* v, Py_ssize_t n) {
    Args a(v, n, 11);
    const Tensor *lg = a.tensor(0), *nc = a.tensor(1, I32), *root = a.tensor(2, I32), *par = a.tensor(4, I32), *tok = a.tensor(5, I32),
                 *pd = a.tensor(6, F32), *ws = a.maybe(7), *level = a.maybe(9, I32), *status = a.maybe(10);
    const long kmax = a.integer(3);
    const float temperature = a.real(8);
    const int dt = dtype(a, lg);
    if (!a.ok || lg->dim() != 3) return answer(kNotMine);
    const int64_t B = lg->size(0), N = lg->size(1);
    a.shape(nc, {B, N});
    a.shape(root, {B});
    a.shape(par, {B, N});
    a.shape(tok, {B, N});
    a.shape(pd, {B, N});
    if (level) a.shape(level, {B, N});
    if (!a.ok) return answer(kNotMine);
    return launch(s4c_build_tree, (int32_t)B, (int32_t)N, (int32_t)lg->size(2), dt, temperature, ptr(lg), (int32_t*)ptr(nc), (int32_t*)ptr(root),
                  (int32_t)kmax, (int32_t*)ptr(par), (int32_t*)ptr(tok), (float*)ptr(pd), (int32_t*)ptr(level),
                  (int32_t*)ptr(status), ptr(ws), bytes(ws), stream());
}

// (e, f, W, out, bias, workspace)
PyObject* draft_linear(PyObject*, PyObject* const* v, Py_ssize_t n) {
    Args a(v, n, 6);
    const Tensor *e = a.tensor(0), *f = a.tensor(1), *W = a.tensor(2), *out = a.tensor(3), *bias = a.maybe(4), *ws = a.maybe(5);
    const int dt = dtype(a, e);
    if (!a.ok || dt == S4C_F32 || e->dim() != 2 || W->dim() != 2) return answer(kNotMine);
    const int64_t T = e->size(0), H = e->size(1), Hout = W->size(0);
    a.same(f, e);
    a.shape(W, {Hout, 2 * H});
    a.shape(out, {T, Hout});
    a.need(W->scalar_type() == e->scalar_type() && out->scalar_type() == e->scalar_type());
    if (bias) {
        a.shape(bias, {Hout});
        a.need(bias->scalar_type() == e->scalar_type());
    }
    if (!a.ok) return answer(kNotMine);
    return launch(s4c_draft_linear, (int32_t)T, (int32_t)H, (int32_t)Hout, dt, ptr(e), ptr(f), ptr(W), ptr(bias), ptr(out), ptr(ws), bytes(ws),
                  stream());
}

// (q, k_tree, v_tree, k_cache, v_cache, cache_len, parent, logits, tokens, mode, p_draft, uniforms, temperature, scale,
//  out, attn_status, attn_workspace, path, accept_len, accepted_tokens, bonus_token, accept_status, accept_workspace,
//  dst_index, compact_status, max_cache_len, max_path)
PyObject* verify_step(PyObject*, PyObject* const* v, Py_ssize_t n) {
    Args a(v, n, 27);
    const AttnTensors t = attn_tensors(a, 0, 1, 3, 14);
    const Tensor *len = a.tensor(5, I32), *par = a.tensor(6, I32), *lg = a.tensor(7), *tok = a.tensor(8, I32), *pd = a.maybe(10, F32),
                 *u = a.maybe(11, F32), *ast = a.maybe(15), *aws = a.maybe(16), *path = a.tensor(17, I32), *alen = a.tensor(18, I32),
                 *acc = a.tensor(19, I32), *bonus = a.tensor(20, I32), *cst = a.maybe(21), *cws = a.maybe(22), *dst = a.maybe(23),
                 *kst = a.maybe(24);
    s4c_step p{};
    p.mode = (int32_t)a.integer(9);
    p.temperature = a.real(12);
    p.scale = a.real(13);
    p.max_cache_len = (int32_t)a.integer(25);
    p.max_path = (int32_t)a.integer(26);
    p.logits_dtype = dtype(a, lg);
    if (!a.ok || lg->dim() != 3) return answer(kNotMine);
    p.shape = t.s;
    p.shape.S_cap = (int32_t)t.kc->size(2);
    p.V = (int32_t)lg->size(2);
    a.shape(t.kc, {t.s.B, t.s.Hkv, p.shape.S_cap, t.s.D});
    a.shape(lg, {t.s.B, t.s.N, p.V});
    a.shape(par, {t.s.B, t.s.N});
    a.shape(tok, {t.s.B, t.s.N});
    if (pd) a.shape(pd, {t.s.B, t.s.N});
    if (u) a.shape(u, {t.s.B, t.s.N});
    a.shape(path, {t.s.B, p.max_path});
    a.shape(acc, {t.s.B, p.max_path});
    if (!a.ok) return answer(kNotMine);
    p.q = ptr(t.q); p.k_tree = ptr(t.kt); p.v_tree = ptr(t.vt); p.k_cache = ptr(t.kc); p.v_cache = ptr(t.vc);
    p.cache_len = (int32_t*)ptr(len); p.parent = (int32_t*)ptr(par); p.tokens = (int32_t*)ptr(tok); p.logits = ptr(lg);
    p.p_draft = (float*)ptr(pd); p.uniforms = (float*)ptr(u); p.out = ptr(t.out); p.path = (int32_t*)ptr(path);
    p.accept_len = (int32_t*)ptr(alen); p.accepted_tokens = (int32_t*)ptr(acc); p.bonus_token = (int32_t*)ptr(bonus);
    p.dst_index = (int32_t*)ptr(dst); p.attn_status = (int32_t*)ptr(ast); p.accept_status = (int32_t*)ptr(cst);
    p.compact_status = (int32_t*)ptr(kst); p.attn_workspace = ptr(aws); p.accept_workspace = ptr(cws);
    p.attn_workspace_bytes = bytes(aws); p.accept_workspace_bytes = bytes(cws);
    return launch(s4c_verify_step, &p, stream());
}

#define S4C_PY(name) {#name, (PyCFunction)(void (*)(void))guarded<name>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {S4C_PY(tree_attn), S4C_PY(tree_attn_paged), S4C_PY(accept_path), S4C_PY(accept_path_static),
                         S4C_PY(accept_resample), S4C_PY(kv_compact), S4C_PY(kv_compact_paged), S4C_PY(commit_path),
                         S4C_PY(commit_path_paged), S4C_PY(build_tree), S4C_PY(draft_linear), S4C_PY(verify_step), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_s4c_py", "libs4c's entry points on torch tensors", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__s4c_py(void) { return PyModule_Create(&module); }
