// Argument marshalling of the Python binding in native code: a call hands over a dozen tensors, and taking each apart in
// Python (type, device, shape, contiguity, address) cost 12 to 20 us per call, as long as the kernels of a small call run.
//
// Every function here is the quick way through a method of binding.Tapout: it looks at the arguments exactly as the Python
// code does and, if all of them are in order, calls the library and returns its status.  At anything unusual (another type,
// a tensor subclass, a wrong shape or device, a missing output) it returns None before anything is called, and the Python
// code, which describes errors, takes over.  No results, addresses or tensors are kept.
#include <torch/csrc/autograd/python_variable.h>
#include <c10/hip/HIPStream.h>
#include <dlfcn.h>

#include "tapout.h"

namespace {

struct Library {
    decltype(&tapout_bandit_select) bandit_select;
    decltype(&tapout_draft_stats) draft_stats;
    decltype(&tapout_verify) verify;
    decltype(&tapout_bandit_update) bandit_update;
    decltype(&tapout_bandit_update_select) bandit_update_select;
    decltype(&tapout_shard_stats) shard_stats;
    decltype(&tapout_draft_stats_sharded) draft_stats_sharded;
    decltype(&tapout_verify_accept_sharded) verify_accept_sharded;
    decltype(&tapout_shard_final_sums) shard_final_sums;
    decltype(&tapout_shard_final_token) shard_final_token;
} g_lib = {};

constexpr auto kF32 = at::kFloat, kF64 = at::kDouble, kI32 = at::kInt, kU8 = at::kByte;

// Collects the arguments of one call; `ok` turns false at the first one that is not in order.
struct Args {
    bool ok = true;

    const at::Tensor *tensor(PyObject *o)
    {
        if (!ok || !THPVariable_CheckExact(o)) { ok = false; return nullptr; }
        const at::Tensor &t = THPVariable_Unpack(o);
        if (!t.is_cuda()) { ok = false; return nullptr; }
        return &t;
    }
    // address of a contiguous tensor of this type and shape; NULL for None
    template <class T = void>
    T *ptr(PyObject *o, at::ScalarType type, std::initializer_list<int64_t> shape)
    {
        if (!o || o == Py_None) return nullptr;
        const at::Tensor *t = tensor(o);
        if (!t || t->scalar_type() != type || t->sizes() != at::IntArrayRef(shape) || !t->is_contiguous()) { ok = false; return nullptr; }
        return (T *)t->data_ptr();
    }
    template <class T = void>
    T *required(PyObject *o, at::ScalarType type, std::initializer_list<int64_t> shape)
    {
        if (!o || o == Py_None) { ok = false; return nullptr; }
        return ptr<T>(o, type, shape);
    }
    // entry of the dict of outputs (absent or None: NULL)
    template <class T = void>
    T *out(PyObject *dict, const char *key, at::ScalarType type, std::initializer_list<int64_t> shape)
    {
        return ok ? ptr<T>(PyDict_GetItemString(dict, key), type, shape) : nullptr;
    }
    template <class T = void>
    T *need(PyObject *dict, const char *key, at::ScalarType type, std::initializer_list<int64_t> shape)
    {
        return ok ? required<T>(PyDict_GetItemString(dict, key), type, shape) : nullptr;
    }
    tapout_logits logits(PyObject *o, int64_t *B, int64_t *K, int64_t *V)
    {
        tapout_logits l = {};
        const at::Tensor *t = tensor(o);
        if (!t || t->dim() != 3 || (t->size(2) > 1 && t->stride(2) != 1)) { ok = false; return l; }
        if (t->scalar_type() == kF32) l.dtype = TAPOUT_F32;
        else if (t->scalar_type() == at::kBFloat16) l.dtype = TAPOUT_BF16;
        else { ok = false; return l; }
        l.ptr = t->data_ptr(); l.stride_b = t->stride(0); l.stride_k = t->stride(1);
        *B = t->size(0); *K = t->size(1); *V = t->size(2);
        if (*B > INT32_MAX || *K > INT32_MAX || *V > INT32_MAX) ok = false;
        return l;
    }
    int64_t integer(PyObject *o)
    {
        if (!ok || !PyLong_CheckExact(o)) { ok = false; return 0; }
        const int64_t v = PyLong_AsLongLong(o);
        if (PyErr_Occurred()) { PyErr_Clear(); ok = false; }
        return v;
    }
    int32_t i32(PyObject *o)
    {
        const int64_t v = integer(o);
        if (v < INT32_MIN || v > INT32_MAX) ok = false;
        return (int32_t)v;
    }
    tapout_ctx *ctx(PyObject *o)
    {
        if (!ok || !PyLong_CheckExact(o)) { ok = false; return nullptr; }
        void *p = PyLong_AsVoidPtr(o);
        if (PyErr_Occurred()) PyErr_Clear();
        if (!p) ok = false;
        return (tapout_ctx *)p;
    }
    PyObject *dict(PyObject *o)
    {
        if (!ok || !PyDict_CheckExact(o)) ok = false;
        return o;
    }
    // None: the current stream of the current device
    void *stream(PyObject *o)
    {
        if (!ok) return nullptr;
        if (o == Py_None) return (void *)c10::hip::getCurrentHIPStream().stream();
        void *p = PyLong_Check(o) ? PyLong_AsVoidPtr(o) : nullptr;
        if (!PyLong_Check(o) || PyErr_Occurred()) { PyErr_Clear(); ok = false; }
        return p;
    }
};

// The library call without the interpreter lock (as ctypes does), its status as the Python result.  An exception out of the
// library is a Python exception, raised with the lock held; None would have the Python code make the call a second time.
template <class F>
PyObject *call(const Args &a, F f)
{
    if (!a.ok) Py_RETURN_NONE;
    tapout_status st = TAPOUT_OK;
    char thrown[256] = "";
    PyThreadState *ts = PyEval_SaveThread();
    try {
        st = f();
    } catch (const std::exception &e) {
        snprintf(thrown, sizeof thrown, "%s", *e.what() ? e.what() : "C++ exception");
    } catch (...) {
        snprintf(thrown, sizeof thrown, "C++ exception");
    }
    PyEval_RestoreThread(ts);
    if (*thrown) { PyErr_SetString(PyExc_RuntimeError, thrown); return nullptr; }
    return PyLong_FromLong((long)st);
}

// fn(args, n) with C++ exceptions turned into "take the Python way".
template <PyObject *(*FN)(PyObject *const *), int N>
PyObject *entry(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != N || !g_lib.verify) Py_RETURN_NONE;
    try {
        return FN(args);
    } catch (...) {
        if (PyErr_Occurred()) PyErr_Clear();
        Py_RETURN_NONE;
    }
}

// (ctx, B, positions, n_arms, u_ts, arm_out, flags, stream)
PyObject *bandit_select(PyObject *const *p)
{
    Args a;
    tapout_ctx *c = a.ctx(p[0]);
    const int64_t B = a.i32(p[1]), P = a.integer(p[2]), A = a.integer(p[3]);
    const float *u = P == 1 ? a.ptr<float>(p[4], kF32, {B, A, TAPOUT_TS_UNIFORMS_PER_ARM}) : a.ptr<float>(p[4], kF32, {B, P, A, TAPOUT_TS_UNIFORMS_PER_ARM});
    int32_t *arm = P == 1 ? a.required<int32_t>(p[5], kI32, {B}) : a.required<int32_t>(p[5], kI32, {B, P});
    uint32_t *flags = a.ptr<uint32_t>(p[6], kI32, {B});
    void *st = a.stream(p[7]);
    return call(a, [&] { return g_lib.bandit_select(c, (int32_t)B, u, arm, flags, st); });
}

struct DraftOut {
    float *lse, *entropy, *p_top1, *p_top2, *margin, *logq; int32_t *top1, *n_stop; uint8_t *fired; uint32_t *flags;
};
DraftOut draft_out(Args &a, PyObject *out, int64_t B, int64_t K, bool tokens, bool arms)
{
    DraftOut o = {};
    o.lse = a.out<float>(out, "lse", kF32, {B, K}); o.entropy = a.out<float>(out, "entropy", kF32, {B, K});
    o.p_top1 = a.out<float>(out, "p_top1", kF32, {B, K}); o.p_top2 = a.out<float>(out, "p_top2", kF32, {B, K});
    o.margin = a.out<float>(out, "margin", kF32, {B, K}); o.top1 = a.out<int32_t>(out, "top1_id", kI32, {B, K});
    if (tokens) o.logq = a.out<float>(out, "logq_tok", kF32, {B, K});
    if (arms) { o.n_stop = a.out<int32_t>(out, "n_stop", kI32, {B}); o.fired = a.out<uint8_t>(out, "stop_fired", kU8, {B, K}); }
    o.flags = a.out<uint32_t>(out, "flags", kI32, {B});
    return o;
}

// (ctx, positions, draft, draft_tok, k_len, arm, u_draft, out, stream)
PyObject *draft_stats(PyObject *const *p)
{
    Args a;
    tapout_ctx *c = a.ctx(p[0]);
    const int64_t P = a.integer(p[1]);
    int64_t B = 0, K = 0, V = 0;
    const tapout_logits l = a.logits(p[2], &B, &K, &V);
    const int32_t *tok = a.ptr<int32_t>(p[3], kI32, {B, K}), *k_len = a.ptr<int32_t>(p[4], kI32, {B});
    const int32_t *arm = P == 1 ? a.ptr<int32_t>(p[5], kI32, {B}) : a.ptr<int32_t>(p[5], kI32, {B, P});
    const float *u = a.ptr<float>(p[6], kF32, {B, K});
    PyObject *out = a.dict(p[7]);
    if (!a.ok) Py_RETURN_NONE;
    const DraftOut o = draft_out(a, out, B, K, p[3] != Py_None || p[6] != Py_None, p[5] != Py_None);
    int32_t *sampled = p[6] != Py_None ? a.out<int32_t>(out, "sampled_tok", kI32, {B, K}) : nullptr;
    void *st = a.stream(p[8]);
    return call(a, [&] {
        return g_lib.draft_stats(c, &l, (int32_t)B, (int32_t)K, (int32_t)V, tok, k_len, arm, u, o.lse, o.entropy, o.p_top1, o.p_top2, o.margin,
                                 o.top1, o.logq, sampled, o.n_stop, o.fired, o.flags, st);
    });
}

// (ctx, target, draft, draft_lse, logq_tok, draft_tok, n_draft, u_accept, u_sample, greedy, out, stream)
PyObject *verify(PyObject *const *p)
{
    Args a;
    tapout_ctx *c = a.ctx(p[0]);
    int64_t B = 0, K1 = 0, V = 0, Bd = 0, K = 0, Vd = 0;
    const tapout_logits t = a.logits(p[1], &B, &K1, &V), d = a.logits(p[2], &Bd, &K, &Vd);
    if (Bd != B || K != K1 - 1 || Vd != V) a.ok = false;
    const float *dl = a.ptr<float>(p[3], kF32, {B, K}), *lq = a.ptr<float>(p[4], kF32, {B, K});
    const int32_t *tok = a.ptr<int32_t>(p[5], kI32, {B, K}), *n = a.ptr<int32_t>(p[6], kI32, {B});
    const float *ua = a.ptr<float>(p[7], kF32, {B, K}), *us = a.ptr<float>(p[8], kF32, {B});
    const uint8_t *greedy = a.ptr<uint8_t>(p[9], kU8, {B});
    PyObject *out = a.dict(p[10]);
    if (!a.ok) Py_RETURN_NONE;
    int32_t *al = a.need<int32_t>(out, "accept_len", kI32, {B}), *ot = a.need<int32_t>(out, "out_tok", kI32, {B, K1}), *no = a.need<int32_t>(out, "n_out", kI32, {B});
    float *tl = a.out<float>(out, "target_lse", kF32, {B, K1}), *lp = a.out<float>(out, "logp_tok", kF32, {B, K});
    int32_t *t1 = a.out<int32_t>(out, "target_top1", kI32, {B, K1});
    uint32_t *fl = a.out<uint32_t>(out, "flags", kI32, {B});
    void *st = a.stream(p[11]);
    return call(a, [&] {
        return g_lib.verify(c, &t, &d, (int32_t)B, (int32_t)K, (int32_t)V, dl, lq, tok, n, greedy, ua, us, al, ot, no, tl, lp, t1, fl, st);
    });
}

// (ctx, B, positions, arm, accept_len, n_draft, gamma, active, stream)
PyObject *bandit_update(PyObject *const *p)
{
    Args a;
    tapout_ctx *c = a.ctx(p[0]);
    const int64_t B = a.i32(p[1]), P = a.integer(p[2]);
    const int32_t *arm = P == 1 ? a.ptr<int32_t>(p[3], kI32, {B}) : a.ptr<int32_t>(p[3], kI32, {B, P});
    const int32_t *al = a.ptr<int32_t>(p[4], kI32, {B}), *n = a.ptr<int32_t>(p[5], kI32, {B}), *g = a.ptr<int32_t>(p[6], kI32, {B});
    const uint8_t *act = a.ptr<uint8_t>(p[7], kU8, {B});
    void *st = a.stream(p[8]);
    return call(a, [&] { return g_lib.bandit_update(c, (int32_t)B, arm, al, n, g, act, st); });
}

// (ctx, B, positions, n_arms, arm, accept_len, n_draft, gamma, active, u_ts, arm_out, flags, stream)
PyObject *bandit_update_select(PyObject *const *p)
{
    Args a;
    tapout_ctx *c = a.ctx(p[0]);
    const int64_t B = a.i32(p[1]), P = a.integer(p[2]), A = a.integer(p[3]);
    const int32_t *arm = P == 1 ? a.ptr<int32_t>(p[4], kI32, {B}) : a.ptr<int32_t>(p[4], kI32, {B, P});
    const int32_t *al = a.ptr<int32_t>(p[5], kI32, {B}), *n = a.ptr<int32_t>(p[6], kI32, {B}), *g = a.ptr<int32_t>(p[7], kI32, {B});
    const uint8_t *act = a.ptr<uint8_t>(p[8], kU8, {B});
    const float *u = P == 1 ? a.ptr<float>(p[9], kF32, {B, A, TAPOUT_TS_UNIFORMS_PER_ARM}) : a.ptr<float>(p[9], kF32, {B, P, A, TAPOUT_TS_UNIFORMS_PER_ARM});
    int32_t *ao = P == 1 ? a.required<int32_t>(p[10], kI32, {B}) : a.required<int32_t>(p[10], kI32, {B, P});
    uint32_t *fl = a.ptr<uint32_t>(p[11], kI32, {B});
    void *st = a.stream(p[12]);
    return call(a, [&] { return g_lib.bandit_update_select(c, (int32_t)B, arm, al, n, g, act, u, ao, fl, st); });
}

// (ctx, shard, vocab_offset, length, rows_mode, tok, out, stream)
PyObject *shard_stats(PyObject *const *p)
{
    Args a;
    tapout_ctx *c = a.ctx(p[0]);
    int64_t B = 0, KK = 0, Vs = 0;
    const tapout_logits l = a.logits(p[1], &B, &KK, &Vs);
    const int32_t off = a.i32(p[2]), mode = a.i32(p[4]);
    const int32_t *len = a.ptr<int32_t>(p[3], kI32, {B}), *tok = a.ptr<int32_t>(p[5], kI32, {B, KK - mode});
    auto *out = a.required<tapout_shard_stat>(p[6], kI32, {B * KK, 8});
    void *st = a.stream(p[7]);
    return call(a, [&] { return g_lib.shard_stats(c, &l, (int32_t)B, (int32_t)KK, (int32_t)Vs, off, len, mode, tok, out, st); });
}

// records of all shards, [G, rows, 8]
const tapout_shard_stat *records(Args &a, PyObject *o, int64_t rows, int64_t *G)
{
    const at::Tensor *t = a.tensor(o);
    if (!t || t->dim() != 3) { a.ok = false; return nullptr; }
    *G = t->size(0);
    return a.required<tapout_shard_stat>(o, kI32, {*G, rows, 8});
}

// (ctx, positions, stats, B, K, V, draft_tok, k_len, arm, out, stream)
PyObject *draft_stats_sharded(PyObject *const *p)
{
    Args a;
    tapout_ctx *c = a.ctx(p[0]);
    const int64_t P = a.integer(p[1]), B = a.i32(p[3]), K = a.i32(p[4]);
    const int32_t V = a.i32(p[5]);
    int64_t G = 0;
    const tapout_shard_stat *s = records(a, p[2], B * K, &G);
    const int32_t *tok = a.ptr<int32_t>(p[6], kI32, {B, K}), *k_len = a.ptr<int32_t>(p[7], kI32, {B});
    const int32_t *arm = P == 1 ? a.ptr<int32_t>(p[8], kI32, {B}) : a.ptr<int32_t>(p[8], kI32, {B, P});
    PyObject *out = a.dict(p[9]);
    if (!a.ok) Py_RETURN_NONE;
    const DraftOut o = draft_out(a, out, B, K, p[6] != Py_None, p[8] != Py_None);
    void *st = a.stream(p[10]);
    return call(a, [&] {
        return g_lib.draft_stats_sharded(c, s, (int32_t)G, (int32_t)B, (int32_t)K, V, tok, k_len, arm, o.lse, o.entropy, o.p_top1, o.p_top2, o.margin,
                                         o.top1, o.logq, o.n_stop, o.fired, o.flags, st);
    });
}

// (ctx, stats, B, K, V, logq_tok, draft_tok, n_draft, u_accept, greedy, draft_lse, out, stream)
PyObject *verify_accept_sharded(PyObject *const *p)
{
    Args a;
    tapout_ctx *c = a.ctx(p[0]);
    const int64_t B = a.i32(p[2]), K = a.i32(p[3]);
    const int32_t V = a.i32(p[4]);
    int64_t G = 0;
    const tapout_shard_stat *s = records(a, p[1], B * (K + 1), &G);
    const float *lq = a.ptr<float>(p[5], kF32, {B, K});
    const int32_t *tok = a.ptr<int32_t>(p[6], kI32, {B, K}), *n = a.ptr<int32_t>(p[7], kI32, {B});
    const float *ua = a.ptr<float>(p[8], kF32, {B, K});
    const uint8_t *greedy = a.ptr<uint8_t>(p[9], kU8, {B});
    const float *dl = a.ptr<float>(p[10], kF32, {B, K});
    PyObject *out = a.dict(p[11]);
    if (!a.ok) Py_RETURN_NONE;
    int32_t *al = a.need<int32_t>(out, "accept_len", kI32, {B}), *ot = a.need<int32_t>(out, "out_tok", kI32, {B, K + 1}), *no = a.need<int32_t>(out, "n_out", kI32, {B});
    float *tl = a.out<float>(out, "target_lse", kF32, {B, K + 1}), *lp = a.out<float>(out, "logp_tok", kF32, {B, K});
    int32_t *t1 = a.out<int32_t>(out, "target_top1", kI32, {B, K + 1});
    auto *jobs = p[10] != Py_None ? a.out<tapout_final_job>(out, "final_jobs", kU8, {B, (int64_t)sizeof(tapout_final_job)}) : nullptr;
    uint32_t *fl = a.out<uint32_t>(out, "flags", kI32, {B});
    void *st = a.stream(p[12]);
    return call(a, [&] {
        return g_lib.verify_accept_sharded(c, s, (int32_t)G, (int32_t)B, (int32_t)K, V, lq, tok, n, greedy, ua, dl, al, ot, no, tl, lp, t1, jobs, fl, st);
    });
}

// (ctx, target_shard, draft_shard, jobs, sums, stream)
PyObject *shard_final_sums(PyObject *const *p)
{
    Args a;
    tapout_ctx *c = a.ctx(p[0]);
    int64_t B = 0, K1 = 0, V = 0, Bd, Kd, Vd;
    const tapout_logits t = a.logits(p[1], &B, &K1, &V), d = a.logits(p[2], &Bd, &Kd, &Vd);
    auto *jobs = a.ptr<tapout_final_job>(p[3], kU8, {B, (int64_t)sizeof(tapout_final_job)});
    double *sums = a.required<double>(p[4], kF64, {B, 5});
    void *st = a.stream(p[5]);
    return call(a, [&] { return g_lib.shard_final_sums(c, &t, &d, (int32_t)B, (int32_t)(K1 - 1), (int32_t)V, jobs, sums, st); });
}

// (ctx, target_shard, draft_shard, vocab_offset, G, g, jobs, sums_all, exact_all, u_sample, tok, mass, need, stream)
PyObject *shard_final_token(PyObject *const *p)
{
    Args a;
    tapout_ctx *c = a.ctx(p[0]);
    int64_t B = 0, K1 = 0, V = 0, Bd, Kd, Vd;
    const tapout_logits t = a.logits(p[1], &B, &K1, &V), d = a.logits(p[2], &Bd, &Kd, &Vd);
    const int32_t off = a.i32(p[3]), g = a.i32(p[5]);
    const int64_t G = a.i32(p[4]);
    auto *jobs = a.ptr<tapout_final_job>(p[6], kU8, {B, (int64_t)sizeof(tapout_final_job)});
    const double *sums = a.ptr<double>(p[7], kF64, {G, B, 5}), *exact = a.ptr<double>(p[8], kF64, {G, B});
    const float *u = a.ptr<float>(p[9], kF32, {B});
    int32_t *tok = a.required<int32_t>(p[10], kI32, {B});
    double *mass = a.required<double>(p[11], kF64, {B});
    uint8_t *need = a.required<uint8_t>(p[12], kU8, {B});
    void *st = a.stream(p[13]);
    return call(a, [&] { return g_lib.shard_final_token(c, &t, &d, (int32_t)B, (int32_t)(K1 - 1), (int32_t)V, off, (int32_t)G, g, jobs, sums, exact, u, tok, mass, need, st); });
}

// load(path): the entry points of this build of the library
PyObject *load(PyObject *, PyObject *arg)
{
    const char *path = PyUnicode_AsUTF8(arg);
    if (!path) return nullptr;
    void *h = dlopen(path, RTLD_NOW | RTLD_LOCAL);
    if (!h) { PyErr_SetString(PyExc_ImportError, dlerror()); return nullptr; }
    Library l = {};
    bool ok = true;
    auto get = [&](auto &f, const char *name) {
        f = reinterpret_cast<std::remove_reference_t<decltype(f)>>(dlsym(h, name));
        ok = ok && f;
    };
    get(l.bandit_select, "tapout_bandit_select"); get(l.draft_stats, "tapout_draft_stats"); get(l.verify, "tapout_verify");
    get(l.bandit_update, "tapout_bandit_update"); get(l.bandit_update_select, "tapout_bandit_update_select");
    get(l.shard_stats, "tapout_shard_stats"); get(l.draft_stats_sharded, "tapout_draft_stats_sharded");
    get(l.verify_accept_sharded, "tapout_verify_accept_sharded"); get(l.shard_final_sums, "tapout_shard_final_sums");
    get(l.shard_final_token, "tapout_shard_final_token");
    if (!ok) { PyErr_Format(PyExc_ImportError, "%s lacks an entry point", path); return nullptr; }
    g_lib = l;
    Py_RETURN_NONE;
}

// current_stream(): handle of the current stream of the current device
PyObject *current_stream(PyObject *, PyObject *)
{
    try {
        return PyLong_FromVoidPtr((void *)c10::hip::getCurrentHIPStream().stream());
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

#define ENTRY(name, n) {#name, (PyCFunction)(void (*)(void))entry<name, n>, METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {
    {"load", load, METH_O, nullptr}, {"current_stream", current_stream, METH_NOARGS, nullptr},
    ENTRY(bandit_select, 8), ENTRY(draft_stats, 9), ENTRY(verify, 12), ENTRY(bandit_update, 9), ENTRY(bandit_update_select, 13),
    ENTRY(shard_stats, 8), ENTRY(draft_stats_sharded, 11), ENTRY(verify_accept_sharded, 13), ENTRY(shard_final_sums, 6), ENTRY(shard_final_token, 14),
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&g_module); }
