// Argument marshalling of the short calls, in C++: what bounds these calls is the host, not the kernels.  A Python call of
// arrol_score took 7.0 us, of which the launch is 2.7: two torch.empty 2.5, checks, pointers and ctypes the rest; from here 4.4.
//
// Every function here does what its namesake in binding.py does, for the ordinary case only: plain tensors (or parameters)
// with storage, of the right type, on the current GPU and contiguous, numbers that fit, no stream given, no function or
// dispatch mode of torch's active and no deterministic mode (which fills new memory).  In any other case it returns None before anything is launched, and binding.py goes the whole way
// itself, its errors included.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/EmptyTensor.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <torch/csrc/autograd/python_variable.h>

#include <atomic>
#include <cstring>

#include "arrol.h"

namespace {

PyObject* g_parameter = nullptr;      // torch.nn.Parameter
PyObject* g_policy = nullptr;         // binding.Policy
PyObject* g_device = nullptr;         // torch._C._cuda_getDevice
PyObject* g_raw_stream = nullptr;     // torch._C._cuda_getCurrentRawStream
PyObject* g_check = nullptr;          // binding._check

struct Odd {};                        // not the ordinary case

const at::Tensor& tensor(PyObject* o) {
    if (reinterpret_cast<PyObject*>(Py_TYPE(o)) != THPVariableClass && reinterpret_cast<PyObject*>(Py_TYPE(o)) != g_parameter) throw Odd();
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || !t.has_storage()) throw Odd();
    return t;
}
void* data(const at::Tensor& t) { return t.data_ptr(); }
// a contiguous tensor of this type; `ptr`: or None
const at::Tensor& tensor(PyObject* o, at::ScalarType type) {
    const at::Tensor& t = tensor(o);
    if (t.scalar_type() != type || !t.is_contiguous()) throw Odd();
    return t;
}
template <class T = void>
T* ptr(PyObject* o, at::ScalarType type) { return o == Py_None ? nullptr : static_cast<T*>(data(tensor(o, type))); }

// 2-D bf16 rows, each contiguous
struct Rows {
    const at::Tensor& t;
    int64_t n, d, stride;
    const int64_t* index;
    Rows(PyObject* o, PyObject* row_index) : t(tensor(o)), index(nullptr) {
        if (t.dim() != 2 || t.scalar_type() != at::kBFloat16 || t.stride(1) != 1) throw Odd();
        d = t.size(1);
        stride = t.size(0) > 1 ? t.stride(0) : (t.stride(0) > d ? t.stride(0) : d);
        n = t.size(0);
        if (row_index != Py_None) {
            const at::Tensor& i = tensor(row_index, at::kLong);
            n = i.numel();
            index = static_cast<const int64_t*>(data(i));
        }
        if (n > INT32_MAX || d > INT32_MAX) throw Odd();
    }
};

double number(PyObject* o) {
    if (PyFloat_CheckExact(o)) return PyFloat_AS_DOUBLE(o);
    if (!PyLong_CheckExact(o)) throw Odd();
    const double v = PyLong_AsDouble(o);
    if (PyErr_Occurred()) { PyErr_Clear(); throw Odd(); }
    return v;
}
int32_t integer(PyObject* o, int32_t least = 0) {
    if (!PyLong_CheckExact(o)) throw Odd();
    int over = 0;
    const long long v = PyLong_AsLongLongAndOverflow(o, &over);
    if (over || v < least || v > INT32_MAX) throw Odd();
    return static_cast<int32_t>(v);
}
bool truth(PyObject* o) {
    if (o != Py_True && o != Py_False) throw Odd();
    return o == Py_True;
}
void none(PyObject* o) {
    if (o != Py_None) throw Odd();
}

struct Unlocked {     // launches go without the interpreter lock, as ctypes calls do
    PyThreadState* save = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(save); }
};
std::atomic<c10::Allocator*> g_allocator{nullptr};      // that of torch.empty's storages
// An output: what torch.empty gives (the same allocator, on the current stream), without its way through the dispatcher
// (0.9 -> 0.5 us).  entry() has seen to it that no mode is to be asked and that nothing fills new memory; the lock is let go,
// since the allocator may wait for the device.
at::Tensor make(at::IntArrayRef shape, at::ScalarType type, const at::Tensor& like) {
    const Unlocked u;
    if (!g_allocator) g_allocator = at::empty({1}, at::TensorOptions().dtype(type).device(like.device())).storage().allocator();
    if (!g_allocator) throw Odd();
    return at::detail::empty_generic(shape, g_allocator.load(), c10::DispatchKeySet(c10::DispatchKey::CUDA), type, std::nullopt);
}
// the current device's current stream, as binding._stream asks for it
void* stream(const at::Tensor& like) {
    PyObject* dev = PyObject_CallNoArgs(g_device);
    if (!dev) { PyErr_Clear(); throw Odd(); }
    if (PyLong_AsLong(dev) != like.device().index()) { Py_DECREF(dev); throw Odd(); }   // make() allocates on the current device
    PyObject* s = PyObject_CallOneArg(g_raw_stream, dev);
    Py_DECREF(dev);
    void* h = s ? PyLong_AsVoidPtr(s) : nullptr;
    Py_XDECREF(s);
    if (PyErr_Occurred()) { PyErr_Clear(); throw Odd(); }
    return h;
}

template <class F>
int launch(F f) {
    const Unlocked u;
    return f();
}
bool failed(const char* name, int rc) {
    if (rc == ARROL_OK) return false;
    PyObject* r = PyObject_CallFunction(g_check, "si", name, rc);   // raises ArrolError
    Py_XDECREF(r);
    return true;
}

PyObject* wrap(at::Tensor t) { return THPVariable_Wrap(std::move(t)); }
PyObject* keep(PyObject* o) { Py_INCREF(o); return o; }
template <class... P>
PyObject* tuple(P*... items) {       // steals them
    PyObject* t = PyTuple_New(sizeof...(items));
    Py_ssize_t i = 0;
    bool ok = t != nullptr;
    for (PyObject* o : {static_cast<PyObject*>(items)...}) {
        ok = ok && o;
        if (t) PyTuple_SET_ITEM(t, i++, o); else Py_XDECREF(o);
    }
    if (!ok) { Py_XDECREF(t); return nullptr; }
    return t;
}
bool put(PyObject* dict, const char* key, PyObject* value) {        // steals value
    const bool ok = value && PyDict_SetItemString(dict, key, value) == 0;
    Py_XDECREF(value);
    return ok;
}

// hidden, w, bias, row_index, out_score, out_prob, want_score
PyObject* score(PyObject* const* a) {
    const Rows h(a[0], a[3]);
    const float bias = static_cast<float>(number(a[2]));
    const bool want = truth(a[6]);
    const float* w = static_cast<const float*>(data(tensor(a[1], at::kFloat)));
    at::Tensor s, q;
    float *ps = ptr<float>(a[4], at::kFloat), *pq = ptr<float>(a[5], at::kFloat);
    void* st = stream(h.t);
    if (a[4] == Py_None && want) { s = make({h.n}, at::kFloat, h.t); ps = static_cast<float*>(data(s)); }
    if (a[5] == Py_None) { q = make({h.n}, at::kFloat, h.t); pq = static_cast<float*>(data(q)); }
    const void* x = data(h.t);
    if (failed("arrol_score", launch([&] { return arrol_score(x, h.stride, h.index, w, bias, h.n, h.d, ps, pq, st); }))) return nullptr;
    return tuple(s.defined() ? wrap(std::move(s)) : keep(a[4]), q.defined() ? wrap(std::move(q)) : keep(a[5]));
}

// w1 [m, d], b1 [m] or None, w2 [m] of a two-layer head
struct Head {
    const void* w1; const float* b1; const float* w2;
    int32_t m;
    Head(PyObject* o1, PyObject* ob, PyObject* o2, int64_t d) {
        const at::Tensor &t1 = tensor(o1, at::kBFloat16), &t2 = tensor(o2, at::kFloat);
        if (t1.dim() != 2 || t1.size(1) != d || t1.size(0) > INT32_MAX || t2.numel() != t1.size(0)) throw Odd();
        m = static_cast<int32_t>(t1.size(0));
        b1 = ptr<const float>(ob, at::kFloat);
        if (b1 && tensor(ob).numel() != m) throw Odd();
        w1 = data(t1);
        w2 = static_cast<const float*>(data(t2));
    }
};

// hidden, w1, b1, w2, b2, row_index, workspace (the default "auto" only)
PyObject* score_mlp(PyObject* const* a) {
    const Rows h(a[0], a[5]);
    const Head p(a[1], a[2], a[3], h.d);
    const float b2 = static_cast<float>(number(a[4]));
    if (!PyUnicode_CheckExact(a[6])) throw Odd();
    void* st = stream(h.t);
    at::Tensor s = make({h.n}, at::kFloat, h.t), q = make({h.n}, at::kFloat, h.t), ws;
    const size_t need = arrol_score_mlp_workspace_bytes(h.n, h.d, p.m);
    if (need) ws = make({static_cast<int64_t>(need)}, at::kByte, h.t);
    void *x = data(h.t), *pw = need ? data(ws) : nullptr;
    float *ps = static_cast<float*>(data(s)), *pq = static_cast<float*>(data(q));
    if (failed("arrol_score_mlp", launch([&] { return arrol_score_mlp(x, h.stride, h.index, p.w1, p.b1, p.w2, b2, h.n, h.d, p.m, ps, pq, pw, need, st); })))
        return nullptr;
    return tuple(wrap(std::move(s)), wrap(std::move(q)));
}

// hidden, w, bias, labels, row_index, workspace (None only)
PyObject* score_grad(PyObject* const* a) {
    const Rows h(a[0], a[4]);
    const at::Tensor &w = tensor(a[1], at::kFloat), &y = tensor(a[3], at::kFloat);
    const float bias = static_cast<float>(number(a[2]));
    none(a[5]);
    if (y.numel() != h.n || w.numel() != h.d) throw Odd();
    void* st = stream(h.t);
    const size_t need = arrol_score_grad_workspace_bytes(h.n, h.d), have = need ? need : 1;
    at::Tensor ws = make({static_cast<int64_t>(have)}, at::kByte, h.t), loss = make({1}, at::kFloat, h.t), gw = make({h.d}, at::kFloat, h.t),
               gb = make({1}, at::kFloat, h.t);
    const void* x = data(h.t);
    const float *pw = static_cast<const float*>(data(w)), *py = static_cast<const float*>(data(y));
    float *pl = static_cast<float*>(data(loss)), *pg = static_cast<float*>(data(gw)), *pb = static_cast<float*>(data(gb));
    void* pws = data(ws);
    if (failed("arrol_score_grad", launch([&] { return arrol_score_grad(x, h.stride, h.index, pw, bias, py, h.n, h.d, pl, pg, pb, pws, have, st); })))
        return nullptr;
    return tuple(wrap(std::move(loss)), wrap(std::move(gw)), wrap(std::move(gb)));
}

// hidden, w1, b1, w2, b2, labels, row_index, delta_terms, workspace (None only)
PyObject* score_mlp_grad(PyObject* const* a) {
    const Rows h(a[0], a[6]);
    const Head p(a[1], a[2], a[3], h.d);
    const float b2 = static_cast<float>(number(a[4]));
    const at::Tensor& y = tensor(a[5], at::kFloat);
    const int32_t terms = integer(a[7]);
    none(a[8]);
    if (y.numel() != h.n) throw Odd();
    void* st = stream(h.t);
    size_t need = arrol_score_mlp_grad_workspace_bytes(h.n, h.d, p.m, terms);
    need = need > 256 ? need : 256;
    at::Tensor ws = make({static_cast<int64_t>(need)}, at::kByte, h.t), loss = make({1}, at::kFloat, h.t), g1 = make({p.m, h.d}, at::kFloat, h.t),
               gb1 = make({p.m}, at::kFloat, h.t), g2 = make({p.m}, at::kFloat, h.t), gb2 = make({1}, at::kFloat, h.t);
    const void* x = data(h.t);
    const float* py = static_cast<const float*>(data(y));
    float *pl = static_cast<float*>(data(loss)), *p1 = static_cast<float*>(data(g1)), *pb1 = static_cast<float*>(data(gb1)),
          *p2 = static_cast<float*>(data(g2)), *pb2 = static_cast<float*>(data(gb2));
    void* pws = data(ws);
    if (failed("arrol_score_mlp_grad", launch([&] {
            return arrol_score_mlp_grad(x, h.stride, h.index, p.w1, p.b1, p.w2, b2, py, h.n, h.d, p.m, pl, p1, pb1, p2, pb2, terms, pws, need, st);
        })))
        return nullptr;
    PyObject* out = PyDict_New();
    if (!out) return nullptr;
    if (!put(out, "loss", wrap(std::move(loss))) || !put(out, "grad_w1", wrap(std::move(g1))) || !put(out, "grad_b1", wrap(std::move(gb1))) ||
        !put(out, "grad_w2", wrap(std::move(g2))) || !put(out, "grad_b2", wrap(std::move(gb2)))) {
        Py_DECREF(out);
        return nullptr;
    }
    return out;
}

// param, grad, m, v, step, lr, beta1, beta2, eps, weight_decay, param_bf16
PyObject* adamw_step(PyObject* const* a) {
    const at::Tensor &p = tensor(a[0], at::kFloat), &g = tensor(a[1], at::kFloat), &m = tensor(a[2], at::kFloat), &v = tensor(a[3], at::kFloat);
    const int64_t n = p.numel();
    void* p16 = ptr(a[10], at::kBFloat16);
    if (g.numel() != n || m.numel() != n || v.numel() != n || (p16 && tensor(a[10]).numel() != n)) throw Odd();
    const int32_t step = integer(a[4]);
    const float lr = static_cast<float>(number(a[5])), b1 = static_cast<float>(number(a[6])), b2 = static_cast<float>(number(a[7])),
                eps = static_cast<float>(number(a[8])), wd = static_cast<float>(number(a[9]));
    float *pp = static_cast<float*>(data(p)), *pm = static_cast<float*>(data(m)), *pv = static_cast<float*>(data(v));
    const float* pg = static_cast<const float*>(data(g));
    void* st = stream(p);
    if (failed("arrol_adamw_step", launch([&] { return arrol_adamw_step(pp, pg, pm, pv, n, step, lr, b1, b2, eps, wd, p16, st); }))) return nullptr;
    return keep(a[0]);
}

// prob, n_groups, G, K, rho, out_keep, out_survivors
PyObject* select(PyObject* const* a) {
    const at::Tensor& prob = tensor(a[0], at::kFloat);
    const int32_t groups = integer(a[1]), G = integer(a[2]), K = integer(a[3]);
    const float rho = static_cast<float>(number(a[4]));
    if (prob.numel() != static_cast<int64_t>(groups) * G) throw Odd();
    uint8_t* pk = ptr<uint8_t>(a[5], at::kByte);
    int32_t* pi = ptr<int32_t>(a[6], at::kInt);
    void* st = stream(prob);
    at::Tensor mask, surv;
    if (a[5] == Py_None) { mask = make({static_cast<int64_t>(groups) * G}, at::kByte, prob); pk = static_cast<uint8_t*>(data(mask)); }
    if (a[6] == Py_None) { surv = make({static_cast<int64_t>(groups) * K}, at::kInt, prob); pi = static_cast<int32_t*>(data(surv)); }
    const float* pp = static_cast<const float*>(data(prob));
    if (failed("arrol_select", launch([&] { return arrol_select(pp, groups, G, K, rho, pk, pi, st); }))) return nullptr;
    return tuple(mask.defined() ? wrap(std::move(mask)) : keep(a[5]), surv.defined() ? wrap(std::move(surv)) : keep(a[6]));
}

// prob, answer_id, n_questions, C, n_answers
PyObject* weighted_vote(PyObject* const* a) {
    const at::Tensor &prob = tensor(a[0], at::kFloat), &ans = tensor(a[1], at::kInt);
    const int32_t Q = integer(a[2]), C = integer(a[3]), A = integer(a[4]);
    if (prob.numel() != static_cast<int64_t>(Q) * C || ans.numel() != static_cast<int64_t>(Q) * C) throw Odd();
    void* st = stream(prob);
    at::Tensor win = make({Q}, at::kInt, prob);
    const float* pp = static_cast<const float*>(data(prob));
    const int32_t* pa = static_cast<const int32_t*>(data(ans));
    int32_t* pw = static_cast<int32_t*>(data(win));
    if (failed("arrol_weighted_vote", launch([&] { return arrol_weighted_vote(pp, pa, Q, C, A, pw, nullptr, st); }))) return nullptr;
    return wrap(std::move(win));
}

// s_norm, label, B
PyObject* histogram(PyObject* const* a) {
    const at::Tensor &s = tensor(a[0], at::kFloat), &l = tensor(a[1], at::kByte);
    const int32_t B = integer(a[2]);
    const int64_t M = s.numel();
    void* st = stream(s);
    at::Tensor pos = make({B}, at::kLong, s), neg = make({B}, at::kLong, s);
    const float* ps = static_cast<const float*>(data(s));
    const uint8_t* pl = static_cast<const uint8_t*>(data(l));
    int64_t *pp = static_cast<int64_t*>(data(pos)), *pn = static_cast<int64_t*>(data(neg));
    if (failed("arrol_histogram", launch([&] { return arrol_histogram(ps, pl, M, B, pp, pn, st); }))) return nullptr;
    return tuple(wrap(std::move(pos)), wrap(std::move(neg)));
}

// c_pos, c_neg, policy
PyObject* calibrate(PyObject* const* a) {
    const at::Tensor &pos = tensor(a[0], at::kLong), &neg = tensor(a[1], at::kLong);
    if (reinterpret_cast<PyObject*>(Py_TYPE(a[2])) != g_policy || pos.numel() > INT32_MAX) throw Odd();
    arrol_policy policy;
    Py_buffer view;
    if (PyObject_GetBuffer(a[2], &view, PyBUF_SIMPLE)) { PyErr_Clear(); throw Odd(); }
    const bool fits = view.len == static_cast<Py_ssize_t>(sizeof policy);
    if (fits) std::memcpy(&policy, view.buf, sizeof policy);
    PyBuffer_Release(&view);
    if (!fits) throw Odd();
    const int32_t B = static_cast<int32_t>(pos.numel());
    void* st = stream(pos);
    at::Tensor q = make({B}, at::kFloat, pos), p = make({B}, at::kFloat, pos), delta = make({1}, at::kDouble, pos);
    const int64_t *pp = static_cast<const int64_t*>(data(pos)), *pn = static_cast<const int64_t*>(data(neg));
    float *fq = static_cast<float*>(data(q)), *fp = static_cast<float*>(data(p));
    double* pd = static_cast<double*>(data(delta));
    if (failed("arrol_calibrate", launch([&] { return arrol_calibrate(pp, pn, B, policy, fq, fp, pd, st); }))) return nullptr;
    return tuple(wrap(std::move(q)), wrap(std::move(p)), wrap(std::move(delta)));
}

// s_norm, uniforms, p_lut, want_p
PyObject* prune_bernoulli(PyObject* const* a) {
    const at::Tensor &s = tensor(a[0], at::kFloat), &u = tensor(a[1], at::kFloat), &lut = tensor(a[2], at::kFloat);
    const bool want = truth(a[3]);
    if (s.numel() > INT32_MAX || lut.numel() > INT32_MAX) throw Odd();
    const int64_t N = s.numel();
    void* st = stream(s);
    at::Tensor mask = make({N}, at::kByte, s), idx = make({N}, at::kInt, s), n = make({1}, at::kInt, s), p;
    if (want) p = make({N}, at::kFloat, s);
    const float *ps = static_cast<const float*>(data(s)), *pu = static_cast<const float*>(data(u)), *pl = static_cast<const float*>(data(lut));
    float* pp = want ? static_cast<float*>(data(p)) : nullptr;
    uint8_t* pm = static_cast<uint8_t*>(data(mask));
    int32_t *pi = static_cast<int32_t*>(data(idx)), *pn = static_cast<int32_t*>(data(n));
    const int32_t B = static_cast<int32_t>(lut.numel());
    if (failed("arrol_prune_bernoulli", launch([&] { return arrol_prune_bernoulli(ps, pu, N, pl, B, pp, pm, pi, pn, st); }))) return nullptr;
    PyObject* out = PyDict_New();
    if (!out) return nullptr;
    if (!put(out, "keep_mask", wrap(std::move(mask))) || !put(out, "survivor_idx", wrap(std::move(idx))) || !put(out, "n_survivors", wrap(std::move(n))) ||
        !put(out, "p", want ? wrap(std::move(p)) : keep(Py_None))) {
        Py_DECREF(out);
        return nullptr;
    }
    return out;
}

// reward, group_offsets, ddof, eps
PyObject* grpo_advantage(PyObject* const* a) {
    const at::Tensor &r = tensor(a[0], at::kFloat), &off = tensor(a[1], at::kLong);
    const int32_t ddof = integer(a[2]);
    const float eps = static_cast<float>(number(a[3]));
    const int64_t N = r.numel(), groups = off.numel() - 1;
    if (groups < 0 || groups > INT32_MAX) throw Odd();
    void* st = stream(r);
    at::Tensor adv = make({N}, at::kFloat, r), wgt = make({N}, at::kFloat, r);
    const float* pr = static_cast<const float*>(data(r));
    const int64_t* po = static_cast<const int64_t*>(data(off));
    float *pa = static_cast<float*>(data(adv)), *pw = static_cast<float*>(data(wgt));
    if (failed("arrol_grpo_advantage", launch([&] { return arrol_grpo_advantage_all(pr, po, N, groups, ddof, eps, pa, pw, st); }))) return nullptr;
    return tuple(wrap(std::move(adv)), wrap(std::move(wgt)));
}

// logp, logp_ref, cu_seqlens, advantage, seq_weight, eps_low, eps_high, beta, want_grad, workspace (None only)
PyObject* grpo_objective(PyObject* const* a) {
    const at::Tensor &lp = tensor(a[0], at::kFloat), &ref = tensor(a[1], at::kFloat), &cu = tensor(a[2], at::kLong), &adv = tensor(a[3], at::kFloat),
                     &wgt = tensor(a[4], at::kFloat);
    const float lo = static_cast<float>(number(a[5])), hi = static_cast<float>(number(a[6])), beta = static_cast<float>(number(a[7]));
    const bool want = truth(a[8]);
    none(a[9]);
    const int64_t T = lp.numel(), n = cu.numel() - 1;
    if (n < 0 || n > INT32_MAX || ref.numel() != T || adv.numel() != n || wgt.numel() != n) throw Odd();
    void* st = stream(lp);
    size_t need = 8 * arrol_grpo_objective_workspace_bytes(static_cast<int32_t>(n));
    need = need > 16 ? need : 16;
    at::Tensor ws = make({static_cast<int64_t>(need)}, at::kByte, lp), J = make({1}, at::kDouble, lp), grad, clip = make({1}, at::kLong, lp);
    if (want) grad = make({T}, at::kFloat, lp);
    const float *pl = static_cast<const float*>(data(lp)), *pr = static_cast<const float*>(data(ref)), *pa = static_cast<const float*>(data(adv)),
                *pw = static_cast<const float*>(data(wgt));
    const int64_t* pc = static_cast<const int64_t*>(data(cu));
    double* pj = static_cast<double*>(data(J));
    float* pg = want ? static_cast<float*>(data(grad)) : nullptr;
    int64_t* pn = static_cast<int64_t*>(data(clip));
    void* pws = data(ws);
    if (failed("arrol_grpo_objective", launch([&] { return arrol_grpo_objective(pl, pr, pc, T, n, pa, pw, lo, hi, beta, pj, pg, pn, pws, need, st); })))
        return nullptr;
    return tuple(wrap(std::move(J)), want ? wrap(std::move(grad)) : keep(Py_None), wrap(std::move(clip)));
}

template <PyObject* (*F)(PyObject* const*), int N>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t n) {
    if (n != N) {
        PyErr_Format(PyExc_TypeError, "%d arguments expected", N);
        return nullptr;
    }
    try {
        if (at::impl::PythonTorchFunctionTLS::stack_len() > 0 || c10::impl::TorchDispatchModeTLS::any_modes_set() ||
            at::globalContext().deterministicAlgorithms())
            throw Odd();
        return F(args);
    } catch (...) {      // nothing has been launched: what can throw comes before
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

PyObject* setup(PyObject*, PyObject* const* args, Py_ssize_t n) {
    if (n != 5) {
        PyErr_SetString(PyExc_TypeError, "5 arguments expected");
        return nullptr;
    }
    PyObject** slots[5] = {&g_parameter, &g_policy, &g_device, &g_raw_stream, &g_check};
    for (int i = 0; i < 5; ++i) {
        Py_INCREF(args[i]);
        Py_XDECREF(*slots[i]);
        *slots[i] = args[i];
    }
    return PyLong_FromLong(arrol_version());
}

#define ENTRY(name, n) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&entry<name, n>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"setup", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&setup)), METH_FASTCALL, nullptr},
    ENTRY(score, 7), ENTRY(score_mlp, 7), ENTRY(score_grad, 6), ENTRY(score_mlp_grad, 9), ENTRY(adamw_step, 11), ENTRY(select, 7),
    ENTRY(weighted_vote, 5), ENTRY(histogram, 3), ENTRY(calibrate, 3), ENTRY(prune_bernoulli, 4), ENTRY(grpo_advantage, 4),
    ENTRY(grpo_objective, 10),
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&module); }
