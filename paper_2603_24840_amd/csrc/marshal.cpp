// Argument marshalling of the short calls, in C++: what bounds these calls is the host, not the kernels.  A Python call of
// arrol_score took 7.0 us, of which the launch is 2.7: two torch.empty 2.5, checks, pointers and ctypes the rest; from here 4.4.
//
// Every function here does what its namesake in binding.py does, for the ordinary case only: plain tensors (or parameters)
// with storage, of the right type, on the current GPU and contiguous, numbers that fit, no stream given, no function or
// dispatch mode of torch's active and no deterministic mode (which fills new memory).  In any other case it returns None before
// anything is launched, and binding.py goes the whole way itself, its errors included.  That is said by a flag and a null
// pointer: with a C++ exception a refusal cost 2.5 to 3.4 us, and so 0.07.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/EmptyTensor.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <atomic>
#include <cstring>

#include "arrol.h"

namespace {

PyObject* g_parameter = nullptr;      // torch.nn.Parameter
PyObject* g_policy = nullptr;         // binding.Policy
PyObject* g_check = nullptr;          // binding._check

void* data(const at::Tensor& t) { return t.data_ptr(); }

// The arguments of one call, read one by one.  What is read after one that is not ordinary is not to be used.
struct Args {
    PyObject* const* a;
    bool odd = false;                 // not the ordinary case

    PyObject* operator[](int i) const { return a[i]; }
    bool given(int i) const { return a[i] != Py_None; }
    bool refuse(bool yes) { return odd = odd || yes; }

    // a GPU tensor, or an undefined one
    const at::Tensor& tensor(int i) {
        static const at::Tensor nothing;
        PyObject* o = a[i];
        if (refuse(reinterpret_cast<PyObject*>(Py_TYPE(o)) != THPVariableClass && reinterpret_cast<PyObject*>(Py_TYPE(o)) != g_parameter)) return nothing;
        const at::Tensor& t = THPVariable_Unpack(o);
        return refuse(!t.defined() || !t.is_cuda() || !t.has_storage()) ? nothing : t;
    }
    // a contiguous one of this type and, where given, number of elements; `ptr`: its memory, or that of None
    const at::Tensor& tensor(int i, at::ScalarType type, int64_t numel = -1) {
        const at::Tensor& t = tensor(i);
        if (!odd) refuse(t.scalar_type() != type || !t.is_contiguous() || (numel >= 0 && t.numel() != numel));
        return t;
    }
    template <class T = void>
    T* ptr(int i, at::ScalarType type, int64_t numel = -1) {
        if (!given(i)) return nullptr;
        const at::Tensor& t = tensor(i, type, numel);
        return odd ? nullptr : static_cast<T*>(data(t));
    }
    double number(int i) {            // as float() gives it, but of no text
        if (PyFloat_CheckExact(a[i])) return PyFloat_AS_DOUBLE(a[i]);
        const PyNumberMethods* as = Py_TYPE(a[i])->tp_as_number;
        if (refuse(!PyLong_CheckExact(a[i]) && !(as && as->nb_float))) return 0.0;
        PyObject* f = PyNumber_Float(a[i]);
        const double v = f ? PyFloat_AsDouble(f) : 0.0;
        if (refuse(!f)) PyErr_Clear();
        Py_XDECREF(f);
        return v;
    }
    int32_t integer(int i, int32_t least = 0) {
        if (refuse(!PyLong_CheckExact(a[i]))) return 0;
        int over = 0;
        const long long v = PyLong_AsLongLongAndOverflow(a[i], &over);
        return refuse(over || v < least || v > INT32_MAX) ? 0 : static_cast<int32_t>(v);
    }
    bool truth(int i) {
        refuse(a[i] != Py_True && a[i] != Py_False);
        return a[i] == Py_True;
    }
};

// 2-D bf16 rows, each contiguous
struct Rows {
    const at::Tensor& t;
    int64_t n = 0, d = 0, stride = 0;
    const int64_t* index = nullptr;
    Rows(Args& a, int rows, int row_index) : t(a.tensor(rows)) {
        if (a.odd || a.refuse(t.dim() != 2 || t.scalar_type() != at::kBFloat16 || t.stride(1) != 1)) return;
        d = t.size(1);
        stride = t.size(0) > 1 ? t.stride(0) : (t.stride(0) > d ? t.stride(0) : d);
        n = t.size(0);
        if (a.given(row_index)) {
            const at::Tensor& i = a.tensor(row_index, at::kLong);
            if (a.odd) return;
            n = i.numel();
            index = static_cast<const int64_t*>(data(i));
        }
        a.refuse(n > INT32_MAX || d > INT32_MAX);
    }
};

struct Unlocked {     // launches go without the interpreter lock, as ctypes calls do
    PyThreadState* save = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(save); }
};
std::atomic<c10::Allocator*> g_allocator{nullptr};      // that of torch.empty's storages
// An output: what torch.empty gives (the same allocator, on the current stream), without its way through the dispatcher
// (0.9 -> 0.5 us).  entry() has seen to it that no mode is to be asked and that nothing fills new memory; called without the
// interpreter lock, since the allocator may wait for the device.
at::Tensor make(at::IntArrayRef shape, at::ScalarType type, const at::Tensor& like) {
    if (!g_allocator) g_allocator = at::empty({1}, at::TensorOptions().dtype(type).device(like.device())).storage().allocator();
    TORCH_CHECK(g_allocator.load());
    return at::detail::empty_generic(shape, g_allocator.load(), c10::DispatchKeySet(c10::DispatchKey::CUDA), type, std::nullopt);
}
template <class T = void>
T* made(at::Tensor& out, at::IntArrayRef shape, at::ScalarType type, const at::Tensor& like) {
    out = make(shape, type, like);
    return static_cast<T*>(data(out));
}
// The current device's current stream, as torch's C layer gives it to binding._stream: asked of c10 itself (two Python calls were 0.25 us)
void* stream(Args& a, const at::Tensor& like) {
    const auto s = c10::hip::getCurrentHIPStream();
    return a.refuse(s.device_index() != like.device().index()) ? nullptr : s.stream();       // make() allocates on the current device
}
// The caller's uint8 tensor, or, for None (`text`: for a text, and nothing for None), one of `need` bytes for the time of the
// call: the allocator hands it out again on the stream that the kernels run on.
struct Scratch {
    at::Tensor own;
    void* p = nullptr;
    size_t bytes = 0;
    bool wanted = false;
    Scratch(Args& a, int i, size_t need, bool text = false) {
        if (text ? PyUnicode_CheckExact(a[i]) : !a.given(i)) {
            wanted = need > 0;
            bytes = need;
        } else if (a.given(i)) {
            const at::Tensor& t = a.tensor(i, at::kByte);
            if (a.odd) return;
            p = data(t);
            bytes = static_cast<size_t>(t.numel());
        }
    }
    void get(const at::Tensor& like) {       // without the interpreter lock
        if (wanted) p = made(own, {static_cast<int64_t>(bytes)}, at::kByte, like);
    }
};

// f makes the outputs and launches
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

// Each of the following returns nullptr where it refuses, and where a Python error is set.

// hidden, w, bias, row_index, out_score, out_prob, want_score
PyObject* score(Args& a) {
    const Rows h(a, 0, 3);
    const float* w = a.ptr<float>(1, at::kFloat);
    const float bias = static_cast<float>(a.number(2));
    const bool want = a.truth(6);
    float *ps = a.ptr<float>(4, at::kFloat), *pq = a.ptr<float>(5, at::kFloat);
    if (a.refuse(!a.given(1))) return nullptr;
    void* st = stream(a, h.t);
    if (a.odd) return nullptr;
    at::Tensor s, q;
    const bool own_s = !a.given(4) && want, own_q = !a.given(5);
    if (failed("arrol_score", launch([&] {
            if (own_s) ps = made<float>(s, {h.n}, at::kFloat, h.t);
            if (own_q) pq = made<float>(q, {h.n}, at::kFloat, h.t);
            return arrol_score(data(h.t), h.stride, h.index, w, bias, h.n, h.d, ps, pq, st);
        })))
        return nullptr;
    return tuple(s.defined() ? wrap(std::move(s)) : keep(a[4]), q.defined() ? wrap(std::move(q)) : keep(a[5]));
}

// w1 [m, d], b1 [m] or None, w2 [m] of a two-layer head
struct Head {
    const void* w1 = nullptr; const float* b1 = nullptr; const float* w2 = nullptr;
    int32_t m = 0;
    Head(Args& a, int o1, int ob, int o2, int64_t d) {
        const at::Tensor& t1 = a.tensor(o1, at::kBFloat16);
        if (a.odd || a.refuse(t1.dim() != 2 || t1.size(1) != d || t1.size(0) > INT32_MAX)) return;
        m = static_cast<int32_t>(t1.size(0));
        w1 = data(t1);
        b1 = a.ptr<float>(ob, at::kFloat, m);
        w2 = a.ptr<float>(o2, at::kFloat, m);
        a.refuse(!a.given(o2));
    }
};

// hidden, w1, b1, w2, b2, row_index, workspace (a text for what the library asks for, None for none, or a tensor)
PyObject* score_mlp(Args& a) {
    const Rows h(a, 0, 5);
    if (a.odd) return nullptr;
    const Head p(a, 1, 2, 3, h.d);
    const float b2 = static_cast<float>(a.number(4));
    if (a.odd) return nullptr;
    void* st = stream(a, h.t);
    if (a.odd) return nullptr;
    Scratch ws(a, 6, arrol_score_mlp_workspace_bytes(h.n, h.d, p.m), true);
    if (a.odd) return nullptr;
    at::Tensor s, q;
    if (failed("arrol_score_mlp", launch([&] {
            ws.get(h.t);
            float *ps = made<float>(s, {h.n}, at::kFloat, h.t), *pq = made<float>(q, {h.n}, at::kFloat, h.t);
            return arrol_score_mlp(data(h.t), h.stride, h.index, p.w1, p.b1, p.w2, b2, h.n, h.d, p.m, ps, pq, ws.p, ws.bytes, st);
        })))
        return nullptr;
    return tuple(wrap(std::move(s)), wrap(std::move(q)));
}

// hidden, w, bias, labels, row_index, workspace
PyObject* score_grad(Args& a) {
    const Rows h(a, 0, 4);
    if (a.odd) return nullptr;
    const float *pw = a.ptr<float>(1, at::kFloat, h.d), *py = a.ptr<float>(3, at::kFloat, h.n);
    const float bias = static_cast<float>(a.number(2));
    if (a.refuse(!a.given(1) || !a.given(3))) return nullptr;
    void* st = stream(a, h.t);
    if (a.odd) return nullptr;
    const size_t need = arrol_score_grad_workspace_bytes(h.n, h.d);
    Scratch ws(a, 5, need ? need : 1);
    if (a.odd) return nullptr;
    at::Tensor loss, gw, gb;
    if (failed("arrol_score_grad", launch([&] {
            ws.get(h.t);
            float *pl = made<float>(loss, {1}, at::kFloat, h.t), *pg = made<float>(gw, {h.d}, at::kFloat, h.t), *pb = made<float>(gb, {1}, at::kFloat, h.t);
            return arrol_score_grad(data(h.t), h.stride, h.index, pw, bias, py, h.n, h.d, pl, pg, pb, ws.p, ws.bytes, st);
        })))
        return nullptr;
    return tuple(wrap(std::move(loss)), wrap(std::move(gw)), wrap(std::move(gb)));
}

// hidden, w1, b1, w2, b2, labels, row_index, delta_terms, workspace
PyObject* score_mlp_grad(Args& a) {
    const Rows h(a, 0, 6);
    if (a.odd) return nullptr;
    const Head p(a, 1, 2, 3, h.d);
    const float b2 = static_cast<float>(a.number(4));
    const float* py = a.ptr<float>(5, at::kFloat, h.n);
    const int32_t terms = a.integer(7);
    if (a.refuse(!a.given(5))) return nullptr;
    void* st = stream(a, h.t);
    if (a.odd) return nullptr;
    const size_t need = arrol_score_mlp_grad_workspace_bytes(h.n, h.d, p.m, terms);
    Scratch ws(a, 8, need > 256 ? need : 256);
    if (a.odd) return nullptr;
    at::Tensor loss, g1, gb1, g2, gb2;
    if (failed("arrol_score_mlp_grad", launch([&] {
            ws.get(h.t);
            float *pl = made<float>(loss, {1}, at::kFloat, h.t), *p1 = made<float>(g1, {p.m, h.d}, at::kFloat, h.t), *pb1 = made<float>(gb1, {p.m}, at::kFloat, h.t),
                  *p2 = made<float>(g2, {p.m}, at::kFloat, h.t), *pb2 = made<float>(gb2, {1}, at::kFloat, h.t);
            return arrol_score_mlp_grad(data(h.t), h.stride, h.index, p.w1, p.b1, p.w2, b2, py, h.n, h.d, p.m, pl, p1, pb1, p2, pb2, terms, ws.p, ws.bytes, st);
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
PyObject* adamw_step(Args& a) {
    const at::Tensor& p = a.tensor(0, at::kFloat);
    if (a.odd) return nullptr;
    const int64_t n = p.numel();
    const float* pg = a.ptr<float>(1, at::kFloat, n);
    float *pp = static_cast<float*>(data(p)), *pm = a.ptr<float>(2, at::kFloat, n), *pv = a.ptr<float>(3, at::kFloat, n);
    const int32_t step = a.integer(4);
    const float lr = static_cast<float>(a.number(5)), b1 = static_cast<float>(a.number(6)), b2 = static_cast<float>(a.number(7)),
                eps = static_cast<float>(a.number(8)), wd = static_cast<float>(a.number(9));
    void* p16 = a.ptr(10, at::kBFloat16, n);
    if (a.refuse(!a.given(1) || !a.given(2) || !a.given(3))) return nullptr;
    void* st = stream(a, p);
    if (a.odd) return nullptr;
    if (failed("arrol_adamw_step", launch([&] { return arrol_adamw_step(pp, pg, pm, pv, n, step, lr, b1, b2, eps, wd, p16, st); }))) return nullptr;
    return keep(a[0]);
}

// prob, n_groups, G, K, rho, out_keep, out_survivors
PyObject* select(Args& a) {
    const int32_t groups = a.integer(1), G = a.integer(2), K = a.integer(3);
    const at::Tensor& prob = a.tensor(0, at::kFloat, static_cast<int64_t>(groups) * G);
    const float rho = static_cast<float>(a.number(4));
    uint8_t* pk = a.ptr<uint8_t>(5, at::kByte);
    int32_t* pi = a.ptr<int32_t>(6, at::kInt);
    if (a.odd) return nullptr;
    void* st = stream(a, prob);
    if (a.odd) return nullptr;
    at::Tensor mask, surv;
    const bool own_mask = !a.given(5), own_surv = !a.given(6);
    if (failed("arrol_select", launch([&] {
            if (own_mask) pk = made<uint8_t>(mask, {static_cast<int64_t>(groups) * G}, at::kByte, prob);
            if (own_surv) pi = made<int32_t>(surv, {static_cast<int64_t>(groups) * K}, at::kInt, prob);
            return arrol_select(static_cast<const float*>(data(prob)), groups, G, K, rho, pk, pi, st);
        })))
        return nullptr;
    return tuple(mask.defined() ? wrap(std::move(mask)) : keep(a[5]), surv.defined() ? wrap(std::move(surv)) : keep(a[6]));
}

// prob, answer_id, n_questions, C, n_answers
PyObject* weighted_vote(Args& a) {
    const int32_t Q = a.integer(2), C = a.integer(3), A = a.integer(4);
    const at::Tensor &prob = a.tensor(0, at::kFloat, static_cast<int64_t>(Q) * C), &ans = a.tensor(1, at::kInt, static_cast<int64_t>(Q) * C);
    if (a.odd) return nullptr;
    void* st = stream(a, prob);
    if (a.odd) return nullptr;
    at::Tensor win;
    const float* pp = static_cast<const float*>(data(prob));
    const int32_t* pa = static_cast<const int32_t*>(data(ans));
    if (failed("arrol_weighted_vote", launch([&] { return arrol_weighted_vote(pp, pa, Q, C, A, made<int32_t>(win, {Q}, at::kInt, prob), nullptr, st); })))
        return nullptr;
    return wrap(std::move(win));
}

// s_norm, label, B
PyObject* histogram(Args& a) {
    const at::Tensor &s = a.tensor(0, at::kFloat), &l = a.tensor(1, at::kByte);
    const int32_t B = a.integer(2);
    if (a.odd) return nullptr;
    const int64_t M = s.numel();
    void* st = stream(a, s);
    if (a.odd) return nullptr;
    at::Tensor pos, neg;
    const float* ps = static_cast<const float*>(data(s));
    const uint8_t* pl = static_cast<const uint8_t*>(data(l));
    if (failed("arrol_histogram", launch([&] {
            int64_t *pp = made<int64_t>(pos, {B}, at::kLong, s), *pn = made<int64_t>(neg, {B}, at::kLong, s);
            return arrol_histogram(ps, pl, M, B, pp, pn, st);
        })))
        return nullptr;
    return tuple(wrap(std::move(pos)), wrap(std::move(neg)));
}

// c_pos, c_neg, policy
PyObject* calibrate(Args& a) {
    const at::Tensor &pos = a.tensor(0, at::kLong), &neg = a.tensor(1, at::kLong);
    if (a.odd || a.refuse(reinterpret_cast<PyObject*>(Py_TYPE(a[2])) != g_policy || pos.numel() > INT32_MAX)) return nullptr;
    arrol_policy policy;
    Py_buffer view;
    if (a.refuse(PyObject_GetBuffer(a[2], &view, PyBUF_SIMPLE) != 0)) { PyErr_Clear(); return nullptr; }
    if (!a.refuse(view.len != static_cast<Py_ssize_t>(sizeof policy))) std::memcpy(&policy, view.buf, sizeof policy);
    PyBuffer_Release(&view);
    if (a.odd) return nullptr;
    const int32_t B = static_cast<int32_t>(pos.numel());
    void* st = stream(a, pos);
    if (a.odd) return nullptr;
    at::Tensor q, p, delta;
    const int64_t *pp = static_cast<const int64_t*>(data(pos)), *pn = static_cast<const int64_t*>(data(neg));
    if (failed("arrol_calibrate", launch([&] {
            float *fq = made<float>(q, {B}, at::kFloat, pos), *fp = made<float>(p, {B}, at::kFloat, pos);
            return arrol_calibrate(pp, pn, B, policy, fq, fp, made<double>(delta, {1}, at::kDouble, pos), st);
        })))
        return nullptr;
    return tuple(wrap(std::move(q)), wrap(std::move(p)), wrap(std::move(delta)));
}

// s_norm, uniforms, p_lut, want_p
PyObject* prune_bernoulli(Args& a) {
    const at::Tensor &s = a.tensor(0, at::kFloat), &u = a.tensor(1, at::kFloat), &lut = a.tensor(2, at::kFloat);
    const bool want = a.truth(3);
    if (a.odd || a.refuse(s.numel() > INT32_MAX || lut.numel() > INT32_MAX)) return nullptr;
    const int64_t N = s.numel();
    void* st = stream(a, s);
    if (a.odd) return nullptr;
    at::Tensor mask, idx, n, p;
    const float *ps = static_cast<const float*>(data(s)), *pu = static_cast<const float*>(data(u)), *pl = static_cast<const float*>(data(lut));
    const int32_t B = static_cast<int32_t>(lut.numel());
    if (failed("arrol_prune_bernoulli", launch([&] {
            uint8_t* pm = made<uint8_t>(mask, {N}, at::kByte, s);
            int32_t *pi = made<int32_t>(idx, {N}, at::kInt, s), *pn = made<int32_t>(n, {1}, at::kInt, s);
            return arrol_prune_bernoulli(ps, pu, N, pl, B, want ? made<float>(p, {N}, at::kFloat, s) : nullptr, pm, pi, pn, st);
        })))
        return nullptr;
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
PyObject* grpo_advantage(Args& a) {
    const at::Tensor &r = a.tensor(0, at::kFloat), &off = a.tensor(1, at::kLong);
    const int32_t ddof = a.integer(2);
    const float eps = static_cast<float>(a.number(3));
    if (a.odd || a.refuse(off.numel() < 1 || off.numel() > INT32_MAX)) return nullptr;
    const int64_t N = r.numel(), groups = off.numel() - 1;
    void* st = stream(a, r);
    if (a.odd) return nullptr;
    at::Tensor adv, wgt;
    const float* pr = static_cast<const float*>(data(r));
    const int64_t* po = static_cast<const int64_t*>(data(off));
    if (failed("arrol_grpo_advantage", launch([&] {
            float *pa = made<float>(adv, {N}, at::kFloat, r), *pw = made<float>(wgt, {N}, at::kFloat, r);
            return arrol_grpo_advantage_all(pr, po, N, groups, ddof, eps, pa, pw, st);
        })))
        return nullptr;
    return tuple(wrap(std::move(adv)), wrap(std::move(wgt)));
}

// logp, logp_ref, cu_seqlens, advantage, seq_weight, eps_low, eps_high, beta, want_grad, workspace
PyObject* grpo_objective(Args& a) {
    const at::Tensor &lp = a.tensor(0, at::kFloat), &cu = a.tensor(2, at::kLong);
    if (a.odd || a.refuse(cu.numel() < 1 || cu.numel() > INT32_MAX)) return nullptr;
    const int64_t T = lp.numel(), n = cu.numel() - 1;
    const float *pr = a.ptr<float>(1, at::kFloat, T), *pa = a.ptr<float>(3, at::kFloat, n), *pw = a.ptr<float>(4, at::kFloat, n);
    const float lo = static_cast<float>(a.number(5)), hi = static_cast<float>(a.number(6)), beta = static_cast<float>(a.number(7));
    const bool want = a.truth(8);
    if (a.refuse(!a.given(1) || !a.given(3) || !a.given(4))) return nullptr;
    void* st = stream(a, lp);
    if (a.odd) return nullptr;
    const size_t need = 8 * arrol_grpo_objective_workspace_bytes(static_cast<int32_t>(n));
    Scratch ws(a, 9, need > 16 ? need : 16);
    if (a.odd) return nullptr;
    at::Tensor J, grad, clip;
    const float* pl = static_cast<const float*>(data(lp));
    const int64_t* pc = static_cast<const int64_t*>(data(cu));
    if (failed("arrol_grpo_objective", launch([&] {
            ws.get(lp);
            double* pj = made<double>(J, {1}, at::kDouble, lp);
            int64_t* pn = made<int64_t>(clip, {1}, at::kLong, lp);
            return arrol_grpo_objective(pl, pr, pc, T, n, pa, pw, lo, hi, beta, pj, want ? made<float>(grad, {T}, at::kFloat, lp) : nullptr, pn, ws.p, ws.bytes, st);
        })))
        return nullptr;
    return tuple(wrap(std::move(J)), want ? wrap(std::move(grad)) : keep(Py_None), wrap(std::move(clip)));
}

template <PyObject* (*F)(Args&), int N>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t n) {
    if (n != N) {
        PyErr_Format(PyExc_TypeError, "%d arguments expected", N);
        return nullptr;
    }
    Args a{args};
    if (at::impl::PythonTorchFunctionTLS::stack_len() > 0 || c10::impl::TorchDispatchModeTLS::any_modes_set() ||
        at::globalContext().deterministicAlgorithms())
        Py_RETURN_NONE;
    PyObject* out = nullptr;
    try {
        out = F(a);
    } catch (...) {      // no memory, before anything was launched: torch.empty says so better
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    if (!out && a.odd) Py_RETURN_NONE;
    return out;
}

// What this file was compiled against: the header's version, and binding.py's interface number (raised there with every change of an
// argument list here), torch and Python (ARROL_BUILT_FOR, a text that the build gives).  binding.py looks at both before it calls anything else.
PyObject* built_for(PyObject*, PyObject*) { return Py_BuildValue("is", ARROL_VERSION, ARROL_BUILT_FOR); }

PyObject* setup(PyObject*, PyObject* const* args, Py_ssize_t n) {
    if (n != 3) {
        PyErr_SetString(PyExc_TypeError, "3 arguments expected");
        return nullptr;
    }
    PyObject** slots[3] = {&g_parameter, &g_policy, &g_check};
    for (int i = 0; i < 3; ++i) {
        Py_INCREF(args[i]);
        Py_XDECREF(*slots[i]);
        *slots[i] = args[i];
    }
    Py_RETURN_NONE;
}

#define ENTRY(name, n) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&entry<name, n>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"built_for", &built_for, METH_NOARGS, nullptr},
    {"setup", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&setup)), METH_FASTCALL, nullptr},
    ENTRY(score, 7), ENTRY(score_mlp, 7), ENTRY(score_grad, 6), ENTRY(score_mlp_grad, 9), ENTRY(adamw_step, 11), ENTRY(select, 7),
    ENTRY(weighted_vote, 5), ENTRY(histogram, 3), ENTRY(calibrate, 3), ENTRY(prune_bernoulli, 4), ENTRY(grpo_advantage, 4),
    ENTRY(grpo_objective, 10),
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&module); }
