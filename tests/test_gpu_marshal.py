"""The C++ marshalling of the short calls (csrc/marshal.cpp) against the Python marshalling of the same calls: the same
results, the same errors, and None - so the Python way - for everything but the ordinary case."""
import inspect
import sys

import numpy as np
import pytest
import torch

import paper_2603_24840_amd as A
from paper_2603_24840_amd import binding

DEV = "cuda:0"


def calls(dev):
    g = torch.Generator().manual_seed(5)

    def f(*shape):
        return torch.randn(shape, generator=g).to(dev)

    def ints(hi, n, dtype):
        return torch.randint(0, hi, (n,), generator=g).to(dtype).to(dev)

    def scratch():                                           # of the caller's own
        return torch.zeros(1 << 20, dtype=torch.uint8, device=dev)
    h, w = f(96, 128).bfloat16(), f(128)
    idx = torch.arange(0, 96, 3).to(dev)
    y96, y32 = ints(2, 96, torch.float32), ints(2, 32, torch.float32)
    w1, b1, w2 = f(40, 128).bfloat16(), f(40), f(40)
    prob, uni = torch.rand(96, generator=g).to(dev), torch.rand(96, generator=g).to(dev)
    cu, off = torch.tensor([0, 20, 50, 96]).to(dev), torch.tensor([0, 48, 90]).to(dev)
    cp, cn = ints(50, 64, torch.int64), ints(50, 64, torch.int64)
    pol = A.Policy(0.5, 0.5, 0.5, 0.05, 0.95, 1.0)
    adam = [f(97), f(97), f(97) * 0.01, f(97).abs() * 0.01]
    return {
        "score": [((h, w), {}), ((h, w, 0.5, idx), {}), ((h[::2], w, 1), dict(want_score=False)), ((h, w, np.float32(0.3)), {}), ((h, w, np.int64(2)), {}),
                  ((h, w, torch.tensor(0.7)), {}), ((h[:1], torch.nn.Parameter(w)), {}),
                  ((h, w), dict(out_score=torch.empty(96, device=dev), out_prob=torch.empty(96, device=dev)))],
        "score_mlp": [((h, w1, b1, w2), {}), ((h, w1, None, w2, 0.25), dict(row_index=idx)), ((h, w1, b1, w2), dict(workspace=None)),
                      ((h, w1, b1, w2), dict(workspace=scratch()))],
        "score_grad": [((h, w, 0.0, y96), {}), ((h, w, 0.5, y32), dict(row_index=idx)), ((h, w, 0.0, y96), dict(workspace=scratch()))],
        "score_mlp_grad": [((h, w1, b1, w2, 0.0, y96), {}), ((h, w1, None, w2, 0.25, y32), dict(row_index=idx, delta_terms=2)),
                           ((h, w1, b1, w2, 0.0, y96), dict(workspace=scratch()))],
        "adamw_step": [((*adam, 3, 1e-3), {}), ((*adam, 7, 1e-3), dict(weight_decay=0.1, param_bf16=torch.zeros(97, dtype=torch.bfloat16, device=dev)))],
        "select": [((prob, 12, 8, 3), {}), ((prob, 6, 16, 16, 0.25), {})],
        "weighted_vote": [((prob, ints(9, 96, torch.int32), 12, 8, 9), {}), ((prob, ints(9, 96, torch.int32), 12, 8, 9), dict(want_tally=True))],
        "histogram": [((prob, ints(2, 96, torch.uint8), 64), {})],
        "calibrate": [((cp, cn, pol), {})],
        "prune_bernoulli": [((prob, uni, torch.rand(64, generator=g).to(dev)), {}), ((prob, uni, torch.rand(64, generator=g).to(dev)), dict(want_p=True))],
        "grpo_advantage": [((f(96), off), {}), ((f(96), off, 1, 1e-6), {})],
        "grpo_objective": [((f(96) * 0.1, f(96) * 0.1, cu, f(3), f(3).abs()), {}), ((f(96), f(96), cu, f(3), f(3).abs(), 0.2, 0.28, 0.04), dict(want_grad=False)),
                           ((f(96), f(96), cu, f(3), f(3).abs()), dict(workspace=scratch()))],
    }


def flat(out):
    if isinstance(out, dict):
        return [(k, out[k]) for k in sorted(out)]
    return list(enumerate(out)) if isinstance(out, tuple) else [(0, out)]


def clone(x):
    return x.clone() if isinstance(x, torch.Tensor) and not isinstance(x, torch.nn.Parameter) and x.is_contiguous() else x


def native(name, args, kw):
    """The extension's own answer to a call of the public function: None where it leaves the call to Python."""
    bound = inspect.signature(getattr(A, "arrol_" + name)).bind(*args, **kw)
    bound.apply_defaults()
    leave = ("stream", "want_tally", "out_winner")           # what the public function looks at before it asks the extension
    return getattr(binding._load_marshal(), name)(*[v for k, v in bound.arguments.items() if k not in leave])


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(calls("cpu")))
def test_native_marshalling_gives_what_python_gives(name):
    """Asked directly, so that a call which the extension leaves to Python is no pass; everything that a call writes is
    compared bit for bit, its own arguments (the optimizer's state, given outputs) among it."""
    print("[case] marshal", name, flush=True)
    public, slow = getattr(A, "arrol_" + name), getattr(binding, "_py_" + name)
    for args, kw in calls(DEV)[name]:
        ways = [lambda a, k: slow(*a, **k), lambda a, k: public(*a, **k)]
        if not kw.get("want_tally"):                         # which the extension is never asked for
            ways.append(lambda a, k: native(name, a, k))
        results = []
        for way in ways:
            a, k = [clone(x) for x in args], {key: clone(v) for key, v in kw.items()}
            out = way(a, k)
            assert out is not None
            results.append(flat(out) + flat(tuple(a)) + [kv for kv in flat(k) if kv[0] != "workspace"])
            assert len(results) == 1 or type(out) is kind
            kind = type(out)
        torch.cuda.synchronize()
        for other in results[1:]:
            assert [k for k, _ in other] == [k for k, _ in results[0]]
            for (k, x), (_, y) in zip(results[0], other):
                assert isinstance(x, torch.Tensor) == isinstance(y, torch.Tensor), k
                if isinstance(x, torch.Tensor):
                    assert x.dtype == y.dtype and x.shape == y.shape, k
                    assert torch.equal(x.reshape(-1).view(torch.uint8), y.reshape(-1).view(torch.uint8)), k


@pytest.mark.gpu
def test_native_marshalling_takes_the_ordinary_case_only():
    m = binding._load_marshal()
    h, w = torch.zeros(8, 64, dtype=torch.bfloat16, device=DEV), torch.zeros(64, device=DEV)
    ok = [h, w, 0.0, None, None, None, True]

    class Sub(torch.Tensor):
        pass
    assert m.score(*ok) is not None
    for i, odd in ((0, h.float()), (0, h[0]), (0, h.t()), (0, h.as_subclass(Sub)), (0, h.cpu()), (1, w.double()), (1, w.cpu()),
                   (1, torch.zeros(128, device=DEV)[::2]), (2, "0"), (2, None), (3, torch.zeros(8, dtype=torch.int32, device=DEV)), (5, w.half()), (6, 1)):
        assert m.score(*ok[:i], odd, *ok[i + 1:]) is None, (i, odd)
    y, ws = torch.zeros(8, device=DEV), torch.zeros(1 << 16, dtype=torch.uint8, device=DEV)
    grad = [h, w, 0.0, y, None]
    assert m.score_grad(*grad, ws) is not None
    for odd in (ws.float(), ws.cpu(), "auto", ws[::2]):
        assert m.score_grad(*grad, odd) is None, odd
    with pytest.raises(A.ArrolError):                        # too small: the library says so
        A.arrol_score_grad(*grad, workspace=ws[:4])
    prob = torch.zeros(16, device=DEV)
    for bad in ((prob, 2, 9, 1), (prob, 2 ** 32 + 2, 8, 1), (prob, -2, -8, 1), (prob, 2.0, 8, 1)):
        assert m.select(*bad, 0.5, None, None) is None
    assert m.calibrate(torch.zeros(4, dtype=torch.int64, device=DEV), torch.zeros(4, dtype=torch.int64, device=DEV), b"x" * 24) is None
    from torch.utils._python_dispatch import TorchDispatchMode

    class Mode(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))
    with Mode():
        assert m.score(*ok) is None
    with torch.device(DEV):
        assert m.score(*ok) is None
    with pytest.raises(A.ArrolError):                        # the library's own refusal: d not a multiple of 8
        A.arrol_score(torch.zeros(2, 12, dtype=torch.bfloat16, device=DEV), torch.zeros(12, device=DEV))
    with pytest.raises(TypeError):
        A.arrol_score(h.float(), w)


def test_native_marshalling_leaves_cpu_tensors_to_python():
    m = binding._load_marshal()
    for name, cases in calls("cpu").items():
        args, kw = cases[0]
        with pytest.raises((TypeError, ValueError)):
            getattr(A, "arrol_" + name)(*args, **kw)
    assert m.histogram(torch.zeros(4), torch.zeros(4, dtype=torch.uint8), 4) is None
    with pytest.raises(TypeError):
        m.histogram(torch.zeros(4))


def test_leaving_a_call_to_python_costs_next_to_nothing():
    """What the extension does not take - a tensor subclass, a strided vector, an active mode - pays for the question on top of
    Python's way: 0.07 us on the machine this was written on, 3 us when the answer was a C++ exception, and a call of the same
    form that does nothing 0.04."""
    import math
    import time
    m = binding._load_marshal()
    x, l = torch.zeros(4), torch.zeros(4, dtype=torch.uint8)

    def best(f, *args):
        times = []
        for _ in range(30):
            t = time.perf_counter()
            for _ in range(500):
                f(*args)
            times.append(time.perf_counter() - t)
        return min(times)
    nothing = best(math.gcd, 4, 6)
    assert best(m.histogram, x, l, 4) < 20 * nothing
    assert best(m.score_grad, x, x, 0.0, x, None, l) < 20 * nothing


@pytest.fixture
def reload_marshal(monkeypatch):
    """The extension is loaded again in the test, and again after it."""
    monkeypatch.setattr(binding, "_marshal", None)


def python_refuses(name="score"):
    args, kw = calls("cpu")[name][0]
    with pytest.warns(RuntimeWarning, match="marshalled in Python"):
        with pytest.raises(TypeError):                       # by the Python marshalling, which looks at the device
            getattr(A, "arrol_" + name)(*args, **kw)
    assert isinstance(binding._marshal, binding._NoMarshal)


def test_calls_go_by_python_where_only_the_library_is_built(reload_marshal, monkeypatch, tmp_path):
    monkeypatch.setattr(binding, "MARSHAL_PATH", str(tmp_path / "_marshal.so"))
    python_refuses()


@pytest.mark.parametrize("what,value", [("ABI_VERSION", 201), ("built_for", lambda: "torch 0.0, python 3.10")])
def test_an_extension_built_for_something_else_is_not_used(reload_marshal, monkeypatch, what, value):
    monkeypatch.setattr(binding, what, value)
    python_refuses()


def test_a_file_that_is_no_extension_is_not_used(reload_marshal, monkeypatch, tmp_path):
    (tmp_path / "_marshal.so").write_bytes(b"not this")
    monkeypatch.setattr(binding, "MARSHAL_PATH", str(tmp_path / "_marshal.so"))
    python_refuses()


# Of the library's version, torch and Python of today, as a file that outlives a change of marshal.cpp is: one without the
# interface in its text, one whose setup() wants other arguments, and one that fits, for the difference
@pytest.mark.parametrize("text,setup,used", [("torch %s, python %d.%d" % ((torch.__version__,) + sys.version_info[:2]), "*a", False),
                                             (binding.built_for(), "a, b, c, d, e", False), (binding.built_for(), "a, b, c", True)])
def test_an_extension_of_another_binding_is_not_used(reload_marshal, monkeypatch, tmp_path, text, setup, used):
    (tmp_path / "_marshal.py").write_text("def built_for(): return %r\ndef setup(%s): pass\ndef score(*a): return 'taken'\n" %
                                          ((binding.ABI_VERSION, text), setup))
    monkeypatch.setattr(binding, "MARSHAL_PATH", str(tmp_path / "_marshal.py"))
    if used:
        assert A.arrol_score(*calls("cpu")["score"][0][0]) == "taken"
    else:
        python_refuses()


def test_the_extension_says_what_it_is_compiled_against():
    import os
    import re
    header = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "include", "arrol.h")
    macro = int(re.search(r"#define ARROL_VERSION (\d+)", open(header).read()).group(1))
    assert binding._load_marshal().built_for() == (macro, binding.built_for())
    assert macro == A.version() == binding.ABI_VERSION


def test_build_without_a_host_compiler_keeps_the_library(monkeypatch, tmp_path):
    from paper_2603_24840_amd import build
    ran = []

    def run(cmd, verbose):
        ran.append(cmd)
        if "marshal.cpp" in " ".join(cmd):
            raise OSError("no such program: " + cmd[0])
    for name, value in (("_run", run), ("LIB_DIR", str(tmp_path)), ("LIB_PATH", str(tmp_path / "libarrol.so")),
                        ("MARSHAL_PATH", str(tmp_path / "_marshal.so")), ("hipcc_path", lambda: "hipcc")):
        monkeypatch.setattr(build, name, value)
    monkeypatch.setenv("CXX", "none -m64")
    (tmp_path / "_marshal.so").write_bytes(b"an older one")
    with pytest.warns(RuntimeWarning, match="built without _marshal.so"):
        assert build.build(verbose=False) == build.LIB_PATH
    assert ran[0][0] == "hipcc" and ran[1][:2] == ["none", "-m64"] and not (tmp_path / "_marshal.so").exists()


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(calls("cpu")))
def test_calls_without_the_extension(monkeypatch, name):
    monkeypatch.setattr(binding, "_marshal", binding._NoMarshal())
    for args, kw in calls(DEV)[name]:
        assert getattr(A, "arrol_" + name)(*[clone(a) for a in args], **{k: clone(v) for k, v in kw.items()}) is not None
    torch.cuda.synchronize()
