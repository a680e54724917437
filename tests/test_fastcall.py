"""The binding's native calls (csrc/fastcall.cpp) against its Python: same results, same refusals.  The native module returns
None for what it does not take, so the comparison is with a binding whose module takes nothing; each call says whether the
native function has to take it."""
import shutil
import sys
import types
import warnings

import pytest
import torch

import paper_2511_19797_amd as tvm
from paper_2511_19797_amd import binding


class _Nothing:
    def __getattr__(self, name):
        return lambda *a: None


def outcome(fn, *a, **kw):
    try:
        r = fn(*a, **kw)
    except Exception as e:   # noqa: BLE001  (any refusal: its type and text are compared)
        return type(e), str(e)
    torch.cuda.synchronize()
    return r


class _Recorder:
    """The native module, noting which of its functions took their call."""

    def __init__(self):
        self.module = binding._load_fast()
        self.calls = []

    def __getattr__(self, name):
        def call(*a):
            r = getattr(self.module, name)(*a)
            self.calls.append((name, "python" if r is None else "native"))
            return r
        return call


def both(monkeypatch, name, route, fn, *a, **kw):
    """The call as it is, whose native function `name` has to take it ("native") or to leave it ("python"), against the call in
    Python."""
    seen = _Recorder()
    with monkeypatch.context() as mp:
        mp.setattr(binding, "_fast", seen)
        fast = outcome(fn, *a, **kw)
        mp.setattr(binding, "_fast", _Nothing())
        slow = outcome(fn, *a, **kw)
    assert seen.calls == [(name, route)]
    assert len(fast) == len(slow)
    for f, s in zip(fast, slow):
        if isinstance(s, torch.Tensor):
            assert f.shape == s.shape and f.stride() == s.stride() and f.dtype == s.dtype and f.device == s.device
            assert torch.equal(f, s) and not f.requires_grad
        else:
            assert f is s or f == s
    return fast


def took(name, *a):
    return getattr(binding._load_fast(), name)(*a) is not None


def test_takes_no_cpu_tensors_numbers_or_missing_arguments():
    """Nothing is taken that is not a plain tensor on the GPU; the Python behind raises as it did."""
    m = binding._load_fast()
    t = torch.zeros(1, 1, 4, 8)
    for name in ("jvp_fwd", "jvp_bwd", "qknorm_fwd", "bwd_qknorm", "adaln_fwd", "adaln_bwd", "gate_fwd", "gate_bwd", "gelu_fwd",
                 "gelu_bwd", "linear_fwd", "linear_bwd"):
        f = getattr(m, name)
        assert f() is None and f(1, 2, 3) is None and f(*[None] * 30) is None and f(*[t] * 28) is None
    with pytest.raises(ValueError, match="device tensors required"):
        tvm.tvmattn_jvp_fwd(t, t, t, t, t, t)
    with pytest.raises(ValueError):
        tvm.tvmattn_gelu_jvp_fwd(t, t)


MODULE = "paper_2511_19797_amd._fastcall"
# no module; one that cannot be loaded; one that is built for another torch or Python (or says nothing of it)
UNUSABLE = [None, "not a module", types.SimpleNamespace(built_for="torch 1.0, cpython-30"), types.SimpleNamespace()]


def without_module(mp, instead):
    mp.setattr(binding, "_fast", None)
    mp.delattr(tvm, "_fastcall", raising=False)
    if isinstance(instead, str):
        mp.setattr(tvm, "__path__", [instead])
        mp.delitem(sys.modules, MODULE, raising=False)
    else:
        mp.setitem(sys.modules, MODULE, instead)


@pytest.mark.parametrize("instead", UNUSABLE)
def test_calls_without_a_usable_module_go_through_python(monkeypatch, tmp_path, instead):
    """One warning, and what Python does from there on (here: its refusal of CPU tensors)."""
    t = torch.zeros(1, 1, 4, 8)
    with monkeypatch.context() as mp:
        if isinstance(instead, str):
            (tmp_path / "_fastcall.so").write_text(instead)
            instead = str(tmp_path)
        without_module(mp, instead)
        with pytest.warns(RuntimeWarning, match="_fastcall.so") as seen:
            for _ in range(2):
                with pytest.raises(ValueError, match="device tensors required"):
                    tvm.tvmattn_jvp_fwd(t, t, t, t, t, t)
        assert len(seen) == 1
    assert binding._load_fast().built_for == binding.native_target()


def test_native_calls_stay_with_the_library_beside_the_module(monkeypatch, tmp_path):
    """Another library in LIB_PATH serves all calls: the module, which is linked to the one beside it, takes none."""
    other = str(tmp_path / "libother.so")
    shutil.copy(binding.LIB_PATH, other)
    with monkeypatch.context() as mp, warnings.catch_warnings():
        warnings.simplefilter("error")
        mp.setattr(binding, "LIB_PATH", other)
        mp.setattr(binding, "_lib", None)
        mp.setattr(binding, "_fast", None)
        assert binding._load_fast() is not sys.modules.get(MODULE) and binding.lib()._name == other
        assert binding._load_fast().gelu_fwd() is None
    assert binding._load_fast() is sys.modules[MODULE]


@pytest.mark.gpu
def test_results_without_a_module(monkeypatch):
    x, tx = torch.randn(4, 64, device="cuda"), torch.randn(4, 64, device="cuda")
    want = tvm.tvmattn_gelu_jvp_fwd(x, tx)
    with monkeypatch.context() as mp:
        without_module(mp, None)
        with pytest.warns(RuntimeWarning, match="_fastcall.so"):
            got = tvm.tvmattn_gelu_jvp_fwd(x, tx)
    torch.cuda.synchronize()
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


def _attention(dtype, strided, seed=0):
    g = torch.Generator(device="cuda").manual_seed(seed)
    if strided:   # slices of fused [B,N,3,H,D] buffers
        buf = [torch.randn(2, 70, 3, 3, 24, generator=g, device="cuda").to(dtype) for _ in range(3)]
        return [b[:, :, i].permute(0, 2, 1, 3) for b in buf[:2] for i in range(3)] + [buf[2][:, :, i].permute(0, 2, 1, 3) for i in (0, 1)]
    return [torch.randn(2, 3, 70, 24, generator=g, device="cuda").to(dtype) for _ in range(8)]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("strided", [False, True])
def test_attention(monkeypatch, dtype, strided):
    q, k, v, tq, tk, tv, gO, gTO = _attention(dtype, strided)
    six = (q, k, v, tq, tk, tv)
    assert took("jvp_fwd", *six, 0.0, True, 0)
    for kw in ({}, {"save": False}, {"scale": 0.3}, {"flags": tvm.TVMATTN_FLAG_PLAIN_ALU}, {"flags": 64}):
        both(monkeypatch, "jvp_fwd", "native", tvm.tvmattn_jvp_fwd, *six, **kw)
    saved = tvm.tvmattn_jvp_fwd(*six)
    for a, b in ((gO, gTO), (gO, None), (None, gTO), (None, None)):
        both(monkeypatch, "jvp_bwd", "native", tvm.tvmattn_jvp_bwd, *six, *saved, a, b)
    both(monkeypatch, "jvp_bwd", "native", tvm.tvmattn_jvp_bwd, q, k, v, None, None, None, saved[0], None, saved[2], None, gO, None)
    half = q[:, :, :35]                         # fewer queries than keys, and layouts that do not match
    both(monkeypatch, "jvp_fwd", "native", tvm.tvmattn_jvp_fwd, half, k, v, tq[:, :, :35], tk, tv)
    both(monkeypatch, "jvp_fwd", "python", tvm.tvmattn_jvp_fwd, half, k, v, tq, tk, tv)
    both(monkeypatch, "jvp_fwd", "python" if strided else "native", tvm.tvmattn_jvp_fwd, q, k, v.contiguous(), tq, tk, tv)
    both(monkeypatch, "jvp_fwd", "python", tvm.tvmattn_jvp_fwd, q.half(), k, v, tq.half(), tk, tv)
    both(monkeypatch, "jvp_fwd", "python", tvm.tvmattn_jvp_fwd, *[t.transpose(2, 3) for t in six])
    both(monkeypatch, "jvp_fwd", "native", tvm.tvmattn_jvp_fwd, *[t[..., :20] for t in six])       # alignment: refused by the entry point
    both(monkeypatch, "jvp_fwd", "python", tvm.tvmattn_jvp_fwd, *[t[0] for t in six])
    both(monkeypatch, "jvp_fwd", "native", tvm.tvmattn_jvp_fwd, *[t.detach().requires_grad_() for t in six])


@pytest.mark.gpu
def test_norm_and_fused_backward(monkeypatch):
    q, k, v, tq, tk, tv, gO, gTO = _attention(torch.bfloat16, True, 1)
    gq, gk = torch.rand(24, device="cuda") + 0.5, torch.rand(24, device="cuda") + 0.5
    qn, tqn, kn, tkn = both(monkeypatch, "qknorm_fwd", "native", tvm.tvmattn_qknorm_jvp_fwd, q, tq, k, tk, gq, gk, 1e-6)
    both(monkeypatch, "qknorm_fwd", "python", tvm.tvmattn_qknorm_jvp_fwd, q, tq, k, tk, gq.bfloat16(), gk, 1e-6)
    both(monkeypatch, "qknorm_fwd", "python", tvm.tvmattn_qknorm_jvp_fwd, q, tq, k, tk, gq[:16], gk, 1e-6)
    saved = tvm.tvmattn_jvp_fwd(qn, kn, v, tqn, tkn, tv)
    make = lambda: tuple(binding._like(t) for t in (q, k, v, tq, tk, tv)) + (torch.empty_like(gq), torch.empty_like(gk))
    args = (q, tq, k, tk, gq, gk, 1e-6, qn, tqn, kn, tkn, v, tv, *saved, gO, gTO)
    out = make()
    assert tvm.tvmattn_jvp_bwd_qknorm(*args, out=out) is out
    both(monkeypatch, "bwd_qknorm", "native", lambda: tvm.tvmattn_jvp_bwd_qknorm(*args, out=make()))
    both(monkeypatch, "bwd_qknorm", "python", lambda: tvm.tvmattn_jvp_bwd_qknorm(*args, out=make()[:6] + (gq.bfloat16(), torch.empty_like(gk))))


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_token_calls(monkeypatch, dtype):
    g = torch.Generator(device="cuda").manual_seed(3)
    x, tx, h, th, gy, gty, r, tr = (torch.randn(2, 33, 64, generator=g, device="cuda").to(dtype) for _ in range(8))
    m = [torch.randn(2, 64, generator=g, device="cuda") for _ in range(4)]
    for route, a in (("native", (x, tx, *m)), ("python", (x, tx[:, :32], *m)), ("python", (x.transpose(0, 1), tx.transpose(0, 1), *m)),
                     ("python", (x, tx, m[0].to(dtype).double(), *m[1:])), ("python", (x, tx, *m[:3], m[3][:1])),
                     ("native", (x[..., :61].contiguous(), tx[..., :61].contiguous(), *[t[:, :61].contiguous() for t in m]))):
        both(monkeypatch, "adaln_fwd", route, tvm.tvmattn_adaln_jvp_fwd, *a, 1e-6)
    both(monkeypatch, "adaln_bwd", "native", tvm.tvmattn_adaln_jvp_bwd, x, tx, *m, 1e-6, gy, gty)
    both(monkeypatch, "adaln_bwd", "native", tvm.tvmattn_adaln_jvp_bwd, x, tx, *m, 1e-6, gy, gty, gres=r, gtres=tr)
    both(monkeypatch, "adaln_bwd", "python", tvm.tvmattn_adaln_jvp_bwd, x, tx, *m, 1e-6, gy, gty, gres=r)
    both(monkeypatch, "gate_fwd", "native", tvm.tvmattn_gate_jvp_fwd, x, tx, h, th, *m[:2], 1e-6)
    both(monkeypatch, "gate_fwd", "python", tvm.tvmattn_gate_jvp_fwd, x, tx, h[:1], th[:1], *m[:2], 1e-6)
    both(monkeypatch, "gate_bwd", "native", tvm.tvmattn_gate_jvp_bwd, h, th, *m[:2], 1e-6, gy, gty)
    both(monkeypatch, "gelu_fwd", "native", tvm.tvmattn_gelu_jvp_fwd, x, tx)
    both(monkeypatch, "gelu_fwd", "python", tvm.tvmattn_gelu_jvp_fwd, x[:, ::2], tx[:, ::2])
    both(monkeypatch, "gelu_bwd", "native", tvm.tvmattn_gelu_jvp_bwd, x, tx, gy, gty)
    both(monkeypatch, "gelu_bwd", "python", tvm.tvmattn_gelu_jvp_bwd, x, tx, gy, gty.double())


@pytest.mark.gpu
def test_linear(monkeypatch):
    g = torch.Generator(device="cuda").manual_seed(4)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").bfloat16()
    x, tx, w, b, gy, gty = rnd(2, 50, 96), rnd(2, 50, 96), rnd(64, 96), rnd(64), rnd(100, 64), rnd(100, 64)
    wide, twide = rnd(100, 200), rnd(100, 200)
    for route, a in (("native", (x, tx, w, b)), ("native", (x, tx, w, None)), ("native", (wide[:, :96], twide[:, :96], w, b)),
                     ("python", (x[:, ::2], tx[:, ::2], w, b)), ("python", (x, tx, w.t(), b)), ("python", (x, tx[:1], w, b)),
                     ("python", (x, tx, w, b[:32])), ("native", (x.float(), tx.float(), w.float(), None)),
                     ("python", (x[..., :40], tx[..., :40], w[:, :40].contiguous(), None)), ("native", (x[:0], tx[:0], w, b))):
        both(monkeypatch, "linear_fwd", route, tvm.tvmattn_linear_jvp_fwd, *a)
    x2, tx2 = x.view(100, 96), tx.view(100, 96)
    for route, a in (("native", (x2, tx2, w, gy, gty)), ("native", (x, tx, w, gy, gty)), ("native", (wide[:, :96], twide[:, :96], w, gy, gty)),
                     ("native", (x2, tx2, w, wide[:, :64], twide[:, :64])), ("python", (x2, tx2, w, gy[:50], gty[:50])),
                     ("python", (x2, tx2, w, gy, gty.float()))):
        both(monkeypatch, "linear_bwd", route, tvm.tvmattn_linear_jvp_bwd, *a)
    r = both(monkeypatch, "linear_bwd", "native", tvm.tvmattn_linear_jvp_bwd, x2, tx2, w, gy, gty, bias_grad=False)
    assert r[3] is None


@pytest.mark.gpu
def test_modes_and_transforms_go_the_python_way():
    x = torch.randn(4, 64, device="cuda")

    class Mode(torch.overrides.TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))

    assert took("gelu_fwd", x, x)
    with Mode():
        assert not took("gelu_fwd", x, x)
    with torch.utils._python_dispatch.TorchDispatchMode():
        assert not took("gelu_fwd", x, x)
    seen = []
    torch.func.vmap(lambda t: (seen.append(took("gelu_fwd", t, t)), t)[1])(x)
    torch.func.jvp(lambda t: (seen.append(took("gelu_fwd", t, t)), t)[1], (x,), (x,))
    assert seen == [False, False]


@pytest.mark.gpu
def test_runs_on_the_current_stream():
    """The call goes to the current stream: work queued behind it there sees its results, a graph captures it."""
    x, tx = torch.randn(1 << 20, device="cuda"), torch.randn(1 << 20, device="cuda")
    ref = tvm.tvmattn_gelu_jvp_fwd(x, tx)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        a, _ = tvm.tvmattn_gelu_jvp_fwd(x, tx)
        c = a.clone()
    s.synchronize()
    assert torch.equal(c, ref[0])
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        r = tvm.tvmattn_gelu_jvp_fwd(x, tx)
    for k in range(3):
        x.mul_(0.5)
        graph.replay()
        torch.cuda.synchronize()
        want = tvm.tvmattn_gelu_jvp_fwd(x, tx)
        torch.cuda.synchronize()
        assert torch.equal(r[0], want[0]) and torch.equal(r[1], want[1])
