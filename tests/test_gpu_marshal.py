"""The marshalling module against the general way through ctypes: the same outputs, the same errors, and calls it leaves alone."""
import numpy as np
import pytest
import torch
from torch.overrides import TorchFunctionMode
from torch.utils._python_dispatch import TorchDispatchMode

from paper_2411_04965_amd import binding as B

pytestmark = pytest.mark.gpu
BF16 = torch.bfloat16


class Sub(torch.Tensor):
    pass


class Quiet(TorchFunctionMode):
    def __torch_function__(self, func, types, args=(), kwargs=None):
        return func(*args, **(kwargs or {}))


def both(monkeypatch, call):
    """(kind, value or error) of `call` natively and through ctypes."""
    got = []
    native = B._native()
    assert native
    for m in (native, False):
        monkeypatch.setattr(B, "_marshal", m)
        if m is False:
            monkeypatch.setattr(B, "_native", lambda: False)
        try:
            got.append(("value", call()))
        except Exception as e:
            got.append((type(e), str(e)))
    return got


def test_same_outputs_and_errors(monkeypatch):
    g = torch.Generator(device="cuda").manual_seed(5)
    M, N, K = 9, 70, 264
    X = torch.randn((M, K), generator=g, device="cuda")
    W = torch.randn((N, K), generator=g, device="cuda")
    packs = {l: B.pack_ternary(W, layout=l) for l in (B.BL_W_GEMM, B.BL_W_MX2, B.BL_W_MX4)}
    p, a = packs[B.BL_W_GEMM]
    Xb = X.to(BF16)
    ws = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    small = torch.empty(16, dtype=torch.uint8, device="cuda")
    calls = []
    for x in (X, Xb, torch.nn.Parameter(X), X.as_subclass(Sub), X.half(), X.T, X.cpu(), X[0], X[:0]):
        calls += [lambda x=x: B.bitlinear_a4(x, p, a, N), lambda x=x: B.bitlinear_a8_sparse(x, 100, p, a, N),
                  lambda x=x: B.bitlinear_a4_gate_up(x, p, a, p, a, N, want=("H",))["H"]]
    for l, (pl, al) in packs.items():
        for fp4 in (False, True):
            calls += [lambda pl=pl, al=al, l=l, f=fp4: B.bitlinear_a4(Xb, pl, al, N, act_fp4=f, y_dtype=torch.float32, layout=l)]
        calls += [lambda pl=pl, al=al, l=l: B.bitlinear_a4_gate_up(Xb, pl, al, pl, al, N, layout=l, want=("H",))["H"]]
    out = torch.empty((M, N), dtype=BF16, device="cuda")
    calls += [lambda: B.bitlinear_a4(Xb, p, a, N, ws=ws, out=out), lambda: B.bitlinear_a8_sparse(Xb, 100, p, a, N, ws=ws, out=out),
              lambda: B.bitlinear_a4_gate_up(Xb, p, a, p, a, N, want=("H",), ws=ws, out={"H": out})["H"],
              lambda: B.bitlinear_a4_gate_up(Xb, p, a, p, a, N, want=("H", "G"))["G"],
              lambda: B.bitlinear_a4(Xb, p, a, N, want_acc=True)[1],
              lambda: B.bitlinear_a4(Xb, p, a, N, ws=small), lambda: B.bitlinear_a8_sparse(Xb, 0, p, a, N),
              lambda: B.bitlinear_a8_sparse(Xb, K + 1, p, a, N), lambda: B.bitlinear_a4(Xb, None, a, N), lambda: B.bitlinear_a4(Xb, p, a, 0),
              lambda: B.bitlinear_a4(Xb, p, a, N, eps=-1.0), lambda: B.bitlinear_a4(Xb, p, a, N, eps=0), lambda: B.bitlinear_a4(Xb, p, a, 1.5),
              lambda: B.bitlinear_a4(Xb, p, a, np.int64(N)), lambda: B.bitlinear_a4(Xb, p, a, True), lambda: B.bitlinear_a4(Xb, p, a, N, layout=3),
              lambda: B.bitlinear_a4(Xb, p, a, N, layout=9), lambda: B.bitlinear_a4(Xb, p, a, N, act_fp4=1),
              lambda: B.bitlinear_a4(Xb, p, a, N, y_dtype=torch.half), lambda: B.bitlinear_a4(Xb, p, a, N, out=out.half()),
              lambda: B.bitlinear_a4(Xb, p, a, 1 << 40), lambda: B.bitlinear_a4(Xb[:, 1:9].contiguous()[:, :], p, a, N)]
    for i, call in enumerate(calls):
        with monkeypatch.context() as mp:
            n, c = both(mp, call)
        assert n[0] == c[0], (i, n, c)
        if n[0] == "value":
            assert type(n[1]) is type(c[1]) and n[1].dtype == c[1].dtype and torch.equal(n[1], c[1]), i
            assert n[1].requires_grad == c[1].requires_grad
        elif issubclass(n[0], B.BitlinearError) or n[0] in (ValueError, TypeError):
            assert n[1] == c[1], i


def test_plain_calls_only():
    """Plain calls are taken by the module itself, returned outputs are the caller's own; function modes and subclasses take the general way."""
    X = torch.randn((3, 256), device="cuda").to(BF16)
    p, a = B.pack_ternary(torch.randn((32, 256), device="cuda"))
    m = B._native()
    out = torch.empty((3, 32), dtype=BF16, device="cuda")
    d = {"H": out}
    assert B.bitlinear_a4(X, p, a, 32, out=out) is out
    r = B.bitlinear_a4_gate_up(X, p, a, p, a, 32, want=("H",), out=d)
    assert r["H"] is out and r is not d and list(r) == ["H"]
    args = (p, a, 32, 1e-5, False, BF16, None, None, 0)
    ws = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    for w, o in ((None, None), (ws, out)):
        for x in (X, X.float(), torch.nn.Parameter(X)):
            assert torch.is_tensor(m.a4(x, p, a, 32, 1e-5, False, BF16, w, o, 0))
            assert torch.is_tensor(m.a8_sparse(x, 8, p, a, 32, 1e-5, 0, BF16, w, o))
            assert type(m.gate_up(x, p, a, p, a, 32, 1e-5, 0, ("H",), w, None if o is None else {"H": o})) is dict
    assert m.a4(X.as_subclass(Sub), *args) is None and m.a4(X.float().half(), *args) is None
    with Quiet():
        assert m.a4(X, *args) is None
        assert torch.equal(B.bitlinear_a4(X, p, a, 32), B.bitlinear_a4(X, p, a, 32, want_acc=True)[0])
    ref = B.bitlinear_a4(X, p, a, 32)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        y = B.bitlinear_a4(X, p, a, 32)
    torch.cuda.current_stream().wait_stream(s)
    y.record_stream(torch.cuda.current_stream())
    assert torch.equal(y, ref)


class Refuses(TorchDispatchMode):
    def __torch_dispatch__(self, func, types, args=(), kwargs=None):
        raise KeyError("no allocation here")


def test_errors_of_a_dispatch_mode(monkeypatch):
    """What a dispatch mode raises in the allocation of workspace or output reaches the caller as it is."""
    X = torch.randn((3, 256), device="cuda").to(BF16)
    p, a = B.pack_ternary(torch.randn((32, 256), device="cuda"))
    for call in (lambda: B.bitlinear_a4(X, p, a, 32), lambda: B.bitlinear_a8_sparse(X, 8, p, a, 32),
                 lambda: B.bitlinear_a4_gate_up(X, p, a, p, a, 32, want=("H",))):
        def inside(call=call):
            with Refuses():
                return call()
        with monkeypatch.context() as mp:
            n, c = both(mp, inside)
        assert n == c and n[0] is KeyError, (n, c)
    assert torch.equal(B.bitlinear_a4(X, p, a, 32), B.bitlinear_a4(X, p, a, 32, want_acc=True)[0])
