"""The launching calls on torch tensors: what the extension module takes and what it leaves to the binding's own marshalling give the
same bits, and the same errors."""
import pytest
import torch

import paper_2507_11978_amd as nt

pytestmark = pytest.mark.gpu


class Tagged(torch.Tensor):
    """A tensor subclass: not the extension module's."""


def t(*shape, dt=torch.float16, seed=0):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float32).to(dt)


def calls():
    a, b, x, w = t(40, 72), t(72, 56, seed=1), t(2, 32, 9, 9, seed=2), t(16, 32, 3, 3, seed=3)
    q, row, full = t(1, 2, 70, 64, seed=4), t(56, seed=5), t(40, 56, seed=6)
    e = lambda *s: torch.full(s, float("nan"), dtype=torch.float16, device="cuda")
    return {
        "gemm": lambda f, **k: nt.gemm(f(a), f(b), e(40, 56), **k),
        "gemm tile": lambda f, **k: nt.gemm(f(a), f(b), e(40, 56), tile=[64, 64, 32], **k),
        "gemm transposed": lambda f, **k: nt.gemm(f(b.t()), f(a.t()), e(56, 40), **k),
        "bmm": lambda f, **k: nt.bmm(f(a.expand(3, 40, 72)), f(b.expand(3, 72, 56)), e(3, 40, 56), **k),
        "addmm row": lambda f, **k: nt.addmm(f(row), f(a), f(b), e(40, 56), alpha=0.5, beta=2, act="silu", **k),
        "addmm full": lambda f, **k: nt.addmm(f(full), f(a), f(b), e(40, 56), **k),
        "addmm one": lambda f, **k: nt.addmm(f(full[:1, :1]), f(a), f(b), e(40, 56), **k),
        "conv2d": lambda f, **k: nt.conv2d_implicit(f(x), f(w), e(2, 16, 5, 5), (2, 2), [1, 1], **k),
        "sdpa": lambda f, **k: nt.sdpa(f(q), f(q), f(q), e(1, 2, 70, 64), **k),
        "softmax": lambda f, **k: nt.softmax(f(a), e(40, 72), **k),
        "rms_norm": lambda f, **k: nt.rms_norm(f(a), e(40, 72), **k),
        "add": lambda f, **k: nt.add(f(row), f(row), e(56), **k),
        "silu": lambda f, **k: nt.silu(f(row), e(56), **k),
    }


@pytest.mark.parametrize("name", ["gemm", "gemm tile", "gemm transposed", "bmm", "addmm row", "addmm full", "addmm one", "conv2d", "sdpa", "softmax", "rms_norm", "add", "silu"])
def test_every_way_gives_the_same_bits(name):
    run = calls()[name]
    want = run(lambda v: v)
    assert torch.isfinite(want).all()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    got = [run(lambda v: torch.nn.Parameter(v, requires_grad=False)), run(lambda v: v.as_subclass(Tagged)), run(lambda v: v, stream=torch.cuda.current_stream())]
    with torch.cuda.stream(side):
        got.append(run(lambda v: v))
    torch.cuda.synchronize()
    assert all(torch.equal(g, want) for g in got)


def test_errors_stay_what_they_were():
    a, b, c = t(8, 16), t(16, 8, seed=1), t(8, 8, seed=2)
    with pytest.raises(nt.NtError) as err:
        nt.gemm(a, b, t(8, 9))
    assert err.value.name == "NT_ERR_SHAPE_MISMATCH" and "output shape" in str(err.value)
    with pytest.raises(nt.NtError, match="2-D"):
        nt.gemm(a[None], b, c)
    with pytest.raises(nt.NtError, match="input shape"):
        nt.addmm(t(8, 8)[:7], a, b, c)
    with pytest.raises(nt.NtError, match="no kernel built"):
        nt.gemm(a, b, c, tile=(48, 64, 32))
    with pytest.raises(ValueError, match="GPU"):
        nt.gemm(a.cpu(), b, c)
    with pytest.raises(ValueError, match="activation"):
        nt.addmm(c, a, b, c, act="tanh")
    with pytest.raises(ValueError, match="dtype"):
        nt.addmm(c.float(), a, b, c)
    with pytest.raises(KeyError):
        nt.gemm(a.double(), b, c)
    with pytest.raises(nt.NtError, match="input dtype"):
        nt.gemm(a.float(), b.float(), c)
    with pytest.raises(AttributeError):
        nt.gemm([[1.0]], b, c)


def test_what_the_module_takes_and_what_it_declines():
    """Its own functions, so that a module that declined everything, or ran nothing, would not pass for the binding."""
    module = nt.binding._calls or nt.binding._load_calls()
    assert type(module).__name__ == "module"
    a, b, row, q = t(40, 72), t(72, 56, seed=1), t(56, seed=5), t(1, 2, 70, 64, seed=4)
    x, w = t(2, 32, 9, 9, seed=2), t(16, 32, 3, 3, seed=3)
    e = lambda *s: torch.full(s, float("nan"), dtype=torch.float16, device="cuda")
    taken = {"gemm": lambda f, o: module.gemm(f(a), f(b), o, None, None), "bmm": lambda f, o: module.bmm(f(a[None]), f(b[None]), o, [64, 64, 32], None),
             "addmm": lambda f, o: module.addmm(f(row), f(a), f(b), o, 1.0, 2.0, 2, None, None), "conv2d": lambda f, o: module.conv2d(f(x), f(w), o, (2, 2), (1, 1), None, None),
             "sdpa": lambda f, o: module.sdpa(f(q), f(q), f(q), o, 0.0, None), "softmax": lambda f, o: module.softmax(f(a), o, None),
             "rms_norm": lambda f, o: module.rms_norm(f(a), o, 1e-6, None), "add": lambda f, o: module.add(f(row), f(row), o, 0, None), "silu": lambda f, o: module.silu(f(row), o, 0, None)}
    shapes = {"gemm": (40, 56), "bmm": (1, 40, 56), "addmm": (40, 56), "conv2d": (2, 16, 5, 5), "sdpa": (1, 2, 70, 64), "softmax": (40, 72), "rms_norm": (40, 72), "add": (56,), "silu": (56,)}
    parameter = lambda v: torch.nn.Parameter(v, requires_grad=False)
    for name, call in taken.items():
        for f in (lambda v: v, parameter):
            out = e(*shapes[name])
            assert call(f, out) == 0
            torch.cuda.synchronize()
            assert torch.isfinite(out).all(), name
        for f in (lambda v: v.as_subclass(Tagged), lambda v: v.cpu(), lambda v: v.double(), lambda v: None, lambda v: [1.0]):
            out = e(*shapes[name])
            assert call(f, out) is None
            torch.cuda.synchronize()
            assert torch.isnan(out).all(), name
        with Mode():
            assert call(lambda v: v, e(*shapes[name])) is None
    stream = torch.cuda.current_stream()
    out = e(40, 56)
    assert module.gemm(a, b, out, None, stream) is None and module.gemm(a, b, out, (64, 64), None) is None and module.gemm(a, b, out, (64.0, 64, 32), None) is None
    assert module.rms_norm(a, e(40, 72), 0, None) is None                    # (an int where a float is due)
    assert module.addmm(row, a, b, out, 1, 2.0, 0, None, None) is None and module.addmm(None, a, b, out, 1.0, 0.0, 2, None, None) is None
    assert module.addmm(row, a, b, out, 1.0, 2.0, None, None, None) is None
    assert module.gemm(a, b, e(40, 55), None, None) != 0                     # (taken: the library's own error)
    torch.cuda.synchronize()
    assert torch.isnan(out).all()


class Mode(torch.overrides.TorchFunctionMode):
    def __torch_function__(self, func, types, args=(), kwargs=None):
        return func(*args, **(kwargs or {}))


def test_the_binding_takes_over_what_the_module_declines():
    run = calls()
    with Mode():
        under_a_mode = {name: f(lambda v: v) for name, f in run.items()}
    a, b = t(40, 72), t(72, 56, seed=1)
    got, want = torch.full((40, 56), float("nan"), dtype=torch.float16, device="cuda"), torch.full((40, 56), float("nan"), dtype=torch.float16, device="cuda")
    nt.addmm(None, a, b, got, alpha=2.0, beta=0.0, act="silu")
    nt.addmm(want.zero_(), a, b, want, alpha=2.0, beta=0, act="silu")
    torch.cuda.synchronize()
    assert torch.equal(got, want)
    for name, f in run.items():
        assert torch.equal(under_a_mode[name], f(lambda v: v)), name


def test_calls_go_to_the_current_stream():
    """Captured on a side stream: a launch on any other would not be in the graph, and its results there before the replay."""
    run = calls()
    want = {name: f(lambda v: v) for name, f in run.items()}
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        got = {name: f(lambda v: v) for name, f in run.items()}
    for _ in range(3):
        for out in got.values():
            out.fill_(float("nan"))
        torch.cuda.synchronize()
        assert all(torch.isnan(out).all() for out in got.values())
        graph.replay()
        torch.cuda.synchronize()
        for name, out in got.items():
            assert torch.equal(out, want[name]), name
