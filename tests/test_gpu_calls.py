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
