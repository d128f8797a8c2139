"""What autograd, threads and callers ask of the native calls (csrc/native.cpp)."""
import pytest
import torch
import torch.autograd.forward_ad as fwd

from paper_2309_15275_amd import binding
from paper_2309_15275_amd.autograd import lbp_wht_linear

pytestmark = pytest.mark.gpu
IDX = [0, 1, 8, 9, 2, 16, 10, 17]


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    yield
    torch.cuda.synchronize()


def _tensors(seed=0, dtype=torch.float32, cin=32, cout=48, shape=(2, 16, 16)):
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn(shape + (cin,), generator=g, device="cuda").to(dtype)
    w = (0.1 * torch.randn(cout, cin, generator=g, device="cuda")).to(dtype)
    b = torch.randn(cout, generator=g, device="cuda").to(dtype)
    gy = torch.randn(shape + (cout,), generator=g, device="cuda").to(dtype)
    return x, w, b, gy


@pytest.mark.parametrize("which", [0, 1, 2])
def test_forward_mode_is_refused(which):
    args = list(_tensors()[:3])
    with fwd.dual_level():
        args[which] = fwd.make_dual(args[which], torch.ones_like(args[which]))
        with pytest.raises(NotImplementedError):
            lbp_wht_linear(*args, 8, IDX)


def test_function_transforms_are_refused():
    x, w, b, _ = _tensors()
    ws = torch.stack([w, 2 * w])
    with pytest.raises(RuntimeError):
        torch.func.vmap(lambda v: lbp_wht_linear(x, v, b, 8, IDX))(ws)
    with pytest.raises(RuntimeError):
        torch.func.vmap(lambda v: lbp_wht_linear(x, w, v, 8, IDX))(torch.stack([b, b]))
    with pytest.raises(RuntimeError):
        torch.func.grad(lambda v: lbp_wht_linear(x, v, b, 8, IDX).sum())(w)
    with pytest.raises(RuntimeError):
        torch.func.jvp(lambda v: lbp_wht_linear(x, v, b, 8, IDX), (w,), (w,))


def test_traces_and_modes_see_the_function():
    x, w, b, _ = _tensors()
    traced = torch.jit.trace(lambda v: lbp_wht_linear(v, w, b, 8, IDX), x, check_trace=False)
    assert "_LbpWhtLinearFn" in str(traced.graph)
    seen = []

    class Mode(torch.overrides.TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            seen.append(getattr(func, "__name__", ""))
            return func(*args, **(kwargs or {}))

    with Mode():
        lbp_wht_linear(x, w, b, 8, IDX)
    assert "linear" in seen
    assert "LbpWhtLinearBackward" in lbp_wht_linear(x, w.requires_grad_(), b, 8, IDX).grad_fn.name()      # and without one: native


def test_bias_gradient_is_differentiable():
    x, w, b, gy = _tensors()
    for t in (x, w, b, gy):
        t.requires_grad_()
    _, _, gb = torch.autograd.grad(lbp_wht_linear(x, w, b, 8, IDX), (x, w, b), gy, create_graph=True)
    torch.testing.assert_close(gb, gy.sum((0, 1, 2)))
    gg, = torch.autograd.grad((gb * gb.detach()).sum(), gy)
    torch.testing.assert_close(gg, gb.detach().expand_as(gy))
    seq = x.detach().reshape(2, 256, 32)
    gb, = torch.autograd.grad(lbp_wht_linear(seq, w, b, 8, IDX, (16, 16)), b, gy.reshape(2, 256, 48), create_graph=True)
    gg, = torch.autograd.grad(gb.sum(), gy)
    torch.testing.assert_close(gg, torch.ones_like(gy))


def test_bias_gradient_keeps_the_tangent_of_the_output_gradient():
    x, w, b, gy = _tensors()
    b.requires_grad_()
    with fwd.dual_level():
        y = lbp_wht_linear(x, w, b, 8, IDX)
        gb, = torch.autograd.grad(y, b, fwd.make_dual(gy, 2 * gy))
        tangent = fwd.unpack_dual(gb).tangent
    torch.testing.assert_close(tangent, 2 * gy.sum((0, 1, 2)))
