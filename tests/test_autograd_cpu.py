"""halo_gather's bookkeeping around the library's kernels, on the CPU: the two
calls it makes (exchange_at, adjoint_at) are played by torch ops on
host tensors, one global gather and its transpose."""
import ctypes

import pytest
import torch

from paper_2309_07337_amd import _lib as L
from paper_2309_07337_amd import autograd as A

COLS = torch.tensor([3, 0, 5, 3])


@pytest.fixture
def ex(monkeypatch):
    ex = A.HaloExchange.__new__(A.HaloExchange)
    ex.x, ex.g_x = torch.zeros(6, 4), torch.zeros(6, 4)
    ex.halo, ex.g_halo = torch.zeros(4, 4), torch.zeros(4, 4)
    ex.generation, ex.batch = 0, object()

    def move(src, bound, out, result, step):    # by address, as a kernel writes
        if src is not None:
            ctypes.memmove(bound.data_ptr(), src, bound.nbytes)
        step()
        if out is not None:
            ctypes.memmove(out, result.data_ptr(), result.nbytes)

    def gather():
        ex.halo.data.copy_(ex.x.detach()[COLS])

    def scatter():
        ex.g_x.data.zero_().index_add_(0, COLS, ex.g_halo.detach())

    monkeypatch.setattr(L, "exchange_at", lambda b, x, halo, stream=None: move(x, ex.x, halo, ex.halo, gather))
    monkeypatch.setattr(L, "adjoint_at", lambda b, g, gx, stream=None: move(g, ex.g_halo, gx, ex.g_x, scatter))
    return ex


@pytest.mark.parametrize("how", ["plain", "strides", "type"])
def test_overwritten_input_is_reported(ex, how):
    """An op that saved ex.x, then a halo_gather that copies into it: the op's
    backward raises, whoever made the copy."""
    w = torch.ones(4, 2, requires_grad=True)
    own = ex.x @ w
    h = torch.rand(6, 4)
    if how == "strides":
        h = torch.rand(4, 6).t()
    elif how == "type":
        h = h.double()
    A.halo_gather(h.requires_grad_(True), ex)
    with pytest.raises(RuntimeError, match="modified by an inplace operation"):
        own.sum().backward()


def test_overwritten_gradient_is_reported(ex):
    w = torch.ones(4, 2, requires_grad=True)
    own = ex.g_halo @ w
    y = A.halo_gather(torch.rand(6, 4, requires_grad=True), ex)
    y.backward(torch.rand(4, 4))
    with pytest.raises(RuntimeError, match="modified by an inplace operation"):
        own.sum().backward()


def test_bound_tensors_are_not_copied(ex):
    """The zero-copy path changes nothing, and reports nothing."""
    ex.x.copy_(torch.rand(6, 4))
    w = torch.ones(4, 2, requires_grad=True)
    own = ex.x @ w
    y = A.halo_gather(ex.x, ex, copy_out=False)
    assert y.data_ptr() == ex.halo.data_ptr() and torch.equal(y, ex.x[COLS])
    own.sum().backward()
    assert torch.equal(w.grad, ex.x.sum(0)[:, None].expand(4, 2))


def test_inference_buffers_stay_refused(ex):
    """Buffers made in inference mode are not written outside it."""
    with torch.inference_mode():
        ex.x = torch.zeros(6, 4)
    with pytest.raises(RuntimeError, match="inference tensor"):
        A.halo_gather(torch.rand(6, 4), ex)


@pytest.mark.parametrize("how", ["class", "object"])
@pytest.mark.parametrize("copy_out", [True, False])
def test_own_steps_are_called(ex, how, copy_out):
    """forward() and backward() of a subclass or of the object itself (a caller's
    own transport) run instead of the library's fused calls."""
    class Transport(A.HaloExchange):
        def forward(self, stream=None):
            self.halo.copy_(2 * self.x[COLS])
            self.generation += 1
            return self.halo

        def backward(self, stream=None):
            self.g_x.zero_().index_add_(0, COLS, 2 * self.g_halo)
            return self.g_x

    if how == "class":
        ex.__class__ = Transport
    else:
        ex.forward, ex.backward = Transport.forward.__get__(ex), Transport.backward.__get__(ex)
    x, g = torch.rand(6, 4, requires_grad=True), torch.rand(4, 4)
    y = A.halo_gather(x, ex, copy_out)
    assert torch.equal(y, 2 * x[COLS]) and ex.generation == 1
    assert (y.data_ptr() == ex.halo.data_ptr()) == (not copy_out)
    y.backward(g)
    assert torch.equal(x.grad, torch.zeros(6, 4).index_add_(0, COLS, 2 * g))
