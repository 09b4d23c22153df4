"""halo_gather with the caller's tensors: copies made by the exchange's kernels
(hx_batch_exchange, hx_batch_adjoint) leave every buffer as the copies before
and after would: the bound ones, the arenas, the output and the gradients, bit
for bit against the oracle, for tensors that lie like the bound buffers and for
ones that do not."""
import numpy as np
import pytest

import paper_2309_07337_amd as P
from oracle import move as OM
from oracle import plan as OP
from tests.gpu_util import bits_equal, dev, gpu_plan, host, need_gpu, say
from workloads import random_small_csr, uniform_pm1

pytestmark = pytest.mark.gpu


def like(values, how, dt):
    """The values as a tensor: laid out plainly, off the 16-byte grid, with
    other strides, or in another type."""
    import torch
    t = dev(values)
    if how == "shift":
        u = torch.empty(t.numel() + 1, dtype=dt, device="cuda")[1:].view(t.shape)
    elif how == "strides":
        u = torch.empty((t.shape[1], t.shape[0]), dtype=dt, device="cuda").t()
    elif how == "type":
        u = torch.empty(t.shape, dtype=torch.float64 if dt == torch.float32 else torch.float32, device="cuda")
    else:
        return t
    return u.copy_(t)


@pytest.mark.parametrize("dtype_name,ncols,sched", [
    ("f32", 64, None), ("f64", 16, None), ("f32", 100, None), ("f32", 25, None), ("f64", 5, None), ("f32", 1, None),
    ("f64", 1, None), ("f32", 4, dict(push_pack=1, tile_rows=37)), ("f64", 9, dict(push_pack=1, tile_rows=2000)),
    ("f32", 64, dict(push_pack=2, tile_rows=33)), ("f32", 1027, dict(push_pack=1)), ("f64", 2050, None),
    ("f64", 1, dict(lds_window=1, pair_rows=2, tile_rows=60))])
@pytest.mark.parametrize("variant,staged", [("plain", False), ("locality", False), ("locality", True)])
def test_halo_gather_buffers(variant, staged, dtype_name, ncols, sched):
    need_gpu()
    import torch
    from paper_2309_07337_amd.autograd import HaloExchange, halo_gather
    dt = torch.float64 if dtype_name == "f64" else torch.float32
    npdt = np.float64 if dtype_name == "f64" else np.float32
    rs, rp, cols = random_small_csr(310, 7, 9, 0.5, 55, True)
    halos = OP.all_halos(rp, cols, rs)
    D = OP.Decomposition(halos, rs, 3)
    n, H = 310, sum(h.size for h in halos)
    ex = HaloExchange(gpu_plan(rs, rp, cols, 3, variant), n, H, ncols, dtype=dt, sched=sched, staged_backward=staged)
    hows = ["plain", "shift", "strides"] + (["type"] if dtype_name == "f64" else [])
    for k, how in enumerate(hows):
        say("beside", variant, staged, dtype_name, ncols, sched, how)
        xh = uniform_pm1(60 + k, n * ncols).reshape(n, ncols).astype(np.float32).astype(npdt)
        gh = uniform_pm1(70 + k, H * ncols).reshape(H, ncols).astype(np.float32).astype(npdt)
        want = xh[np.concatenate(halos)]
        gy = np.split(gh, np.cumsum([h.size for h in halos])[:-1])
        if staged:
            want_g = OM.staged_adjoint_reference([D.plan(r, variant) for r in range(7)], gy, rs)["g_x"]
        else:
            want_g = OM.exchange_adjoint_reference(halos, gy, n)
        for t in (ex.x, ex.halo, ex.g_halo, ex.g_x):
            t.fill_(float("nan"))
        x = like(xh, how, dt).requires_grad_(True)
        y = halo_gather(x, ex)
        assert y.data_ptr() != ex.halo.data_ptr()
        g = like(gh, how, dt)
        gx, = torch.autograd.grad(y, x, g.to(y.dtype) if how == "type" else g)
        assert bits_equal(host(y), want) and bits_equal(host(ex.halo), want)
        assert bits_equal(host(ex.x), xh) and bits_equal(host(ex.g_halo), gh)
        # (autograd returns the gradient in the input's type)
        assert bits_equal(host(gx), want_g.astype(host(gx).dtype)) and bits_equal(host(ex.g_x), want_g)
        send = host(P.batch_arena_view(ex.batch, P.HX_ARENA_SEND, ncols, dt))
        recv = host(P.batch_arena_view(ex.batch, P.HX_ARENA_RECV, ncols, dt))
        assert np.isfinite(send).all() and np.isfinite(recv).all()
        if variant == "plain":
            assert bits_equal(recv, want)
            back = host(P.batch_arena_view(ex.batch, P.HX_ARENA_GRAD_SEND, ncols, dt))
            assert np.array_equal(np.sort(back[:, 0]), np.sort(gh[:, 0]))
    # without a copy out, and a gradient that is one value for all
    x = dev(xh).requires_grad_(True)
    y = halo_gather(x, ex, copy_out=False)
    assert y.data_ptr() == ex.halo.data_ptr() and bits_equal(host(y), want) and bits_equal(host(ex.x), xh)
    y.sum().backward()
    assert (host(ex.g_halo) == 1).all() and bits_equal(host(x.grad), host(ex.g_x))


def test_exchange_refuses():
    need_gpu()
    import torch
    from paper_2309_07337_amd.autograd import HaloExchange
    rs, rp, cols = random_small_csr(310, 7, 9, 0.5, 55, True)
    H = sum(h.size for h in OP.all_halos(rp, cols, rs))
    ex = HaloExchange(gpu_plan(rs, rp, cols, 3, "plain"), 310, H, 16, dtype=torch.float32)
    off = torch.zeros(310 * 16 + 1, device="cuda")[1:].view(310, 16)
    for call in (lambda: P.hx_batch_exchange(ex.batch, off), lambda: P.hx_batch_adjoint(ex.batch, None, off)):
        with pytest.raises(P.HXError) as e:
            call()
        assert e.value.code == P.HX_ERR_ARG
    P.hx_batch_start(ex.batch)
    with pytest.raises(P.HXError) as e:
        P.hx_batch_exchange(ex.batch)
    assert e.value.code == P.HX_ERR_STATE
    P.hx_batch_wait(ex.batch)
    torch.cuda.synchronize()
