"""The caller's buffers of hx_batch_exchange and hx_batch_adjoint: what is not
laid out as the bound buffer is refused, what overlaps it too, and buffers that
lie in the batch's own arenas give what copies before and after would."""
import numpy as np
import pytest

import paper_2309_07337_amd as P
from oracle import move as OM
from oracle import plan as OP
from tests.gpu_util import bits_equal, dev, gpu_plan, host, need_gpu, say
from workloads import random_small_csr, uniform_pm1

pytestmark = pytest.mark.gpu
N = 310


def exchange(ncols, variant="plain", staged=False):
    from paper_2309_07337_amd.autograd import HaloExchange
    rs, rp, cols = random_small_csr(N, 7, 9, 0.5, 55, True)
    halos = OP.all_halos(rp, cols, rs)
    H = sum(h.size for h in halos)
    return HaloExchange(gpu_plan(rs, rp, cols, 3, variant), N, H, ncols, staged_backward=staged), halos, H


def test_refuses_other_layouts():
    need_gpu()
    import torch
    ex, halos, H = exchange(16)
    kw = dict(device="cuda")
    wrong = lambda rows: (torch.zeros(rows, 16, dtype=torch.float64, **kw), torch.zeros(rows, 15, **kw),
                          torch.zeros(rows - 1, 16, **kw), torch.zeros(16, rows, **kw).t(),
                          torch.zeros(rows, 32, **kw)[:, ::2], torch.zeros(rows, 16))
    calls = [lambda t: P.hx_batch_exchange(ex.batch, t), lambda t: P.hx_batch_exchange(ex.batch, None, t),
             lambda t: P.hx_batch_adjoint(ex.batch, t), lambda t: P.hx_batch_adjoint(ex.batch, None, t)]
    for call, rows in zip(calls, (N, H, H, N)):
        for t in wrong(rows):
            with pytest.raises(P.HXError) as e:
                call(t)
            assert e.value.code == P.HX_ERR_ARG
    big = torch.zeros(2 * N, 16, **kw)
    b = P.hx_batch_from_plan(ex.batch._keep[0], big[:N], ex.halo, flags=P.HX_WORLD_SIM_TRANSFER)
    with pytest.raises(P.HXError) as e:     # rows 8.. of the bound vector
        P.hx_batch_exchange(b, big[8:N + 8])
    assert e.value.code == P.HX_ERR_ARG
    P.hx_batch_exchange(b, big[N:])


@pytest.mark.parametrize("ncols", [1, 5, 64])
@pytest.mark.parametrize("variant,staged", [("plain", False), ("locality", False), ("locality", True)])
def test_buffers_in_the_arenas(variant, staged, ncols):
    """Every buffer of the caller's in the send, receive and gradient arenas, where
    they hold it."""
    need_gpu()
    import torch
    say("arenas", variant, staged, ncols)
    ex, halos, H = exchange(ncols, variant, staged)
    views = [P.batch_arena_view(ex.batch, w, ncols, torch.float32)
             for w in (P.HX_ARENA_SEND, P.HX_ARENA_RECV)]
    if variant == "plain" or staged:
        views.append(P.batch_arena_view(ex.batch, P.HX_ARENA_GRAD_SEND, ncols, torch.float32))
    xh = uniform_pm1(1, N * ncols).reshape(N, ncols).astype(np.float32)
    gh = uniform_pm1(2, H * ncols).reshape(H, ncols).astype(np.float32)
    gy = np.split(gh, np.cumsum([h.size for h in halos])[:-1])
    if staged:
        rs, rp, cols = random_small_csr(N, 7, 9, 0.5, 55, True)
        D = OP.Decomposition(halos, rs, 3)
        want_g = OM.staged_adjoint_reference([D.plan(r, variant) for r in range(7)], gy, rs)["g_x"]
    else:
        want_g = OM.exchange_adjoint_reference(halos, gy, N)
    done = 0
    for v in views + [ex.g_halo]:
        for first in (0, 8):
            def part(rows):
                ok = v.shape[0] >= first + rows and (first * ncols) % 4 == 0
                return v[first:first + rows] if ok else None
            x, y, g, gx = part(N), part(H), part(H), part(N)
            if x is not None:
                x.copy_(dev(xh))
                P.hx_batch_exchange(ex.batch, x)
                assert bits_equal(host(ex.halo), xh[np.concatenate(halos)]) and bits_equal(host(ex.x), xh)
                done += 1
            ex.x.copy_(dev(xh))
            if y is not None:
                P.hx_batch_exchange(ex.batch, None, y)
                assert bits_equal(host(y), host(ex.halo)) and bits_equal(host(y), xh[np.concatenate(halos)])
                done += 1
            if g is not None and v is not ex.g_halo:
                g.copy_(dev(gh))
                P.hx_batch_adjoint(ex.batch, g)
                assert bits_equal(host(ex.g_x), want_g) and bits_equal(host(ex.g_halo), gh)
                done += 1
            ex.g_halo.copy_(dev(gh))
            if gx is not None:
                P.hx_batch_adjoint(ex.batch, None, gx)
                assert bits_equal(host(gx), want_g) and bits_equal(host(ex.g_x), want_g)
                done += 1
    assert done >= 8
