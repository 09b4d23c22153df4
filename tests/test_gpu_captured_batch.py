"""A batch's steps in a graph of the caller's: captured after one eager step and
replayed with new inputs, with eager steps and other work between the replays;
every replay against the oracle, bit for bit."""
import numpy as np
import pytest

import paper_2309_07337_amd as P
from oracle import move as OM
from oracle import plan as OP
from tests.gpu_util import bits_equal, dev, gpu_plan, host, need_gpu, say
from tests.test_gpu_batch import build_members, check_members, reset
from workloads import random_small_csr, uniform_pm1

pytestmark = pytest.mark.gpu
N, R = 700, 9


def capture(step):
    import torch
    step()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    return graph


@pytest.mark.parametrize("dtype_name,ncols", [("f64", 16), ("f32", 1), ("f64", 3)])
def test_members(dtype_name, ncols):
    need_gpu()
    import torch
    say("captured members", dtype_name, ncols)
    dt = torch.float64 if dtype_name == "f64" else torch.float32
    mem = build_members(10, 9000, ncols, dt)
    b = P.hx_batch_init([m["req"] for m in mem])

    def step():
        P.hx_batch_start(b)
        P.hx_batch_wait(b)
        P.hx_batch_backward(b)

    graph = capture(step)
    for it in range(3):
        for k, m in enumerate(mem):
            for name, seed in (("x", 1), ("recv", 2), ("g_send", 3)):
                m[name].copy_(dev(uniform_pm1(100 * it + 10 * k + seed, m["h"] * ncols).reshape(m["h"], ncols)))
            P.req_arena_view(m["req"], P.HX_ARENA_RECV, ncols, dt).copy_(m["recv"])
        reset(mem)
        torch.cuda.synchronize()
        graph.replay()
        check_members(mem, ncols, dt)
        reset(mem)
        step()
        check_members(mem, ncols, dt)
    del graph
    b.free()


@pytest.mark.parametrize("dtype_name,ncols", [("f32", 64), ("f64", 1), ("f64", 5)])
@pytest.mark.parametrize("variant,staged", [("plain", False), ("locality", False), ("locality", True),
                                            ("locality3", True)])
def test_world(variant, staged, dtype_name, ncols):
    """Start, Wait and the backward on the bound buffers, then hx_batch_exchange
    and hx_batch_adjoint beside the caller's, in one graph."""
    need_gpu()
    import torch
    from paper_2309_07337_amd.autograd import HaloExchange
    say("captured world", variant, staged, dtype_name, ncols)
    dt, npdt = (torch.float64, np.float64) if dtype_name == "f64" else (torch.float32, np.float32)
    rs, rp, cols = random_small_csr(N, R, 9, 0.5, 55, True)
    halos = OP.all_halos(rp, cols, rs)
    D = OP.Decomposition(halos, rs, 3)
    H = sum(h.size for h in halos)
    ex = HaloExchange(gpu_plan(rs, rp, cols, 3, variant), N, H, ncols, dtype=dt, staged_backward=staged)
    x, g = (torch.zeros((r, ncols), dtype=dt, device="cuda") for r in (N, H))
    y, gx = torch.empty_like(g), torch.empty_like(x)
    first = [torch.empty_like(g), torch.empty_like(x)]      # what the first half left

    def step():
        P.hx_batch_start(ex.batch)
        P.hx_batch_wait(ex.batch)
        P.hx_batch_backward(ex.batch)
        first[0].copy_(ex.halo)
        first[1].copy_(ex.g_x)
        P.hx_batch_exchange(ex.batch, x, y)
        P.hx_batch_adjoint(ex.batch, g, gx)

    def adjoint(gh):
        gy = np.split(gh, np.cumsum([h.size for h in halos])[:-1])
        if staged:
            return OM.staged_adjoint_reference([D.plan(r, variant) for r in range(R)], gy, rs)["g_x"]
        return OM.exchange_adjoint_reference(halos, gy, N)

    graph = capture(step)
    for it in range(6):
        values = [uniform_pm1(9000 + 10 * it + k, r * ncols).reshape(r, ncols).astype(npdt)
                  for k, r in enumerate((N, H, N, H))]
        for t, v in zip((ex.x, ex.g_halo, x, g), values):
            t.copy_(dev(v))
        for t in (ex.halo, ex.g_x, y, gx, *first):
            t.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay() if it % 2 == 0 else step()
        want, want2 = (v[np.concatenate(halos)] for v in (values[0], values[2]))
        assert bits_equal(host(first[0]), want) and bits_equal(host(first[1]), adjoint(values[1])), it
        assert bits_equal(host(y), want2) and bits_equal(host(ex.halo), want2), it
        assert bits_equal(host(gx), adjoint(values[3])) and bits_equal(host(ex.g_x), host(gx)), it
        assert bits_equal(host(ex.x), values[2]) and bits_equal(host(ex.g_halo), values[3]), it
