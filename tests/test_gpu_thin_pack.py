"""Packs of few of a large source's rows (a rank's surface) and of more, on both
sides of the default's lines, bit for bit against the oracle."""
import numpy as np
import pytest

import paper_2309_07337_amd as P
from oracle import move as OM
from tests.gpu_util import bits_equal, dev, host, need_gpu, say
from workloads import splitmix64, uniform_pm1

pytestmark = pytest.mark.gpu


def in_messages(idx, k=8):
    """The list as k messages of ascending rows."""
    return np.concatenate([np.sort(part) for part in np.array_split(idx, k)])


@pytest.mark.parametrize("dtype_name,ncols", [("f64", 1), ("f32", 2), ("f64", 3), ("f64", 8), ("f64", 32)])
@pytest.mark.parametrize("share", [700, 33, 5, 4, 3, 2, 1])
def test_default_pack(dtype_name, ncols, share):
    """One in `share` of the rows packed, for a request and a batch."""
    need_gpu()
    import torch
    dt, npdt = (torch.float64, np.float64) if dtype_name == "f64" else (torch.float32, np.float32)
    n = 700_000 if ncols < 8 else 90_001
    E = n // share
    say("thin pack", dtype_name, ncols, n, E)
    idx = in_messages((splitmix64(7, 0, E) % np.uint64(n)).astype(np.int32))
    counts = [E // 3, E - E // 3]
    xh = uniform_pm1(8, n * ncols).reshape(n, ncols).astype(npdt)
    x, halo = dev(xh), torch.zeros((E, ncols), dtype=dt, device="cuda")
    topo = P.hx_topo_create(0, 8, [1, 2], [1, 2])
    req = P.hx_neighbor_alltoallv_init(x, counts, None, idx, halo, counts, None, topo)
    send = P.req_arena_view(req, P.HX_ARENA_SEND, ncols, dt)
    want = OM.pack(xh, idx)
    b = P.hx_batch_init([req])
    push = P.hx_batch_get_sched(b, 0)["push_pack"] == 1
    assert push == (2 * E >= n)
    for start, wait, h in ((P.hx_start, P.hx_wait, req), (P.hx_batch_start, P.hx_batch_wait, b)):
        send.fill_(float("nan"))
        start(h)
        assert bits_equal(host(send), want)
        wait(h)
    b.free()


@pytest.mark.parametrize("order", ["ascending", "none"])
def test_large_lists(order):
    """12 M packed rows of 24 bytes, beyond the Infinity Cache, in messages of
    ascending rows and in no order."""
    need_gpu()
    import torch
    n = 12_000_000
    say("large lists", order)
    idx = (splitmix64(7, 0, n) % np.uint64(n)).astype(np.int32)
    if order == "ascending":
        idx = in_messages(idx)
    x = torch.rand((n, 3), dtype=torch.float64, device="cuda")
    halo = torch.zeros((n, 3), dtype=torch.float64, device="cuda")
    req = P.hx_neighbor_alltoallv_init(x, [n], None, idx, halo, [n], None, P.hx_topo_create(0, 2, [1], [1]))
    b = P.hx_batch_init([req])
    assert (P.hx_batch_get_sched(b, 0)["push_pack"] == 1) == (order == "ascending")
    send = P.req_arena_view(req, P.HX_ARENA_SEND, 3, torch.float64)
    want = x[torch.from_numpy(idx).cuda().long()]
    for start, wait, h in ((P.hx_start, P.hx_wait, req), (P.hx_batch_start, P.hx_batch_wait, b)):
        send.fill_(float("nan"))
        start(h)
        assert torch.equal(send, want)
        wait(h)
    b.free()


@pytest.mark.parametrize("dtype_name,ncols", [("f32", 1), ("f32", 2), ("f64", 3), ("f64", 7)])
@pytest.mark.parametrize("runs,times", [(1, 0.7), (4, 1), (5, 1), (8, 2), (9, 2)])
def test_dense_messages(dtype_name, ncols, runs, times):
    """Messages that take every fourth row or more, on both sides of the line."""
    need_gpu()
    import torch
    dt, npdt = (torch.float64, np.float64) if dtype_name == "f64" else (torch.float32, np.float32)
    n = 1_300_003
    E = int(n * times)
    say("dense messages", dtype_name, ncols, runs, times)
    idx = in_messages((splitmix64(9, 0, E) % np.uint64(n)).astype(np.int32), runs)
    xh = uniform_pm1(8, n * ncols).reshape(n, ncols).astype(npdt)
    x, halo = dev(xh), torch.zeros((E, ncols), dtype=dt, device="cuda")
    req = P.hx_neighbor_alltoallv_init(x, [E], None, idx, halo, [E], None, P.hx_topo_create(0, 2, [1], [1]))
    b = P.hx_batch_init([req])
    dense = 4 * E >= runs * n and (xh.itemsize * ncols <= 8 or E <= n)
    assert (P.hx_batch_get_sched(b, 0)["push_pack"] == 1) == (not dense)
    send = P.req_arena_view(req, P.HX_ARENA_SEND, ncols, dt)
    want = OM.pack(xh, idx)
    for start, wait, h in ((P.hx_start, P.hx_wait, req), (P.hx_batch_start, P.hx_batch_wait, b)):
        send.fill_(float("nan"))
        start(h)
        assert bits_equal(host(send), want)
        wait(h)
    b.free()
