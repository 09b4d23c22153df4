"""Packs of few of a large source's rows (a rank's surface) and of more, on both
sides of the default's lines, bit for bit against the oracle."""
import numpy as np
import pytest

import paper_2309_07337_amd as P
from oracle import move as OM
from tests.gpu_util import bits_equal, dev, host, need_gpu, say
from workloads import splitmix64, uniform_pm1

pytestmark = pytest.mark.gpu


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
    idx = np.sort(splitmix64(7, 0, E) % np.uint64(n)).astype(np.int32)
    counts = [E // 3, E - E // 3]
    xh = uniform_pm1(8, n * ncols).reshape(n, ncols).astype(npdt)
    x, halo = dev(xh), torch.zeros((E, ncols), dtype=dt, device="cuda")
    topo = P.hx_topo_create(0, 8, [1, 2], [1, 2])
    req = P.hx_neighbor_alltoallv_init(x, counts, None, idx, halo, counts, None, topo)
    send = P.req_arena_view(req, P.HX_ARENA_SEND, ncols, dt)
    want = OM.pack(xh, idx)
    b = P.hx_batch_init([req])
    push = P.hx_batch_get_sched(b, 0)["push_pack"] == 1
    assert push == (xh.itemsize * ncols >= 64 or 2 * E >= n)
    for start, wait, h in ((P.hx_start, P.hx_wait, req), (P.hx_batch_start, P.hx_batch_wait, b)):
        send.fill_(float("nan"))
        start(h)
        assert bits_equal(host(send), want)
        wait(h)
    b.free()


@pytest.mark.parametrize("order", ["ascending", "none"])
def test_large_lists(order):
    """12 M packed rows of 24 bytes, beyond the Infinity Cache, in ascending order
    and in none."""
    need_gpu()
    import torch
    n = 12_000_000
    say("large lists", order)
    idx = (splitmix64(7, 0, n) % np.uint64(n)).astype(np.int32)
    if order == "ascending":
        idx.sort()
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
