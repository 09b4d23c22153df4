"""Calls that fail for want of memory leave requests and batches as they were:
every allocation of a rebinding, a new schedule or a first launch refused in
turn, then the steps run on the former state, bit for bit against the oracle."""
import numpy as np
import pytest

import paper_2309_07337_amd as P
from paper_2309_07337_amd import _lib as L
from oracle import move as OM
from oracle import plan as OP
from tests.gpu_util import bits_equal, dev, gpu_plan, host, need_gpu, say
from tests.test_gpu_alloc import _Counting
from workloads import random_small_csr, splitmix64, uniform_pm1

pytestmark = pytest.mark.gpu
N, R, NCOLS = 400, 9, 3


def refused(call, after):
    """Refuses the k-th allocation of call for k = 0, 1, ... until it succeeds;
    after(False) follows every failure, after(True) the success."""
    k = 0
    while True:
        a = _Counting(k)
        P.hx_set_allocator(a.alloc, a.free)
        try:
            call()
            done = True
        except P.HXError as e:
            assert e.code == P.HX_ERR_NOMEM, k
            done = False
        finally:
            L.use_torch_allocator()
        after(done)
        if done:
            _keep.append(a)     # (what it handed out goes back through it)
            return k
        assert not a.live, (k, a.live)
        k += 1


_keep = []


def values(seed, rows):
    return uniform_pm1(seed, rows * NCOLS).reshape(rows, NCOLS)


@pytest.mark.parametrize("variant,staged", [("plain", False), ("locality", False), ("locality", True)])
def test_world(variant, staged):
    need_gpu()
    import torch
    say("rollback, world", variant, staged)
    rs, rp, cols = random_small_csr(N, R, 9, 0.5, 55, True)
    halos = OP.all_halos(rp, cols, rs)
    H = sum(h.size for h in halos)
    D = OP.Decomposition(halos, rs, 3)
    xh, gh = values(1, N), [values(2, H), values(3, H)]
    x, halo = dev(xh), torch.empty((H, NCOLS), dtype=torch.float64, device="cuda")
    g, gx = [dev(v) for v in gh], [torch.empty((N, NCOLS), dtype=torch.float64, device="cuda") for _ in gh]
    gy = [np.split(v, np.cumsum([h.size for h in halos])[:-1]) for v in gh]
    if staged:
        want = [OM.staged_adjoint_reference([D.plan(r, variant) for r in range(R)], v, rs)["g_x"] for v in gy]
    else:
        want = [OM.exchange_adjoint_reference(halos, v, N) for v in gy]
    b = P.hx_batch_from_plan(gpu_plan(rs, rp, cols, 3, variant), x, halo,
                             flags=P.HX_WORLD_SIM_TRANSFER | (P.HX_WORLD_STAGED_BACKWARD if staged else 0))

    def check(bound):
        halo.fill_(float("nan"))
        P.hx_batch_start(b)
        P.hx_batch_wait(b)
        assert bits_equal(host(halo), xh[np.concatenate(halos)])
        if bound is None:
            with pytest.raises(P.HXError) as e:
                P.hx_batch_backward(b)
            assert e.value.code == P.HX_ERR_STATE
            return
        for t in gx:
            t.fill_(float("nan"))
        P.hx_batch_backward(b)
        assert bits_equal(host(gx[bound]), want[bound]) and torch.isnan(gx[1 - bound]).all()
        gx[bound].fill_(float("nan"))
        P.hx_batch_backward_plain(b)
        assert bits_equal(host(gx[bound]), want[bound]) and torch.isnan(gx[1 - bound]).all()

    assert refused(lambda: P.hx_batch_bind_grad(b, g[0], gx[0]), lambda done: check(0 if done else None)) > 2
    assert refused(lambda: P.hx_batch_bind_grad(b, g[1], gx[1]), lambda done: check(1 if done else 0)) > 2
    for ph, sched in ((0, dict(tile_rows=33, push_pack=1)), (0, dict(tile_rows=17, push_pack=2)),
                      (3, dict(tile_rows=40))):
        old = P.hx_batch_get_sched(b, ph)

        def after(done):
            check(1)
            assert (P.hx_batch_get_sched(b, ph) != old) == done

        assert refused(lambda: P.hx_batch_set_sched(b, ph, sched), after) > 2
    b.free()


def test_requests():
    need_gpu()
    import torch
    say("rollback, requests")
    E = N + 50
    idx = (splitmix64(5, 0, E) % np.uint64(N)).astype(np.int32)
    xh, rh, gh = values(1, N), values(2, E), [values(3, E), values(4, E), values(5, E)]
    x, halo = dev(xh), torch.empty((E, NCOLS), dtype=torch.float64, device="cuda")
    g = [dev(v) for v in gh]
    gx = [torch.empty((N, NCOLS), dtype=torch.float64, device="cuda") for _ in gh]
    topo = P.hx_topo_create(0, 8, [1, 2], [1, 2])
    req = P.hx_neighbor_alltoallv_init(x, [E // 3, E - E // 3], None, idx, halo, [E // 3, E - E // 3], None, topo)
    P.req_arena_view(req, P.HX_ARENA_RECV, NCOLS, torch.float64).copy_(dev(rh))
    send = P.req_arena_view(req, P.HX_ARENA_SEND, NCOLS, torch.float64)
    want = [OM.pack_transpose(v, *OP.transpose_csr(idx, N)) for v in gh]

    def check(bound, start=P.hx_start, wait=P.hx_wait, backward=P.hx_backward, h=None):
        h = h or req
        for t in [halo, send] + gx:
            t.fill_(float("nan"))
        start(h)
        wait(h)
        assert bits_equal(host(halo), rh) and bits_equal(host(send), OM.pack(xh, idx))
        if bound is None:
            with pytest.raises(P.HXError) as e:
                backward(h)
            assert e.value.code == P.HX_ERR_STATE
            return
        backward(h)
        assert bits_equal(host(gx[bound]), want[bound])
        assert all(torch.isnan(t).all() for k, t in enumerate(gx) if k != bound)

    # the first launch builds the tables
    started = []

    def first():
        P.hx_start(req)
        started.append(True)

    refused(first, lambda done: None)
    assert started == [True]
    P.hx_wait(req)
    check(None)
    refused(lambda: P.hx_req_bind_grad(req, g[0], gx[0]), lambda done: check(0 if done else None))
    refused(lambda: P.hx_req_bind_grad(req, g[1], gx[1]), lambda done: check(1 if done else 0))
    b = P.hx_batch_init([req])
    batch = dict(start=P.hx_batch_start, wait=P.hx_batch_wait, backward=P.hx_batch_backward, h=b)
    check(1, **batch)
    # a member's new gradients reach the batch when its backward can be rebuilt
    P.hx_req_bind_grad(req, g[2], gx[2])

    def rebuilt(done):
        for t in [halo] + ([] if done else gx):
            t.fill_(float("nan"))
        P.hx_batch_start(b)
        P.hx_batch_wait(b)
        assert bits_equal(host(halo), rh)
        assert done or all(torch.isnan(t).all() for t in gx)

    assert refused(lambda: P.hx_batch_backward(b), rebuilt) > 2
    assert bits_equal(host(gx[2]), want[2])
    check(2, **batch)
    b.free()
