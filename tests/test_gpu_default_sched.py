"""Default schedules follow the work (rows, row size, what a job reads): results
stay bit for bit the oracle's on either side of each line, for one request, a
batch and a world, from one row to enough to fill the chip."""
import numpy as np
import pytest

import paper_2309_07337_amd as P
from oracle import move as OM
from oracle import plan as OP
from tests.gpu_util import bits_equal, dev, host, need_gpu, say
from tests.test_gpu_world import check_world_against_oracle
from workloads import random_small_csr, splitmix64, uniform_pm1

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype_name,ncols", [("f64", 1), ("f32", 1), ("f64", 2), ("f32", 3), ("f64", 5), ("f64", 16)])
@pytest.mark.parametrize("n", [1, 63, 700, 20000, 900_000])
def test_request_and_batch(dtype_name, ncols, n):
    """n rows of source: 900,000 are beyond an XCD's L2 at every row size but
    one FP32 value; E slots, some of them repeated."""
    need_gpu()
    import torch
    if n * ncols > 6_000_000:
        n = 6_000_000 // ncols
    say("default schedules", dtype_name, ncols, n)
    dt = torch.float64 if dtype_name == "f64" else torch.float32
    npdt = np.float64 if dtype_name == "f64" else np.float32
    E = n + n // 3
    idx = (splitmix64(5, 0, E) % np.uint64(n)).astype(np.int32)
    counts = [E // 2, E - E // 2] if E > 1 else [1]
    xh, rh, gh = (uniform_pm1(s, r * ncols).reshape(r, ncols).astype(npdt) for s, r in ((1, n), (2, E), (3, E)))
    halo = torch.empty((E, ncols), dtype=dt, device="cuda")
    x, g, gx = dev(xh), dev(gh), torch.empty((n, ncols), dtype=dt, device="cuda")
    topo = P.hx_topo_create(0, 8, [1, 2][:len(counts)], [1, 2][:len(counts)])
    req = P.hx_neighbor_alltoallv_init(x, counts, None, idx, halo, counts, None, topo)
    P.req_arena_view(req, P.HX_ARENA_RECV, ncols, dt).copy_(dev(rh))
    P.hx_req_bind_grad(req, g, gx)
    ptr, perm = OP.transpose_csr(idx, n)
    want_send, want_gx = OM.pack(xh, idx), OM.pack_transpose(gh, ptr, perm)
    send = P.req_arena_view(req, P.HX_ARENA_SEND, ncols, dt)

    def check(step):
        for t in (halo, gx, send):
            t.fill_(float("nan"))
        step()
        assert bits_equal(host(send), want_send)
        assert bits_equal(host(halo), rh)
        assert bits_equal(host(gx), want_gx)

    check(lambda: (P.hx_start(req), P.hx_wait(req), P.hx_backward(req)))
    check(lambda: (P.hx_start(req), P.hx_wait(req), P.hx_backward_noalloc(req, g, gx)))
    b = P.hx_batch_init([req])
    check(lambda: (P.hx_batch_start(b), P.hx_batch_wait(b), P.hx_batch_backward(b)))
    check(lambda: (P.hx_batch_start_plain(b), P.hx_batch_wait_plain(b), P.hx_batch_backward_plain(b)))
    b.free()


@pytest.mark.parametrize("dtype_name,ncols", [("f64", 1), ("f32", 1), ("f64", 2), ("f64", 3)])
@pytest.mark.parametrize("variant", ["plain", "locality", "locality3"])
def test_world_of_many_ranks(variant, dtype_name, ncols):
    """More ranks than CUs (no smaller tiles), few rows each."""
    need_gpu()
    say("many ranks", variant, dtype_name, ncols)
    rs, rp, cols = random_small_csr(3000, 300, 6, 0.5, 91, True)
    check_world_against_oracle(rs, rp, cols, 16, variant, ncols, dtype_name, n_variants=2)
