"""Rows of any number of values (the flat forms of the gathers, the push pack
and the segmented sum), bit for bit against the oracle: row sizes around the
vector widths and the form's limits, buffers off the 16-byte grid, tiles
beyond the staging limits, and a row with more terms than a tile stages."""
import numpy as np
import pytest

import paper_2309_07337_amd as P
from oracle import move as OM
from oracle import plan as OP
from tests.gpu_util import bits_equal, dev, host, need_gpu, say
from workloads import splitmix64, uniform_pm1

pytestmark = pytest.mark.gpu

# values per row: 4-, 8- and 16-byte vectors, and 1023, 1024 and 1025 vectors a
# row on either side of the largest flat row
SIZES = [("f32", c, 5000) for c in (3, 5, 7, 9, 12, 25, 100)] + [("f64", c, 5000) for c in (3, 5, 6, 25)] + \
        [("f32", 1023, 60), ("f32", 1025, 60), ("f64", 1023, 60), ("f64", 2046, 30), ("f64", 2048, 30), ("f64", 2050, 30)]
SCHEDS = [None,
          dict(tile_rows=16384, unroll=1, push_pack=2),            # chunks of a tile, no staging
          dict(tile_rows=333, unroll=2, push_pack=1, nontemporal=1),
          dict(tile_rows=512, block_threads=512, blocks_per_cu=2, push_pack=1, unroll=4),
          dict(tile_rows=7, blocks_per_cu=1 << 20, push_pack=2, per_neighbor=1)]


@pytest.mark.parametrize("dtype_name,ncols,n", SIZES)
@pytest.mark.parametrize("shift", [0, 1])
def test_any_row_size(dtype_name, ncols, n, shift):
    """shift: every caller buffer starts one value past a 16-byte boundary."""
    need_gpu()
    import torch
    say("row size", dtype_name, ncols, n, shift)
    dt = torch.float64 if dtype_name == "f64" else torch.float32
    npdt = np.float64 if dtype_name == "f64" else np.float32

    def buf(rows, values=None):
        t = torch.full((rows * ncols + shift,), float("nan"), dtype=dt, device="cuda")[shift:].view(rows, ncols)
        if values is not None:
            t.copy_(dev(values))
        return t

    hot = 2500 if n > 100 else 10   # slots of one row
    counts = [n // 2, 1, n - n // 2, hot]
    idx = (splitmix64(ncols, 0, sum(counts)) % np.uint64(n)).astype(np.int32)
    idx[-hot:] = n // 3
    E = idx.size
    xh, rh, gh = (uniform_pm1(s, r * ncols).reshape(r, ncols).astype(npdt) for s, r in ((1, n), (2, E), (3, E)))
    x, halo, g, gx = buf(n, xh), buf(E), buf(E, gh), buf(n)
    topo = P.hx_topo_create(0, 8, [1, 2, 3, 4], [1, 2, 3, 4])
    req = P.hx_neighbor_alltoallv_init(x, counts, None, idx, halo, counts, None, topo)
    P.req_arena_view(req, P.HX_ARENA_RECV, ncols, dt).copy_(dev(rh))
    P.hx_req_bind_grad(req, g, gx)
    ptr, perm = OP.transpose_csr(idx, n)
    want_send, want_gx = OM.pack(xh, idx), OM.pack_transpose(gh, ptr, perm)
    for sched in SCHEDS:
        say("  sched", sched)
        for t in (halo, gx, P.req_arena_view(req, P.HX_ARENA_SEND, ncols, dt)):
            t.fill_(float("nan"))
        b = P.hx_batch_init([req], sched=sched)
        P.hx_batch_start(b)
        P.hx_batch_wait(b)
        P.hx_batch_backward(b)
        assert bits_equal(host(P.req_arena_view(req, P.HX_ARENA_SEND, ncols, dt)), want_send)
        assert bits_equal(host(halo), rh)
        assert bits_equal(host(gx), want_gx)
        b.free()
    gx.fill_(float("nan"))
    P.hx_backward_noalloc(req, g, gx)
    assert bits_equal(host(gx), want_gx)
