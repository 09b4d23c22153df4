"""Grouping by key (the transpose of the pack map, the adjoint of the halo) at
the edges of its radix sort: keys at and past a digit's range, entries around
a workgroup's share, and one key that every rank's entries share."""
import numpy as np
import pytest

import paper_2309_07337_amd as P
from oracle import move as OM
from oracle import plan as OP
from tests.gpu_util import bits_equal, dev, host, need_gpu, say
from workloads import splitmix64, uniform_pm1

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,ranks,halo", [(2, 2, 1), (2048, 2, 700), (2049, 3, 700), (4096, 5, 1640), (4096, 9, 910),
                                          (4097, 9, 911), ((1 << 22) + 1, 3, 4096), (60_000, 40, 9000)])
def test_transposes_of_a_plan(n, ranks, halo):
    """Plain plan of `ranks` ranks with up to `halo` random halo columns each
    (column 0 or n - 1 in every halo that may hold it): every rank's pack
    transpose and the exchange's backward equal the oracle's."""
    need_gpu()
    import torch
    say("group", n, ranks, halo)
    rs = np.arange(ranks + 1, dtype=np.int64) * n // ranks
    halos = []
    for r in range(ranks):
        c = np.concatenate([[0, n - 1], (splitmix64(n + r, 0, halo) % np.uint64(n)).astype(np.int64)])
        halos.append(np.unique(c[(c < rs[r]) | (c >= rs[r + 1])]))
    ptr = np.concatenate([[0], np.cumsum([h.size for h in halos])]).astype(np.int64)
    cols = np.concatenate(halos).astype(np.int32)
    plan = P.hx_plan_from_halos(ranks, rs, 1, P.HX_PLAIN, ptr, dev(cols))
    for r in range(ranks):
        idx = P.hx_plan_field(plan, r, "s1_idx")
        want_ptr, want_perm = OP.transpose_csr(idx, int(rs[r + 1] - rs[r]))
        assert np.array_equal(P.hx_plan_field(plan, r, "bt_ptr"), want_ptr)
        assert np.array_equal(P.hx_plan_field(plan, r, "bt_perm"), want_perm)
    g = uniform_pm1(5, cols.size).reshape(-1, 1)
    x, gx = torch.zeros(n, 1, dtype=torch.float64, device="cuda"), torch.full((n, 1), float("nan"),
                                                                               dtype=torch.float64, device="cuda")
    hal = torch.zeros(cols.size, 1, dtype=torch.float64, device="cuda")
    b = P.hx_batch_from_plan(plan, x, hal, flags=P.HX_WORLD_SIM_TRANSFER)
    P.hx_batch_bind_grad(b, dev(g), gx)
    P.hx_batch_backward(b)
    aptr, aperm = OP.transpose_csr(cols, n)
    assert bits_equal(host(gx), OM.pack_transpose(g, aptr, aperm))
