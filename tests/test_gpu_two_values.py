"""Backward of rows of two FP32 values under the default schedules: few and many
terms a row, windows that fit and that do not, one request, worlds and the call
that allocates nothing, bit for bit against the oracle."""
import numpy as np
import pytest

import paper_2309_07337_amd as P
from oracle import move as OM
from oracle import plan as OP
from tests.gpu_util import bits_equal, dev, host, need_gpu, say
from tests.test_gpu_world import check_world_against_oracle
from workloads import random_small_csr, splitmix64, uniform_pm1

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,E", [(1, 1), (300, 90), (9000, 8000), (900, 9000), (1000, 30_000), (40_000, 300_000),
                                 (400_000, 350_000)])
def test_request(n, E):
    need_gpu()
    import torch
    say("two values", n, E)
    idx = (splitmix64(3, 0, E) % np.uint64(n)).astype(np.int32)
    gh = uniform_pm1(4, 2 * E).reshape(E, 2).astype(np.float32)
    x, halo = torch.zeros((n, 2), device="cuda"), torch.zeros((E, 2), device="cuda")
    topo = P.hx_topo_create(0, 8, [1], [1])
    req = P.hx_neighbor_alltoallv_init(x, [E], None, idx, halo, [E], None, topo)
    g, gx = dev(gh), torch.empty((n, 2), device="cuda")
    P.hx_req_bind_grad(req, g, gx)
    want = OM.pack_transpose(gh, *OP.transpose_csr(idx, n))
    b = P.hx_batch_init([req])
    for step in (lambda: P.hx_backward(req), lambda: P.hx_backward_noalloc(req, g, gx), lambda: P.hx_batch_backward(b)):
        gx.fill_(float("nan"))
        step()
        assert bits_equal(host(gx), want)
    b.free()


@pytest.mark.parametrize("variant", ["plain", "locality", "locality3"])
@pytest.mark.parametrize("rows,ranks,nnz", [(3000, 300, 6), (4000, 8, 30), (2000, 40, 12)])
def test_world(variant, rows, ranks, nnz):
    need_gpu()
    say("two values", variant, rows, ranks, nnz)
    rs, rp, cols = random_small_csr(rows, ranks, nnz, 0.5, 91, True)
    check_world_against_oracle(rs, rp, cols, max(2, ranks // 8), variant, 2, "f32", n_variants=2)
