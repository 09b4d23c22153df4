"""The simulated transfer as the packs' second destination: send and receive
arenas of every stage bit for bit against the oracle, over the kernel forms
(row sizes around the vector widths and the flat form's limit, pull and push),
and left alone where no transfer is asked for."""
import numpy as np
import pytest

import paper_2309_07337_amd as P
from oracle import plan as OP
from tests.gpu_util import bits_equal, dev, gpu_plan, host, need_gpu, say
from tests.test_gpu_world import check_world_against_oracle
from workloads import random_small_csr, uniform_pm1

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant", ["plain", "locality", "locality3"])
@pytest.mark.parametrize("dtype_name,ncols", [("f64", 1), ("f32", 1), ("f32", 2), ("f64", 2), ("f64", 5), ("f32", 7),
                                              ("f64", 16), ("f32", 100), ("f32", 1025), ("f64", 2050)])
def test_delivery_row_sizes(variant, dtype_name, ncols):
    need_gpu()
    say("delivery", variant, dtype_name, ncols)
    rs, rp, cols = random_small_csr(300, 9, 9, 0.5, 77, True)
    check_world_against_oracle(rs, rp, cols, 4, variant, ncols, dtype_name)


@pytest.mark.parametrize("push", [1, 2])
def test_no_delivery_without_a_transfer(push):
    """One phase's kernel alone, and a world without the simulated transfer,
    write the send arena only."""
    need_gpu()
    import torch
    say("no delivery", push)
    rs, rp, cols = random_small_csr(300, 9, 9, 0.5, 78, False)
    halos = OP.all_halos(rp, cols, rs)
    x = dev(uniform_pm1(3, 300).reshape(300, 1))
    halo = torch.zeros((sum(h.size for h in halos), 1), dtype=torch.float64, device="cuda")
    plan = gpu_plan(rs, rp, cols, 4, "locality")
    for flags in (P.HX_WORLD_SIM_TRANSFER, 0):
        b = P.hx_batch_from_plan(plan, x, halo, flags=flags, sched=dict(push_pack=push))
        recv = P.batch_arena_view(b, P.HX_ARENA_RECV, 1, torch.float64)
        recv.fill_(float("nan"))
        P.hx_batch_launch_phase(b, 0)
        P.hx_batch_launch_phase(b, 1)
        if not flags:
            P.hx_batch_start(b)
            P.hx_batch_wait(b)
        assert np.isnan(host(recv)).all()
        if flags:   # the whole step afterwards delivers
            P.hx_batch_start(b)
            P.hx_batch_wait(b)
            assert bits_equal(host(halo), host(x)[np.concatenate(halos)])
        b.free()
