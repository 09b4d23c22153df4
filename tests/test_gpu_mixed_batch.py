"""Batches whose members unpack in both ways, as one contiguous copy (plain
requests) and through an index list (locality requests): every form of the
batch against the oracle, bit for bit."""
import numpy as np
import pytest

import paper_2309_07337_amd as P
from oracle import move as OM
from oracle import plan as OP
from tests.gpu_util import bits_equal, dev, gpu_plan, host, need_gpu, plan_rank, say
from workloads import random_small_csr, splitmix64, uniform_pm1

pytestmark = pytest.mark.gpu


def filled(seed, rows, ncols, dt):
    return dev(uniform_pm1(seed, rows * ncols).reshape(rows, ncols)).to(dt)


def plain_member(seed, n, ncols, dt):
    import torch
    E = n + 7
    idx = (splitmix64(seed, 0, E) % np.uint64(n)).astype(np.int32)
    counts = [E // 3, E - E // 3]
    x, halo = filled(seed, n, ncols, dt), torch.empty((E, ncols), dtype=dt, device="cuda")
    topo = P.hx_topo_create(0, 8, [1, 2], [1, 2])
    req = P.hx_neighbor_alltoallv_init(x, counts, None, idx, halo, counts, None, topo)
    return dict(req=req, x=x, halo=halo, s1_idx=idx, s2_src=idx[:0], unpack=np.arange(E))


def locality_member(plan, rs, rank, seed, ncols, dt):
    import torch
    f = plan_rank(plan, rank)
    x = filled(seed, int(rs[rank + 1] - rs[rank]), ncols, dt)
    halo = torch.empty((f["halo"].size, ncols), dtype=dt, device="cuda")
    req = P.hx_req_from_plan(plan, rank, x, halo)
    return dict(req=req, x=x, halo=halo, s1_idx=f["s1_idx"], s2_src=f["s2_src"], unpack=f["unpack_src"])


@pytest.mark.parametrize("dtype_name,ncols", [("f64", 1), ("f32", 1), ("f32", 3), ("f64", 5), ("f64", 16)])
def test_plain_and_locality_members(dtype_name, ncols):
    need_gpu()
    import torch
    say("mixed batch", dtype_name, ncols)
    dt = torch.float64 if dtype_name == "f64" else torch.float32
    rs, rp, cols = random_small_csr(900, 12, 9, 0.5, 17, True)
    plan = gpu_plan(rs, rp, cols, 4, "locality")
    mem = [plain_member(31, 400, ncols, dt), locality_member(plan, rs, 3, 32, ncols, dt),
           plain_member(33, 1, ncols, dt), locality_member(plan, rs, 8, 34, ncols, dt)]
    for k, m in enumerate(mem):
        m["recv"] = P.req_arena_view(m["req"], P.HX_ARENA_RECV, ncols, dt)
        m["recv"].copy_(filled(50 + k, m["recv"].shape[0], ncols, dt))
        m["send"] = P.req_arena_view(m["req"], P.HX_ARENA_SEND, ncols, dt)
        m["g"] = filled(60 + k, m["s1_idx"].size, ncols, dt)
        m["gx"] = torch.empty_like(m["x"])
        P.hx_req_bind_grad(m["req"], m["g"], m["gx"])
        ptr, perm = OP.transpose_csr(m["s1_idx"], m["x"].shape[0])
        recv = host(m["recv"])
        m["want"] = (np.concatenate([OM.pack(host(m["x"]), m["s1_idx"]), recv[m["s2_src"]]]), recv[m["unpack"]],
                     OM.pack_transpose(host(m["g"]), ptr, perm))

    def check(step):
        for m in mem:
            for t in (m["send"], m["halo"], m["gx"]):
                t.fill_(float("nan"))
        step()
        for m in mem:
            for t, want in zip((m["send"], m["halo"], m["gx"]), m["want"]):
                assert bits_equal(host(t), want)

    def batched(b):
        check(lambda: (P.hx_batch_start(b), P.hx_batch_wait(b), P.hx_batch_backward(b)))

    for sched in (None, dict(tile_rows=33, per_neighbor=1), dict(pair_rows=1, lds_window=1, tile_rows=100)):
        b = P.hx_batch_init([m["req"] for m in mem], sched=sched)
        batched(b)
        check(lambda: (P.hx_batch_start_plain(b), P.hx_batch_wait_plain(b), P.hx_batch_backward_plain(b)))
        P.hx_batch_set_sched(b, 2, dict(tile_rows=17))
        batched(b)
        check(lambda: [P.hx_batch_launch_phase(b, ph) for ph in range(4)])
        if sched is None:
            P.hx_batch_tune(b)
            batched(b)
        b.free()
    check(lambda: [(P.hx_start(m["req"]), P.hx_wait(m["req"]), P.hx_backward(m["req"])) for m in mem])
