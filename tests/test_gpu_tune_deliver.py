"""Tuning a world with the simulated transfer times the kernels that its steps
launch (each row written to its receiver too), and keeps their schedules apart
from those of a world without it."""
import numpy as np
import pytest

import paper_2309_07337_amd as P
from oracle import move as OM
from oracle import plan as OP
from tests.gpu_util import bits_equal, dev, gpu_plan, host, need_gpu, say
from workloads import random_small_csr, uniform_pm1

pytestmark = pytest.mark.gpu
N, R, NCOLS = 700, 9, 3
PACK, REDIST, UNPACK, BWD = range(4)


def world(flags):
    import torch
    rs, rp, cols = random_small_csr(N, R, 9, 0.5, 55, True)
    halos = OP.all_halos(rp, cols, rs)
    H = sum(h.size for h in halos)
    x, g = (uniform_pm1(k, r * NCOLS).reshape(r, NCOLS) for k, r in ((1, N), (2, H)))
    t = [dev(x), torch.empty((H, NCOLS), dtype=torch.float64, device="cuda"), dev(g),
         torch.empty((N, NCOLS), dtype=torch.float64, device="cuda")]
    b = P.hx_batch_from_plan(gpu_plan(rs, rp, cols, 3, "locality"), t[0], t[1], flags=flags)
    P.hx_batch_bind_grad(b, t[2], t[3])
    D = OP.Decomposition(halos, rs, 3)
    want_g = OM.staged_adjoint_reference([D.plan(r, "locality") for r in range(R)],
                                         np.split(g, np.cumsum([h.size for h in halos])[:-1]), rs)["g_x"]
    return b, t, x[np.concatenate(halos)], want_g


def keys(path):
    return [line.split()[0] for line in path.read_text().splitlines()]


def test_tuned_deliveries(tmp_path, monkeypatch):
    need_gpu()
    import torch
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("HX_TUNE_CACHE", str(cache))
    say("tune, delivering")
    staged = P.HX_WORLD_STAGED_BACKWARD
    b, t, want, want_g = world(P.HX_WORLD_SIM_TRANSFER | staged)
    recv = P.batch_arena_view(b, P.HX_ARENA_RECV, NCOLS, torch.float64)
    back = P.batch_arena_view(b, P.HX_ARENA_GRAD_SEND, NCOLS, torch.float64)
    recv.fill_(float("nan"))
    back.fill_(float("nan"))
    P.hx_batch_tune(b)
    assert torch.isfinite(recv).all() and torch.isfinite(back).all()     # the candidates delivered
    for a in (recv, back, t[1], t[3]):
        a.fill_(float("nan"))
    P.hx_batch_start(b)
    P.hx_batch_wait(b)
    P.hx_batch_backward(b)
    assert bits_equal(host(t[1]), want) and bits_equal(host(t[3]), want_g)
    tuned, mine = [P.hx_batch_get_sched(b, ph) for ph in range(4)], keys(cache)
    assert len(mine) == 4
    again = world(P.HX_WORLD_SIM_TRANSFER | staged)[0]
    assert [P.hx_batch_get_sched(again, ph) for ph in range(4)] == tuned
    # a world that does not deliver shares the unpack's schedule alone
    other = world(staged)[0]
    P.hx_batch_tune(other)
    theirs = keys(cache)[4:]
    assert [mine[ph] == theirs[ph] for ph in range(4)] == [False, False, True, False]
    # a file without deliveries' own keys serves the shape
    old = [line for line in cache.read_text().splitlines() if line.split()[0] in theirs]
    cache.write_text("\n".join(old) + "\n")
    scheds = [P.hx_batch_get_sched(other, ph) for ph in range(4)]
    served = world(P.HX_WORLD_SIM_TRANSFER | staged)[0]
    assert [P.hx_batch_get_sched(served, ph) for ph in range(4)] == scheds
