"""Pack transposes with rows packed for many ranks, at the lengths where the
sorting changes hands (one lane, the workgroup), and what such rows cost the
plan; against numpy."""
import time

import numpy as np
import pytest

import paper_2309_07337_amd as P
from tests.gpu_util import dev, need_gpu, say

pytestmark = pytest.mark.gpu


def fan_plan(R, lengths, rows=None, variant=None, reps=1):
    """Plan of R ranks in which row i of every rank goes to the next lengths[i]
    ranks; and the shortest time it took to build."""
    import torch
    rows = len(lengths) if rows is None else rows
    lengths = np.asarray(lengths)
    halos = []
    for r in range(R):
        owner = (r - np.arange(1, R)) % R                       # owners, 1 .. R - 1 ranks before r
        i, d = np.nonzero(lengths[:, None] > np.arange(R - 1)[None, :])
        halos.append(np.sort(owner[d] * rows + i))
    ptr = np.concatenate([[0], np.cumsum([h.size for h in halos])]).astype(np.int64)
    cols, rs = dev(np.concatenate(halos).astype(np.int32)), np.arange(R + 1, dtype=np.int64) * rows
    best = 1e9
    for _ in range(reps):
        torch.cuda.synchronize()
        t = time.perf_counter()
        plan = P.hx_plan_from_halos(R, rs, 4, P.HX_PLAIN if variant is None else variant, ptr, cols)
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t)
    return plan, best


def check(plan, R):
    io, idx = P.hx_plan_field_all(plan, "s1_idx")
    po, ptr = P.hx_plan_field_all(plan, "bt_ptr")
    qo, perm = P.hx_plan_field_all(plan, "bt_perm")
    longest = 0
    for q in range(R):
        i, p, e = idx[io[q]:io[q + 1]], ptr[po[q]:po[q + 1]], perm[qo[q]:qo[q + 1]]
        assert np.array_equal(e, np.argsort(i, kind="stable"))
        assert np.array_equal(p, np.searchsorted(np.sort(i), np.arange(p.size)))
        longest = max(longest, int(np.diff(p).max()))
    return longest


@pytest.mark.parametrize("R,lengths", [
    (270, [0, 24, 25, 1, 26, 63, 64, 65, 2, 128, 129, 255, 256, 257, 269, 0]), (270, [269]), (270, [0] * 700 + [257]),
    (270, [25] * 130), (270, [269] * 100), (100, [24, 25] * 400), (600, [599, 3, 513, 0, 512, 400])])
def test_lengths(R, lengths):
    need_gpu()
    say("long rows", R, lengths[:4], len(lengths))
    plan, _ = fan_plan(R, lengths)
    assert check(plan, R) == max(lengths)


def test_three_steps():
    """Rows of a node's ranks; the aggregated messages share theirs."""
    need_gpu()
    plan, _ = fan_plan(120, [100, 3, 119, 60], variant=P.HX_LOCALITY_3STEP)
    check(plan, 120)


@pytest.mark.parametrize("R,lengths,rows,long_lengths", [
    (64, [3] * 5000, 20_000, [63] + [3] * 4999),            # one long row among many
    (64, [24] * 900, None, [25] * 900)])                    # every row a slot longer
def test_cost(R, lengths, rows, long_lengths):
    """Longer rows cost what their slots do, not a walk over every row each."""
    need_gpu()
    short, long = (fan_plan(R, v, rows, reps=7)[1] for v in (lengths, long_lengths))
    say(f"long rows, plan {short * 1e6:.0f} -> {long * 1e6:.0f} us")
    assert long < 2 * short
