"""Transposes of the pack maps where their forms change: few ranks and ranks too
large for LDS (radix grouping), many small ones (one workgroup a rank), rows
packed for few ranks and for more than a lane sorts; against numpy."""
import numpy as np
import pytest

import paper_2309_07337_amd as P
from tests.gpu_util import dev, need_gpu, say
from workloads import splitmix64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R,rows,per_rank,hot", [(7, 40, 30, 0), (8, 40, 30, 0), (9, 1, 3, 0), (30, 500, 300, 0),
                                                 (24, 70, 100, 1), (25, 70, 100, 2), (26, 70, 100, 70), (300, 20, 60, 3),
                                                 (9, 19_000, 18_000, 1), (9, 40_000, 2_000, 0)])
@pytest.mark.parametrize("variant", ["plain", "2step", "3step"])
def test_pack_transpose(R, rows, per_rank, hot, variant):
    """Every rank needs per_rank columns of the others, among them the first hot
    rows of each (a row packed for R - 1 ranks)."""
    need_gpu()
    say("transpose", R, rows, per_rank, hot, variant)
    n = R * rows
    rs = np.arange(R + 1, dtype=np.int64) * rows
    cols = []
    for r in range(R):
        c = (splitmix64(1000 + r, 0, per_rank) % np.uint64(n)).astype(np.int64)
        first = (np.arange(R)[:, None] * rows + np.arange(hot)[None, :]).reshape(-1)
        c = np.unique(np.concatenate([c, first]))
        cols.append(c[(c < rs[r]) | (c >= rs[r + 1])])
    ptr = np.concatenate([[0], np.cumsum([c.size for c in cols])]).astype(np.int64)
    plan = P.hx_plan_from_halos(R, rs, 4, {"plain": P.HX_PLAIN, "2step": P.HX_LOCALITY_2STEP,
                                           "3step": P.HX_LOCALITY_3STEP}[variant], ptr,
                                dev(np.concatenate(cols).astype(np.int32)))
    io, idx = P.hx_plan_field_all(plan, "s1_idx")
    po, bt_ptr = P.hx_plan_field_all(plan, "bt_ptr")
    qo, bt_perm = P.hx_plan_field_all(plan, "bt_perm")
    for q in range(R):
        i, p, e = idx[io[q]:io[q + 1]], bt_ptr[po[q]:po[q + 1]], bt_perm[qo[q]:qo[q + 1]]
        assert np.array_equal(e, np.argsort(i, kind="stable"))
        assert np.array_equal(p, np.searchsorted(np.sort(i), np.arange(p.size)))
