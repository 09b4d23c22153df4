"""Halo discovery where its forms change: few ranks (one bitmap pass over all of
them) and many (a rank's bitmap in LDS), one to four segments of 2^20 columns
and more, empty ranks and rows, entries off the 16-byte grid; against numpy."""
import numpy as np
import pytest

import paper_2309_07337_amd as P
from tests.gpu_util import dev, need_gpu, say
from workloads import splitmix64

pytestmark = pytest.mark.gpu

S = 1 << 20


def matrix(n, R, seed):
    """Ranks of uneven sizes, one of them empty; rows of 0 to 4 entries, half of
    them near; the entries start at row_ptr[0] = 3 of a larger array."""
    u = splitmix64(seed, 0, n).astype(np.uint64)
    cuts = np.sort(splitmix64(seed + 1, 0, R - 1) % np.uint64(n + 1)).astype(np.int64) if R > 1 else np.zeros(0, np.int64)
    rs = np.concatenate([[0], cuts, [n]])
    if R > 3:
        rs[2] = rs[1]
    rp = np.concatenate([[0], np.cumsum((u >> np.uint64(40)) % np.uint64(5))]).astype(np.int64) + 3
    v = splitmix64(seed + 2, 0, int(rp[-1]))
    row = np.repeat(np.arange(n), np.diff(rp))
    near = np.clip(row + (v[3:] >> np.uint64(50)).astype(np.int64) - 8192, 0, n - 1)
    cols = np.zeros(int(rp[-1]), np.int32)
    cols[3:] = np.where(v[3:] & np.uint64(1), near, (v[3:] >> np.uint64(8)).astype(np.int64) % n)
    return rs, rp, cols


@pytest.mark.parametrize("n,R", [(1, 1), (5, 2), (1000, 7), (1000, 8), (4099, 23), (S, 9), (S + 1, 9), (2 * S + 129, 7),
                                 (2 * S + 129, 17), (4 * S, 8), (4 * S + 3, 8)])
def test_halo_discovery(n, R):
    need_gpu()
    say("discovery", n, R)
    rs, rp, cols = matrix(n, R, 100 + R)
    row = np.repeat(np.arange(n), np.diff(rp))
    rank = np.searchsorted(rs, row, side="right") - 1
    c = cols[3:].astype(np.int64)
    off = (c < rs[rank]) | (c >= rs[rank + 1])
    key = np.unique(rank[off] * n + c[off])
    want = (key % n).astype(np.int32)
    off_want = np.searchsorted(key, np.arange(R + 1) * n)
    drp, dcols = dev(rp), dev(cols)
    for variant in (P.HX_PLAIN, P.HX_LOCALITY_2STEP):
        plan = P.hx_plan_from_csr(R, rs, 3, variant, drp, dcols)
        offs, halo = P.hx_plan_field_all(plan, "halo")
        assert np.array_equal(offs, off_want) and np.array_equal(halo, want)
        # the lists built from the discovered halos and from given ones are the same
        other = P.hx_plan_from_halos(R, rs, 3, variant, off_want, dev(want))
        for f in P.FIELDS:
            (oa, a), (ob, b) = P.hx_plan_field_all(plan, f), P.hx_plan_field_all(other, f)
            assert np.array_equal(oa, ob) and np.array_equal(a, b), f


@pytest.mark.parametrize("R", [2, 9])
def test_discovery_refuses(R):
    need_gpu()
    n = 1000
    rs, rp, cols = matrix(n, R, 7)
    for bad_rp, bad_col in ((True, None), (False, -1), (False, n)):
        say("refused", R, bad_rp, bad_col)
        p, c = rp.copy(), cols.copy()
        if bad_rp:
            p[n // 2] = p[n // 2 + 1] + 1
        else:
            c[10] = bad_col
        with pytest.raises(P.HXError) as e:
            P.hx_plan_from_csr(R, rs, 3, P.HX_PLAIN, dev(p), dev(c))
        assert e.value.code == (-1 if bad_rp else -2)
