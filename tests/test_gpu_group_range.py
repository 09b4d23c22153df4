"""Grouping by key refuses keys outside its range before it writes a pointer for
them: the pointer array and what lies around it stay as they were."""
import ctypes as C

import numpy as np
import pytest

import paper_2309_07337_amd as P
from tests.gpu_util import dev, host, need_gpu, say

pytestmark = pytest.mark.gpu

# int hx::dev_group_by_key(const int32_t* keys, int64_t n, int64_t nkeys, int32_t* ptr, int32_t* perm,
#                          hipStream_t s, bool checked)
NAME = "_ZN2hx16dev_group_by_keyEPKillPiS2_P12ihipStream_tb"


@pytest.mark.parametrize("n,nkeys", [(1, 1), (5, 3), (4097, 300), (9000, 70_000)])
@pytest.mark.parametrize("bad", [None, -1, -9, "nkeys", 1 << 30])
@pytest.mark.parametrize("where", ["first", "last", "all"])
def test_keys_outside(n, nkeys, bad, where):
    need_gpu()
    import torch
    say("group range", n, nkeys, bad, where)
    group = getattr(P.load(), NAME)
    group.restype, group.argtypes = C.c_int, [C.c_void_p, C.c_int64, C.c_int64] + [C.c_void_p] * 3 + [C.c_bool]
    keys = (np.arange(n, dtype=np.int64) * 7919 % nkeys).astype(np.int32)
    if bad is not None:
        keys[{"first": 0, "last": n - 1, "all": slice(None)}[where]] = nkeys if bad == "nkeys" else bad
    k, guard = dev(keys), 64
    ptr = torch.full((nkeys + 1 + 2 * guard,), -7, dtype=torch.int32, device="cuda")
    perm = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    rc = group(k.data_ptr(), n, nkeys, ptr.data_ptr() + 4 * guard, perm.data_ptr(), None, False)
    got = host(ptr)
    assert (got[:guard] == -7).all() and (got[-guard:] == -7).all()
    if bad is not None:
        assert rc == P.HX_ERR_RANGE and (got == -7).all()
        return
    assert rc == P.HX_SUCCESS
    assert np.array_equal(got[guard:-guard], np.searchsorted(np.sort(keys), np.arange(nkeys + 1)))
    assert np.array_equal(host(perm), np.argsort(keys, kind="stable"))
