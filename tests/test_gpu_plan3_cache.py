"""The cache of 3-D mode lists drops the list that was used least recently: a
list that every step uses stays, however many others come and go.  The cached
object is looked at through the library's own lookup (a shared pointer of 16
bytes, kept, so that a dropped object's address is not given out again)."""
from __future__ import annotations

import ctypes
import os

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_a_list_in_use_is_kept():
    import paper_2409_19156_amd as zp
    from paper_2409_19156_amd import _lib

    lib = _lib.load()
    lookup = getattr(lib, "_ZN2zp9get_plan3EPKiS1_S1_lPSt10shared_ptrINS_5Plan3EE")
    lookup.argtypes = [ctypes.c_void_p] * 3 + [ctypes.c_int64, ctypes.c_void_p]
    x = torch.full((4,), 0.5, dtype=torch.float64, device="cuda")

    def modes(l):
        return tuple(np.array([v], np.int32) for v in (2, 0, l))

    def use(l):
        zp.series3d_forward(*modes(l), x, x, x, torch.ones(1, 1, dtype=torch.float64, device="cuda"))

    def cached(l):
        out = (ctypes.c_void_p * 2)()
        n, m, ll = modes(l)
        assert lookup(n.ctypes.data, m.ctypes.data, ll.ctypes.data, 1, ctypes.addressof(out)) == 0
        return out[0]

    lib.zp_cache_clear()
    first = cached(0)
    for l in range(1, 3 * int(os.environ.get("ZP_PLAN_CACHE", "16"))):
        use(l)
        use(0)
    assert cached(0) == first
    torch.cuda.synchronize()
