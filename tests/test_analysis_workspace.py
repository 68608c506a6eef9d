"""The analysis asks for the planar backward's workspace and nothing for the
samples, which it weighs where it reads them; a byte less than the minimum is
refused before any device work (host only)."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest

ERR_WS = 4
FAKE = ctypes.c_void_p(0x10000)


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("M,P,B", [(1, 1, 1), (91, 4257, 64), (2145, 131072, 1024)])
def test_no_room_for_a_copy(M, P, B, prec):
    from paper_2409_19156_amd import _lib

    lib = _lib.load()
    a, b, c, d = (ctypes.c_size_t() for _ in range(4))
    assert lib.zp_series_analysis_workspace(M, P, B, prec, ctypes.byref(a), ctypes.byref(b)) == 0
    assert lib.zp_series_workspace(M, P, B, prec, ctypes.byref(c), ctypes.byref(d)) == 0
    assert (a.value, b.value) == (c.value, d.value)
    n = np.zeros(M, np.int32)
    st = lib.zp_series_analysis(n.ctypes.data, n.ctypes.data, M, FAKE, FAKE, FAKE, P, FAKE, B, prec, FAKE, FAKE,
                                b.value - 1, None)
    assert st == ERR_WS
