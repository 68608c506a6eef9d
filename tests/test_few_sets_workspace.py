"""FP64 calls of few sets store no basis planes and ask for no room for them: the
full workspace of up to 32 sets is 64 MiB at most, or what the smallest one or the
gradient's partial sums take, whatever the number of points (host only), and more
room changes no bit."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest

import zp_workloads as W

MIB = 1 << 20


def _full(lib, name, *args):
    full, least = ctypes.c_size_t(), ctypes.c_size_t()
    assert getattr(lib, name)(*args, ctypes.byref(full), ctypes.byref(least)) == 0
    assert full.value >= least.value
    return full.value


@pytest.mark.parametrize("name", ["zp_series_workspace", "zp_series_bwd2_workspace", "zp_series_analysis_workspace"])
def test_no_room_for_planes(name):
    from paper_2409_19156_amd import _lib

    lib = _lib.load()
    for P in (65536, 1 << 24):
        for B in (1, 16, 32):
            assert _full(lib, name, 2145, P, B, 0) <= 64 * MIB, (P, B)
        assert _full(lib, name, 2145, P, 33, 0) > 8 * 2145 * P  # a plane of the basis
        assert _full(lib, name, 2145, P, 32, 1) > 4 * 2145 * P


@pytest.mark.gpu
@pytest.mark.parametrize("B", [1, 17, 32])
def test_more_room_changes_nothing(B):
    import torch

    import paper_2409_19156_amd as zp

    n, m = W.ansi_modes(20)
    P = 20000
    gen = torch.Generator(device="cuda").manual_seed(B)
    rand = lambda *s: torch.rand(*s, dtype=torch.float64, device="cuda", generator=gen)  # noqa: E731
    r, th, c, g, uc, ur, ut = rand(P), rand(P), rand(n.size, B), rand(P, B), rand(n.size, B), rand(P), rand(P)
    big = torch.empty(512 * MIB, dtype=torch.uint8, device="cuda")
    args = (n, m, r, th, c)
    assert torch.equal(zp.series_forward(*args, "fp64"), zp.series_forward(*args, "fp64", ws=big))
    for a, b in zip(zp.series_backward(*args, g, "fp64"), zp.series_backward(*args, g, "fp64", ws=big)):
        assert torch.equal(a, b)
    a, b = (zp.series_jvp(*args, uc, ur, ut, "fp64", **kw) for kw in ({}, {"ws": big}))
    assert torch.equal(a, b)
    for a, b in zip(zp.series_backward2(*args, g, uc, ur, ut, "fp64"),
                    zp.series_backward2(*args, g, uc, ur, ut, "fp64", ws=big)):
        assert torch.equal(a, b)
    w = rand(P)
    assert torch.equal(zp.series_analysis(n, m, r, th, w, g, "fp64"),
                       zp.series_analysis(n, m, r, th, w, g, "fp64", ws=big))
