"""The forward contraction's small workgroup tiles against its wide ones: an
output element's sum does not depend on the tile, the number of points or the
other sets, so a call on few points and sets returns the bits that a call
whose launch takes wide tiles returned for the same points and sets.  (That
the wide call is right is tested against the oracle in test_gpu_series.py.)
"""
from __future__ import annotations

import pytest
import torch

import zp_workloads as W

pytestmark = pytest.mark.gpu

# tile edges: 64 points x 64 sets (FP32, FP64), 128 x 32 (bf16 x 3)
EDGES = [(1, 1), (63, 31), (64, 32), (65, 33), (127, 63), (128, 64), (129, 65), (300, 127), (1000, 128), (20000, 100)]


@pytest.mark.parametrize("prec", ["fp32", "bf16x3", "fp64"])
def test_small_tiles_return_the_bits_of_wide_ones(prec):
    import paper_2409_19156_amd as zp

    n, m = W.ansi_modes(13)
    P, extra = 65536, 128 if prec == "fp64" else 0  # (fewer FP64 sets take another kernel)
    gen = torch.Generator(device="cuda").manual_seed(5)
    r = torch.rand(P, dtype=torch.float64, device="cuda", generator=gen).sqrt()
    th = 6.28 * torch.rand(P, dtype=torch.float64, device="cuda", generator=gen)
    c = torch.randn(n.size, 128 + extra, dtype=torch.float64, device="cuda", generator=gen)
    wide = zp.series_forward(n, m, r, th, c, prec)
    for p, b in EDGES:
        b += extra
        print(f"  {prec} {p} points, {b} sets", flush=True)
        small = zp.series_forward(n, m, r[:p].clone(), th[:p].clone(), c[:, :b].contiguous(), prec)
        assert torch.equal(small, wide[:p, :b]), (prec, p, b)
