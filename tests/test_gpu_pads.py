"""The backward contractions leave the pad modes of their basis operand as the
workspace held them: whatever that was (here NaN bit patterns), the results are
the bits that a zeroed workspace gives.
"""
from __future__ import annotations

import pytest
import torch

import zp_workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("points", [256, 300])
@pytest.mark.parametrize("sets", [40, 130])
def test_stale_workspace_reaches_no_result(prec, points, sets):
    import paper_2409_19156_amd as zp

    n, m = W.ansi_modes(12)  # 91 modes, padded to 128
    gen = torch.Generator(device="cuda").manual_seed(7)

    def rand(*shape):
        return torch.rand(*shape, dtype=torch.float64, device="cuda", generator=gen)

    r, th, ur, ut, w = rand(points), 6.28 * rand(points), rand(points), rand(points), rand(points)
    c, uc, g = rand(n.size, sets) - 0.5, rand(n.size, sets) - 0.5, rand(points, sets) - 0.5
    full = zp.series_sizes(n.size, points, sets, prec)[0]

    def run(byte):
        def ws():
            return torch.full((full,), byte, dtype=torch.uint8, device="cuda")

        out = list(zp.series_backward(n, m, r, th, c, g, prec, ws=ws()))
        out += list(zp.series_backward(n, m, r, th, c, g, prec, ws=ws(), need=(True, False, False)))
        torch.empty(64 << 20, dtype=torch.uint8, device="cuda").fill_(byte)  # what the next workspaces start from
        out += list(zp.series_backward2(n, m, r, th, c, g, uc, ur, ut, prec))
        out.append(zp.series_analysis(n, m, r, th, w, g, prec))
        return [x for x in out if x is not None]

    for clean, stale in zip(run(0), run(255)):
        assert torch.isfinite(clean).all() and torch.equal(clean, stale)
