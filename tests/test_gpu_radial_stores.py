"""Radial tables on both sides of the lines between plain and non-temporal
stores (size of the table, alignment and length of its columns): every value is
that of a small call on the same points, bit for bit."""
from __future__ import annotations

import pytest
import torch

import zp_workloads as W

pytestmark = pytest.mark.gpu

MIB = 1 << 20


@pytest.mark.parametrize("orders", [0, 1, 2, 3])
@pytest.mark.parametrize("mib,step,odd", [(71, 8, 2), (73, 8, 2), (91, 8, 0), (93, 8, 0), (287, 8, 0), (289, 8, 0),
                                          (1023, 8, 6), (1025, 8, 6), (1501, 32, 0)])
def test_store_kinds(orders, mib, step, odd):
    import paper_2409_19156_amd as zp

    n, m = W.ansi_modes(30)
    n, m = n[m >= 0], m[m >= 0]
    P = mib * MIB // (8 * n.size * (orders + 1)) // step * step + odd
    gen = torch.Generator(device="cuda").manual_seed(mib)
    r = torch.rand(P, dtype=torch.float64, device="cuda", generator=gen)
    out = torch.full((orders + 1, n.size, P), float("nan"), dtype=torch.float64, device="cuda")
    zp.radial(n, m, r, orders, out=out)
    assert not torch.isnan(out).any()
    for lo in (0, P // 2, P - 700):
        assert torch.equal(out[:, :, lo:lo + 700], zp.radial(n, m, r[lo:lo + 700].clone(), orders)), lo
