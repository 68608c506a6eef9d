"""zp_series_fwd_noalloc keeps its tables in place while the mode list stays the
same, whatever the sizes of the calls: captured calls replay to the eager
result's bits with other calls in between, and a call of another size can be
captured after the first.

The list has every order to |m| = 1000 at its largest degree (the longest
recurrence tables there are), the large call nearly fills the array.  Both
forwards sum in the same order, so the results are identical.
"""
from __future__ import annotations

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _list():
    m = np.arange(1001, dtype=np.int32)
    return (1000 - (1000 - m) % 2).astype(np.int32), m


def test_tables_stay_in_place():
    import paper_2409_19156_amd as zp
    from paper_2409_19156_amd import _lib

    lib = _lib.load()
    n, m = _list()
    gen = torch.Generator(device="cuda").manual_seed(5)

    def case(P, B):
        r = torch.sqrt(torch.rand(P, dtype=torch.float64, device="cuda", generator=gen))
        th = 6.0 * torch.rand(P, dtype=torch.float64, device="cuda", generator=gen)
        c = torch.randn(n.size, B, dtype=torch.float64, device="cuda", generator=gen)
        return r, th, c, zp.series_forward(n, m, r, th, c, "fp64")

    def call(r, th, c, f):
        st = lib.zp_series_fwd_noalloc(n.ctypes.data, m.ctypes.data, n.size, r.data_ptr(), th.data_ptr(), r.numel(),
                                       c.data_ptr(), c.shape[1], 0, f.data_ptr(),
                                       torch.cuda.current_stream().cuda_stream)
        assert st == 0, lib.zp_last_error()

    small, large = case(300, 3), case(200, 5000)
    graphs = []
    out = torch.empty_like(small[3])
    call(*small[:3], out)  # the list's tables go to the device
    torch.cuda.synchronize()
    assert torch.equal(out, small[3])
    for x in (small, large):
        f = torch.empty_like(x[3])
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            call(*x[:3], f)
        graphs.append((g, f, x[3]))
    for rep in range(3):
        for x in (large, small):
            out = torch.empty_like(x[3])
            call(*x[:3], out)
            torch.cuda.synchronize()
            assert torch.equal(out, x[3]), rep
        for g, f, ref in graphs:
            f.fill_(float("nan"))
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(f, ref), rep
