"""The binding's shortcuts: the current stream and device with and without
torch's private functions, and gradients without a graph node only where nothing differentiates
them (a tangent on what the backward reads is refused, not dropped)."""
from __future__ import annotations

import pytest
import torch
from torch.autograd import forward_ad

import zp_workloads as W

pytestmark = pytest.mark.gpu


def _case():
    import paper_2409_19156_amd as zp

    n, m = W.ansi_modes(6)
    gen = torch.Generator(device="cuda").manual_seed(1)
    rand = lambda *s: torch.rand(*s, dtype=torch.float64, device="cuda", generator=gen)  # noqa: E731
    return zp, n, m, rand(n.size, 3), rand(50), rand(50), rand(50, 3)


@pytest.mark.parametrize("raw", [True, False])
def test_current_stream(monkeypatch, raw):
    zp, n, m, c, r, th, _ = _case()
    if not raw:
        monkeypatch.setattr(zp, "_raw_stream", None)
        monkeypatch.setattr(zp, "_current_device", torch.cuda.current_device)
    ref = zp.series_forward(n, m, r, th, c)
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        assert zp._stream(r.device) == s.cuda_stream
        f = zp.series_forward(n, m, r, th, c)
    s.synchronize()
    assert torch.equal(f, ref)


@pytest.mark.parametrize("which", ["g", "r"])
def test_tangents_are_not_dropped(which):
    zp, n, m, c, r, th, g = _case()
    with forward_ad.dual_level():
        c.requires_grad_()
        rr = forward_ad.make_dual(r, torch.ones_like(r)) if which == "r" else r
        f = zp.series(c, rr, th, n, m, "fp64")
        gg = forward_ad.make_dual(g, torch.ones_like(g)) if which == "g" else g
        with pytest.raises((RuntimeError, NotImplementedError)):
            torch.autograd.grad(f, c, gg)
        f = zp.series(c, r, th, n, m, "fp64")  # no tangent anywhere: as outside the level
        (gc,) = torch.autograd.grad(f, c, g)
    assert torch.equal(gc, zp.series_backward(n, m, r, th, c.detach(), g, need=(True, False, False))[0])
