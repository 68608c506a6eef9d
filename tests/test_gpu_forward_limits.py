"""The FP64 forward on both sides of the lines between the fused kernel and the
basis + contraction (sets, and modes from 97 sets on): against the oracle, the
same bits with and without a basis cache, and a gradient through autograd.

Bounds as for the fused kernels: every basis value to 1e-13, doubled for the
contraction's rounding."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import zp_workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [192, 193])
@pytest.mark.parametrize("B", [96, 97, 128, 129])
def test_forward_limits(oracle_mod, M, B):
    import paper_2409_19156_amd as zp

    n, m = (x[:M] for x in W.ansi_modes(19))
    P = 300
    rng = np.random.default_rng([M, B])
    r, th = np.sqrt(rng.random(P)), 2 * np.pi * rng.random(P)
    c, g = rng.standard_normal((M, B)) / (n + 1.0)[:, None], rng.standard_normal((P, B))
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    rd, td, cd, gd = dev(r), dev(th), dev(c), dev(g)
    Z = oracle_mod.basis(n, m, r, th, 1)[0]
    f = zp.series_forward(n, m, rd, td, cd, "fp64")
    assert np.all(np.abs(f.cpu().numpy() - Z.T @ c) <= 2e-13 * np.abs(c).sum(0)[None, :])
    cache = torch.empty(zp.series_sizes(M, P, B, "fp64")[2], dtype=torch.uint8, device="cuda")
    assert torch.equal(zp.series_forward(n, m, rd, td, cd, "fp64", cache=cache), f)
    kept = zp.series_backward(n, m, rd, td, cd, gd, "fp64", cache=cache)
    ca, ra, ta = (x.clone().requires_grad_() for x in (cd, rd, td))
    fa = zp.series(ca, ra, ta, n, m, "fp64")
    assert torch.equal(fa, f)
    for a, b in zip(torch.autograd.grad(fa, (ca, ra, ta), gd), kept):
        assert torch.equal(a, b)
    assert np.all(np.abs(kept[0].cpu().numpy() - Z @ g) <= 2e-13 * np.abs(g).sum(0)[None, :])
