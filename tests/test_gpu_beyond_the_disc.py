"""Points beyond the unit disc are evaluated as polynomials, also where a mode's
neighbours in the tables would overflow at degrees that nobody asked for: the
modes (800, 0) and (600, 600) share a group of chains, whose second one would be
infinite at degree 400 and r = 1.3, while both modes and their derivatives are
finite.

The outputs are sums of two products with the oracle's values; the larger is
about 1e261 and rounds by K^2 ulp at most (K = 400 steps of the recurrence,
each within a few ulp of a sum of growing terms)."""
from __future__ import annotations

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_sums_stay_finite(oracle_mod):
    import paper_2409_19156_amd as zp

    n, m = np.array([800, 600], np.int32), np.array([0, 600], np.int32)
    r, th = np.array([1.3, 0.9, 1.3]), np.array([0.4, 1.0, 2.0])
    c, g = np.array([[1.0, 2.0], [0.5, -1.0]]), np.array([[1.0, 0.25], [2.0, 1.0], [0.5, 0.125]])
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    Z, Zr, Zt = oracle_mod.series_basis(n, m, r, th)
    assert np.all(np.isfinite(Zr)) and Zr.max() > 1e260
    args = (n, m, dev(r), dev(th), dev(c), dev(g))

    def close(got, *terms):
        size = sum(np.abs(t) for t in terms)
        assert np.all(np.abs(got.cpu().numpy() - sum(terms)) <= 400 ** 2 * 2.3e-16 * size)

    h = c @ g.T  # [M, P]
    gc, gr, gt = zp.series_backward(*args)
    close(gr, h[0] * Zr[0], h[1] * Zr[1])
    close(gt, h[0] * Zt[0], h[1] * Zt[1])
    _, _, orr, ot = zp.series_backward2(*args, uc=dev(c), ur=dev(np.zeros(3)), ut=dev(np.zeros(3)))
    close(orr, h[0] * Zr[0], h[1] * Zr[1])
    close(ot, h[0] * Zt[0], h[1] * Zt[1])
