"""The launch shapes of the FP64 series kernels that form the basis inside the
contraction which need many points (two and four point blocks per wave with each
number of set blocks and set steps), and the coefficient gradient of row tiles
whose chains take more recurrence steps than a workgroup keeps in LDS.

Bounds as for the small sizes: an output is a weighted sum of basis values, each
held to 1e-13 (n+1)^(2j) for j r-derivatives and 1e-13 (n+1) for one
theta-derivative, doubled for the contraction's own rounding; a sum over P points
adds P roundings of the sum of absolute terms."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import zp_workloads as W

pytestmark = pytest.mark.gpu


def _modes(name):
    if name == "ansi4":
        return W.ansi_modes(4)
    k = np.arange(0, 251, dtype=np.int32)
    if name == "chain250":  # one chain: tiles begin far up
        return 2 * k + 1, np.where(k % 2, 1, -1).astype(np.int32)
    if name == "sparse":  # a few steep chains in one tile
        a = np.arange(0, 40, dtype=np.int32)
        return (a + 2 * (60 + a)).astype(np.int32), np.where(a % 3, a, -a).astype(np.int32)
    raise KeyError(name)


CASES = [("ansi4", 33000, 1), ("ansi4", 33000, 16), ("ansi4", 17000, 7), ("ansi4", 17000, 16), ("ansi4", 17000, 20),
         ("ansi4", 17000, 40), ("ansi4", 17000, 64), ("ansi4", 9000, 90), ("chain250", 200, 3), ("chain250", 70, 20),
         ("sparse", 200, 3), ("sparse", 70, 20)]


@pytest.mark.parametrize("modes,P,B", CASES)
def test_launch_shapes(oracle_mod, modes, P, B):
    import paper_2409_19156_amd as zp

    n, m = _modes(modes)
    print(f"fused launches: {modes} M={n.size} P={P} B={B}", flush=True)
    rng = np.random.default_rng([P, B, n.size])
    r, th = np.sqrt(rng.random(P)), 2 * np.pi * rng.random(P)
    c, tc = (rng.standard_normal((n.size, B)) / (n + 1.0)[:, None] for _ in range(2))
    g, tr, tt = rng.standard_normal((P, B)), rng.standard_normal(P), rng.standard_normal(P)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    rd, td, cd, gd, ud = dev(r), dev(th), dev(c), dev(g), dev(tc)
    Z, Zr, Zt = oracle_mod.series_basis(n, m, r, th)
    Zrr, Zrt, Ztt = oracle_mod.series_basis2(n, m, r, th)
    t0 = np.full(n.size, 2e-13)
    t1, t2 = 2e-13 * (n + 1.0) ** 2, 2e-13 * (n + 1.0)
    t11, t20 = 2e-13 * (n + 1.0) ** 3, 2e-13 * (n + 1.0) ** 4
    ac, at, ag = np.abs(c), np.abs(tc), np.abs(g)

    def close(got, ref, bound, what):
        got = got.cpu().numpy()
        worst = np.max(np.abs(got - ref) / (bound + 1e-300))
        assert np.all(np.isfinite(got)) and worst <= 1.0, (what, worst)

    close(zp.series_forward(n, m, rd, td, cd, "fp64"), Z.T @ c, (t0 @ ac)[None, :], "f")
    D = tr * Zr + tt * Zt
    tD = np.abs(tr) * t1[:, None] + np.abs(tt) * t2[:, None]
    close(zp.series_jvp(n, m, rd, td, cd, ud, dev(tr), dev(tt), "fp64"), Z.T @ tc + D.T @ c,
          (t0 @ at)[None, :] + tD.T @ ac, "tf")
    gc, gr, gt = zp.series_backward(n, m, rd, td, cd, gd, "fp64")
    dot = lambda d, x: (g * (d.T @ x)).sum(1)  # noqa: E731
    close(gr, dot(Zr, c), ag @ (t1 @ ac), "grad_r")
    close(gt, dot(Zt, c), ag @ (t2 @ ac), "grad_theta")
    sums = lambda z: 2.3e-16 * P * (np.abs(z) @ ag)  # noqa: E731
    close(gc, Z @ g, t0[:, None] * ag.sum(0)[None, :] + sums(Z), "grad_c")
    og, oc, orr, ot = zp.series_backward2(n, m, rd, td, cd, gd, ud, dev(tr), dev(tt), "fp64")
    close(og, Z.T @ tc + D.T @ c, (t0 @ at)[None, :] + tD.T @ ac, "out_g")
    close(oc, D @ g, tD @ ag + sums(D), "out_c")
    close(orr, dot(Zr, tc) + dot(tr * Zrr + tt * Zrt, c),
          ag @ (t1 @ at) + np.abs(tr) * (ag @ (t20 @ ac)) + np.abs(tt) * (ag @ (t11 @ ac)), "out_r")
    close(ot, dot(Zt, tc) + dot(tr * Zrt + tt * Ztt, c),
          ag @ (t2 @ at) + np.abs(tr) * (ag @ (t11 @ ac)) + np.abs(tt) * (ag @ (t1 @ ac)), "out_t")
