"""The FP64 series kernels that form the basis inside the contraction, against
the oracle, at the sizes where their tiles, windows and mode tables have edges:
point and set counts around the 16-wide tiles and the launch shapes, degrees
beyond the 32-step table window, chains of unequal length, sin-only and
cos-only lists, missing and repeated modes.

Bounds, per output element: every basis value is held to 1e-13 (n+1)^(2j) for
j r-derivatives and 1e-13 (n+1) for one theta-derivative (tests/gpu_util.py);
an output is a weighted sum of basis values, so its error is at most the same
sum with absolute weights and these bounds, doubled for the contraction's own
rounding (at most (M + B) 1.1e-16 of the sum of absolute terms).
"""
from __future__ import annotations

import numpy as np
import pytest
import torch

import zp_workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def zp():
    import paper_2409_19156_amd as zp

    assert torch.cuda.is_available()
    return zp


def _mode_list(name):
    n, m = W.ansi_modes(12)
    if name == "ansi12":
        return n, m
    if name == "one":
        return np.array([3], np.int32), np.array([-1], np.int32)
    if name == "cos":  # m >= 0 only
        return n[m >= 0], m[m >= 0]
    if name == "sin":
        return n[m < 0], m[m < 0]
    if name == "repeated":  # repeated, unsorted columns
        idx = np.random.default_rng(3).integers(0, n.size, 150)
        return n[idx], m[idx]
    if name == "sparse":  # few orders far apart, unequal chain lengths
        return (np.array([70, 5, 66, 90, 64, 2, 40, 75], np.int32),
                np.array([0, 5, -2, 40, 64, 0, -40, 1], np.int32))
    if name == "long":  # one chain past several windows of steps
        k = np.arange(0, 151, dtype=np.int32)
        return 2 * k + 1, np.where(k % 2, 1, -1).astype(np.int32)
    raise KeyError(name)


CASES = [  # modes, points, sets
    ("ansi12", 1, 1), ("ansi12", 15, 2), ("ansi12", 16, 15), ("ansi12", 17, 16), ("ansi12", 33, 17),
    ("ansi12", 65, 33), ("ansi12", 129, 49), ("ansi12", 40, 64), ("ansi12", 70, 65), ("ansi12", 50, 97),
    ("ansi12", 20, 128), ("ansi12", 31, 129), ("ansi12", 20000, 3), ("ansi12", 9000, 40),
    ("one", 5, 3), ("cos", 100, 5), ("sin", 100, 5), ("repeated", 77, 7), ("sparse", 130, 9), ("long", 90, 4),
]


def _case(modes, P, B):
    n, m = _mode_list(modes)
    rng = np.random.default_rng([P, B, n.size])
    r = np.sqrt(rng.random(P))
    r[: min(P, 2)] = [0.0, 1.0][: min(P, 2)]
    th = 2 * np.pi * rng.random(P)
    c = rng.standard_normal((n.size, B)) / (n + 1.0)[:, None]
    return rng, n, m, r, th, c


def _dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float64)).cuda()


def _close(got, ref, bound, what):
    got = got.cpu().numpy()
    assert got.shape == ref.shape and np.all(np.isfinite(got)), what
    worst = np.max(np.abs(got - ref) / bound)
    print(f"  {what}: {worst:.3g} of the bound", flush=True)
    assert worst <= 1.0, (what, worst)


@pytest.mark.parametrize("modes,P,B", CASES)
def test_forward_and_forward_mode(zp, oracle_mod, modes, P, B):
    rng, n, m, r, th, c = _case(modes, P, B)
    print(f"fused forward: {modes} M={n.size} P={P} B={B}", flush=True)
    Z, Zr, Zt = oracle_mod.series_basis(n, m, r, th)
    t0, t1, t2 = 2e-13, 2e-13 * (n + 1.0) ** 2, 2e-13 * (n + 1.0)
    f = zp.series_forward(n, m, _dev(r), _dev(th), _dev(c), "fp64")
    _close(f, Z.T @ c, t0 * np.abs(c).sum(0)[None, :] + 1e-300, "f")
    tc = rng.standard_normal(c.shape) / (n + 1.0)[:, None]
    tr, tt = rng.standard_normal(P), rng.standard_normal(P)
    for use_c, use_r, use_t in ((1, 1, 1), (0, 1, 0), (0, 0, 1), (1, 0, 0)):
        ref = use_c * (Z.T @ tc) + use_r * tr[:, None] * (Zr.T @ c) + use_t * tt[:, None] * (Zt.T @ c)
        bound = (use_c * t0 * np.abs(tc).sum(0)[None, :] + use_r * np.abs(tr)[:, None] * (t1 @ np.abs(c))[None, :]
                 + use_t * np.abs(tt)[:, None] * (t2 @ np.abs(c))[None, :] + 1e-300)
        tf = zp.series_jvp(n, m, _dev(r), _dev(th), _dev(c), _dev(tc) if use_c else None,
                           _dev(tr) if use_r else None, _dev(tt) if use_t else None, "fp64")
        _close(tf, ref, bound, f"tf {use_c}{use_r}{use_t}")


@pytest.mark.parametrize("modes,P,B", CASES)
def test_backward_and_second_order(zp, oracle_mod, modes, P, B):
    rng, n, m, r, th, c = _case(modes, P, B)
    print(f"fused backward: {modes} M={n.size} P={P} B={B}", flush=True)
    g = rng.standard_normal((P, B))
    Z, Zr, Zt = oracle_mod.series_basis(n, m, r, th)
    Zrr = oracle_mod.basis(n, m, r, th, 4)[0]
    a = np.abs(m).astype(np.float64)[:, None]
    R1 = oracle_mod.radial(n, m, r, 1)[1]
    Zrt = np.where(m[:, None] >= 0, -a * np.sin(a * th), a * np.cos(a * th)) * R1
    Ztt = -a * a * Z
    t0, t1, t2 = 2e-13 + 0 * n, 2e-13 * (n + 1.0) ** 2, 2e-13 * (n + 1.0)
    t11, t20, t02 = 2e-13 * (n + 1.0) ** 3, 2e-13 * (n + 1.0) ** 4, 2e-13 * (n + 1.0) ** 2
    ag, ac = np.abs(g), np.abs(c)
    dot = lambda d, x: (g * (d.T @ x)).sum(1)  # noqa: E731
    bnd = lambda t, x: ag @ (t @ np.abs(x)) + 1e-300  # noqa: E731
    gc, gr, gt = zp.series_backward(n, m, _dev(r), _dev(th), _dev(c), _dev(g), "fp64")
    _close(gr, dot(Zr, c), bnd(t1, c), "grad_r")
    _close(gt, dot(Zt, c), bnd(t2, c), "grad_theta")
    _close(gc, Z @ g, t0[:, None] * ag.sum(0)[None, :] + 1e-300, "grad_c")
    uc = rng.standard_normal(c.shape) / (n + 1.0)[:, None]
    ur, ut = rng.standard_normal(P), rng.standard_normal(P)
    for wc, wr, wt in ((1, 1, 1), (1, 0, 0), (0, 1, 0), (0, 0, 1)):
        D = wr * ur * Zr + wt * ut * Zt
        tD = wr * np.abs(ur) * t1[:, None] + wt * np.abs(ut) * t2[:, None]  # [M, P]
        og, oc, orr, ot = zp.series_backward2(n, m, _dev(r), _dev(th), _dev(c), _dev(g), _dev(uc) if wc else None,
                                              _dev(ur) if wr else None, _dev(ut) if wt else None, "fp64")
        what = f"{wc}{wr}{wt}"
        _close(orr, wc * dot(Zr, uc) + dot(wr * ur * Zrr + wt * ut * Zrt, c),
               wc * bnd(t1, uc) + wr * np.abs(ur) * bnd(t20, c) + wt * np.abs(ut) * bnd(t11, c), "out_r " + what)
        _close(ot, wc * dot(Zt, uc) + dot(wr * ur * Zrt + wt * ut * Ztt, c),
               wc * bnd(t2, uc) + wr * np.abs(ur) * bnd(t11, c) + wt * np.abs(ut) * bnd(t02, c), "out_t " + what)
        _close(oc, D @ g, tD @ ag + 1e-300, "out_c " + what)
        _close(og, wc * (Z.T @ uc) + D.T @ c, wc * t0[0] * np.abs(uc).sum(0)[None, :] + tD.T @ ac + 1e-300,
               "out_g " + what)


def test_backward_rows_and_smallest_workspace(zp):
    """dL/dr and dL/dtheta of a point do not depend on the other points, and
    with the smallest workspace every gradient is the full workspace's."""
    rng, n, m, r, th, c = _case("ansi12", 3000, 70)
    g = _dev(rng.standard_normal((3000, 70)))
    rd, td, cd = _dev(r), _dev(th), _dev(c)
    gc, gr, gt = zp.series_backward(n, m, rd, td, cd, g, "fp64")
    for P in (1, 31, 700):
        _, a, b = zp.series_backward(n, m, rd[:P], td[:P], cd, g[:P], "fp64")
        assert torch.equal(a, gr[:P]) and torch.equal(b, gt[:P]), P
    _, mn, _ = zp.series_sizes(n.size, 3000, 70, "fp64")
    ws = torch.empty(mn, dtype=torch.uint8, device="cuda")
    gc2, gr2, gt2 = zp.series_backward(n, m, rd, td, cd, g, "fp64", ws=ws)
    assert torch.equal(gr2, gr) and torch.equal(gt2, gt)
    assert ((gc2 - gc).abs().max() / gc.abs().max()).item() <= 1e-13


def test_forward_rows_and_caches(zp):
    """A point's row does not depend on the other points or on whether the
    basis is kept; NaN and infinite inputs stay in their rows and columns."""
    _, n, m, r, th, c = _case("ansi12", 3000, 24)
    rd, td, cd = _dev(r), _dev(th), _dev(c)
    f = zp.series_forward(n, m, rd, td, cd, "fp64")
    for P in (1, 31, 700):
        assert torch.equal(zp.series_forward(n, m, rd[:P], td[:P], cd, "fp64"), f[:P]), P
    _, _, cb = zp.series_sizes(n.size, 3000, 24, "fp64")
    cache = torch.empty(cb, dtype=torch.uint8, device="cuda")
    assert torch.equal(zp.series_forward(n, m, rd, td, cd, "fp64", cache=cache), f)
    bad = rd.clone()
    bad[5] = float("nan")
    g = zp.series_forward(n, m, bad, td, cd, "fp64")
    keep = torch.ones(3000, dtype=torch.bool, device="cuda")
    keep[5] = False
    assert torch.isnan(g[5]).all() and torch.equal(g[keep], f[keep])
    cbad = cd.clone()
    cbad[7, 3] = float("inf")
    g = zp.series_forward(n, m, rd, td, cbad, "fp64")
    cols = [b for b in range(24) if b != 3]
    assert torch.equal(g[:, cols], f[:, cols]) and not torch.isfinite(g[10:, 3]).any()


def test_angles_outside_one_turn(zp, oracle_mod):
    """theta many turns away: the exact angle of the given double."""
    _, n, m, r, th, c = _case("ansi12", 64, 3)
    far = th + 2 * np.pi * np.repeat([0.0, -1.0, 1e3, 1e6], 16)
    Z = oracle_mod.basis(n, m, r, far, 1)[0]
    f = zp.series_forward(n, m, _dev(r), _dev(far), _dev(c), "fp64")
    _close(f, Z.T @ c, 2e-13 * np.abs(c).sum(0)[None, :], "f")
