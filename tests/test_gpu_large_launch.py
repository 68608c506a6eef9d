"""Calls whose work takes more than one launch's 2^32 work items: the kernels
that give 256 threads to 16 to 64 points, to one row of the upstream gradient, to
64 coefficients or to 256.  (Beyond that a launch leaves work out without an error.)  Rows are compared bit for bit with calls on a few of the points
(a point's row does not depend on the others), coefficients with the closed form
of the one-point case.
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
    yield zp
    torch.cuda.empty_cache()


def test_one_set_on_a_billion_points(zp):
    n, m = W.ansi_modes(1)
    P = (1 << 30) + 37
    gen = torch.Generator(device="cuda").manual_seed(1)
    rand = lambda *s: torch.rand(*s, dtype=torch.float64, device="cuda", generator=gen)  # noqa: E731
    r, th, g, tr = rand(P), rand(P), rand(P, 1), rand(P)
    c, tc = rand(n.size, 1), rand(n.size, 1)
    where = [slice(0, 40), slice((1 << 28) - 20, (1 << 28) + 20), slice((1 << 30) - 40, P)]
    f = zp.series_forward(n, m, r, th, c, "fp64")
    for w in where:
        assert torch.equal(zp.series_forward(n, m, r[w].clone(), th[w].clone(), c, "fp64"), f[w]), w
    del f
    tf = zp.series_jvp(n, m, r, th, c, tc, tr, None, "fp64")
    for w in where:
        part = zp.series_jvp(n, m, r[w].clone(), th[w].clone(), c, tc, tr[w].clone(), None, "fp64")
        assert torch.equal(part, tf[w]), w
    del tf
    gc, gr, gt = zp.series_backward(n, m, r, th, c, g, "fp64")
    for w in where:
        _, a, b = zp.series_backward(n, m, r[w].clone(), th[w].clone(), c, g[w].clone(), "fp64")
        assert torch.equal(a, gr[w]) and torch.equal(b, gt[w]), w
    # dL/dc: Z = 1, r sin, r cos; two sums of 2^30 positive terms are within 2^30 roundings of each other
    ref = torch.stack([g.sum(), (r * torch.sin(th) * g[:, 0]).sum(), (r * torch.cos(th) * g[:, 0]).sum()])
    assert ((gc[:, 0] - ref).abs() <= 2.0 ** -23 * ref.abs()).all()


def test_gradient_of_more_than_2_24_rows(zp):
    n, m = W.ansi_modes(1)
    P = (1 << 24) + 200
    gen = torch.Generator(device="cuda").manual_seed(4)
    rand = lambda *s: torch.rand(*s, dtype=torch.float64, device="cuda", generator=gen)  # noqa: E731
    r, th, g, c = rand(P), rand(P), 0.5 + rand(P, 1), rand(n.size, 1)
    _, gr, gt = zp.series_backward(n, m, r, th, c, g, "fp32")
    for w in (slice(0, 40), slice(P - 250, P)):
        _, a, b = zp.series_backward(n, m, r[w].clone(), th[w].clone(), c, g[w].clone(), "fp32")
        assert torch.equal(a, gr[w]) and torch.equal(b, gt[w]), w


@pytest.mark.parametrize("what", ["backward", "analysis"])
def test_more_than_2_32_coefficients(zp, what):
    n, m = W.ansi_modes(64)
    B = (1 << 32) // n.size + 1000
    gen = torch.Generator(device="cuda").manual_seed(2)
    g = 0.5 + torch.rand(1, B, dtype=torch.float64, device="cuda", generator=gen)
    r = torch.tensor([0.7], dtype=torch.float64, device="cuda")
    th = torch.tensor([0.3], dtype=torch.float64, device="cuda")
    z = zp.basis(n, m, r, th)[0, :, 0]
    if what == "backward":
        c = torch.empty(n.size, B, dtype=torch.float64, device="cuda")  # not read
        out = zp.series_backward(n, m, r, th, c, g, "fp32", need=(True, False, False))[0]
        del c
        scale = torch.ones(n.size, dtype=torch.float64, device="cuda")
    else:
        out = zp.series_analysis(n, m, r, th, torch.ones_like(r), g, "fp32")
        scale = torch.from_numpy(np.where(m == 0, 1.0, 2.0) * (n + 1.0) / np.pi).cuda()
    for k in list(range(0, n.size, 97)) + [n.size - 1]:
        # a product of two values rounded to FP32
        assert ((out[k] - z[k] * g[0] * scale[k]).abs() <= 2.0 ** -22 * (z[k] * g[0] * scale[k]).abs()).all(), k


def test_more_than_2_30_unmixed_coefficients(zp):
    n2, m2 = W.ansi_modes(2)
    ls = np.arange(-25, 26, dtype=np.int32)
    n, m, l = np.tile(n2, ls.size), np.tile(m2, ls.size), np.repeat(ls, n2.size)
    B = (1 << 30) // n.size + 1000
    gen = torch.Generator(device="cuda").manual_seed(3)
    g = 0.5 + torch.rand(1, 1, B, dtype=torch.float64, device="cuda", generator=gen)
    one = lambda x: torch.tensor([x], dtype=torch.float64, device="cuda")  # noqa: E731
    r, th, phi = one(0.7), one(0.3), one(0.2)
    c = torch.empty(n.size, B, dtype=torch.float64, device="cuda").zero_()
    out = zp.series3d_backward(n, m, l, r, th, phi, c, g, "fp64", need=(True, False, False, False))[0]
    z = zp.basis(n2, m2, r, th)[0, :, 0].repeat(ls.size)
    F = torch.from_numpy(np.where(l >= 0, np.cos(l * 0.2), np.sin(-l * 0.2))).cuda()
    for j in list(range(0, n.size, 7)) + [n.size - 1]:
        assert ((out[j] - z[j] * F[j] * g[0, 0]).abs() <= 1e-13 * g[0, 0]).all(), j
