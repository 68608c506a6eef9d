"""Tables of more points than one launch has work items (2^32): the values past
the first launch's are those of a small call on the same points, bit for bit."""
from __future__ import annotations

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

P = (1 << 32) + 301
ONE = np.array([1], np.int32)


@pytest.fixture(scope="module")
def zp():
    import paper_2409_19156_amd as zp

    assert torch.cuda.is_available()
    yield zp
    torch.cuda.empty_cache()


def _rand(n, seed):
    return torch.rand(n, dtype=torch.float64, device="cuda", generator=torch.Generator(device="cuda").manual_seed(seed))


def test_point_lists(zp):
    r, th = _rand(P, 1), _rand(P, 2)
    where = [slice(0, 70), slice((1 << 32) - 300, P)]
    calls = {"radial": lambda w: zp.radial(ONE, ONE, r[w].clone()), "basis": lambda w: zp.basis(ONE, ONE, r[w].clone(), th[w].clone()),
             "direct": lambda w: zp.radial_direct(ONE, ONE, r[w].clone()),
             "recursion": lambda w: zp.radial_zernike_recursion(ONE, ONE, r[w].clone())}
    full = {"radial": lambda: zp.radial(ONE, ONE, r), "basis": lambda: zp.basis(ONE, ONE, r, th),
            "direct": lambda: zp.radial_direct(ONE, ONE, r), "recursion": lambda: zp.radial_zernike_recursion(ONE, ONE, r)}
    for name, call in full.items():
        out = call()
        for w in where:
            assert torch.equal(out[:, :, w], calls[name](w)), (name, w)
        del out


def test_polar_grid(zp):
    nr = nt = 65537
    r, th = _rand(nr, 3), _rand(nt, 4)
    out = zp.basis_polar(ONE, ONE, r, th).view(nr, nt)
    for i in (0, 65534, 65535, 65536):
        assert torch.equal(out[i], zp.basis_polar(ONE, ONE, r[i:i + 1].clone(), th)[0, 0]), i


def test_fill(zp):
    out = torch.zeros((1 << 33) + 3, dtype=torch.float64, device="cuda")
    zp.stream_fill(out, 2.0)
    assert out.min().item() == 2.0 == out.max().item()
