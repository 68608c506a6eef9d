"""The Fourier kernels of the three-dimensional series at the edges of their
tiles: planes around the 64 lanes of a wave and the 256-plane LDS tile, modes
per pair and in all around the four waves and the partial-sum rows, one and
several sets, large |l|.  Against the oracle, relative to the largest entry,
at the 1e-12 the FP64 series is held to (tests/test_gpu_series3d.py)."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import zp_workloads as W

pytestmark = pytest.mark.gpu


def _rel(got, ref):
    got = got.cpu().numpy()
    assert got.shape == ref.shape and np.all(np.isfinite(got))
    return float(np.abs(got - ref).max() / max(np.abs(ref).max(), 1e-300))


@pytest.mark.parametrize("J,Q,B,lmax", [(1, 1, 1, 0), (2, 63, 1, 3), (3, 64, 2, 1), (33, 65, 1, 4), (200, 257, 1, 16),
                                        (40, 300, 3, 1000), (900, 7, 1, 40), (5, 520, 1, 1 << 20)])
def test_mix_unmix_and_phi_gradient(oracle_mod, J, Q, B, lmax):
    import paper_2409_19156_amd as zp

    print(f"fourier kernels: J={J} Q={Q} B={B} lmax={lmax}", flush=True)
    rng = np.random.default_rng([J, Q, B])
    n2, m2 = W.ansi_modes(3)
    pick = rng.integers(0, n2.size, J)
    n, m, l = n2[pick], m2[pick], rng.integers(-lmax, lmax + 1, J).astype(np.int32)
    P = 20
    r, th = W.disc_points(J + Q, P)
    phi = 2 * np.pi * rng.random(Q)
    c, g = rng.standard_normal((J, B)), rng.standard_normal((P, Q, B))
    Z, Zr, Zt = oracle_mod.series_basis(n, m, r, th)
    F, dF = oracle_mod.fourier(l, phi), oracle_mod.fourier(l, phi, 1)
    ref = (oracle_mod.series3d_fwd(Z, F, c), *oracle_mod.series3d_bwd(Z, Zr, Zt, F, dF, c, g))
    d = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (r, th, phi, c, g)]
    got = (zp.series3d_forward(n, m, l, *d[:4], "fp64"), *zp.series3d_backward(n, m, l, *d, "fp64"))
    for name, a, b in zip(("f", "grad_c", "grad_r", "grad_theta", "grad_phi"), got, ref):
        e = _rel(a, b)
        print(f"  {name}: {e:.2e}", flush=True)
        assert e <= 1e-12, (name, e)
