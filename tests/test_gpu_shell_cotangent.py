"""Cotangent of the P(k) loss on large meshes.  P_b is quadratic in the density, so its derivative
along v is (P_b(d + v) - P_b(d - v)) / 2 without a differencing error, and the loss's is
Sum_b dL/dP_b times that."""
import numpy as np
import pytest
import torch

from gpu_util import context

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nb", [(256, 5), (256, 128), (512, 512), (1024, 300)])
def test_directional_derivative(n, nb):
    pm = context(8, n, 30.0, 1)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    d = torch.randn((n, n, n), generator=gen, device="cuda")
    p = pm.power_spectrum(d, nb)[1]
    used = np.isfinite(p)   # shells beyond the corner of the mesh hold no modes
    target = np.where(used, p * np.linspace(0.6, 1.5, nb), 0.0)
    weight = 0.7
    _, g = pm.loss_pk(d, target, nb, weight=weight)
    slope = np.zeros(nb)   # dL/dP_b
    slope[used] = weight * 2.0 * (p[used] / target[used] - 1.0) / target[used] / used.sum()
    for kind in ("all", "half"):
        v = d.clone()
        if kind == "half":
            v[:, :n // 2] = 0.0
        got = float((g.double() * v).sum())
        up, down = pm.power_spectrum(d + v, nb)[1], pm.power_spectrum(d - v, nb)[1]
        want = 0.5 * np.sum(slope[used] * (up - down)[used])
        # 32-bit transforms: log2(n^3) 2^-24 = 1.8e-6 of each amplitude, twice in |d_k|^2, in each
        # of the two spectra, once more in the cotangent: 1e-5 of the terms' absolute sum
        size = 0.5 * np.sum(np.abs(slope[used]) * (up + down)[used])
        assert abs(got - want) < 1e-5 * size, (kind, got, want, size)
