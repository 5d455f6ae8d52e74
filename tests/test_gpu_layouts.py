"""Transforms between callers' arrays and the workspace layout: the first and last FFT passes read
and write plain [n]^3 meshes and [n][n][n/2+1] half spectra of any 4-byte alignment, against FP64
transforms.  An n^3 transform in 32 bits rounds at most log2(n^3) times per value, each by 2^-24
relative to the result's RMS: the bars are log2(n^3) 2^-24."""
import math

import numpy as np
import pytest
import torch

from gpu_util import context, dev, host, rel_l2
from synthetic import normal

pytestmark = pytest.mark.gpu


def shifted(x, words):
    """A contiguous copy of x that starts `words` 32-bit words into its allocation."""
    y = torch.empty(x.numel() + 8, dtype=torch.float32, device="cuda")[words:words + x.numel()]
    y.copy_(x.reshape(-1))
    return y.view(x.shape)


@pytest.mark.parametrize("n", [8, 16, 32, 128, 256])
@pytest.mark.parametrize("words", [0, 1, 2])
def test_transforms_of_callers_arrays(n, words):
    pm = context(8, n, 10.0, 1)
    bar = math.log2(n ** 3) * 2.0 ** -24
    x = dev(normal((n, n, n), 3))
    want = np.fft.rfftn(host(x))
    spec = pm.fft_r2c(shifted(x, words))
    assert rel_l2(torch.view_as_real(spec).double().cpu().numpy(),
                  np.stack([want.real, want.imag], -1)) < bar
    sp = torch.as_tensor(np.fft.rfftn(normal((n, n, n), 4)).astype(np.complex64), device="cuda")
    back = np.fft.irfftn(sp.cpu().numpy().astype(np.complex128), s=(n, n, n), axes=(0, 1, 2))
    assert rel_l2(host(pm.fft_c2r(sp)), back * float(n) ** 3) < bar


@pytest.mark.parametrize("words", [1, 3])
def test_misaligned_meshes_give_the_same_bits(words):
    """Noise in, density in, density cotangent out and noise gradient out through views that are
    only 4-byte aligned: the same bits as aligned arrays."""
    pm = context(16, 32, 40.0, 2)
    noise = dev(normal((16, 16, 16), 5))
    outs = []
    for w in (0, words):
        disp, mom, dens = pm.forward(shifted(noise, w))
        _, g = pm.loss_mse(dens, dev(normal((32, 32, 32), 6)))
        g_noise, _, _ = pm.adjoint(g_dens=shifted(g, w))
        loss, gp = pm.loss_pk(shifted(dens, w), np.full(16, 3.0), 16)
        outs.append((disp, mom, dens, g_noise, gp))
    for name, a, b in zip(("disp", "mom", "dens", "g_noise"), *outs):
        assert torch.equal(a, b), name
    # the shell sums behind the P(k) cotangent add in an order that varies (FP64)
    assert rel_l2(host(outs[1][4]), host(outs[0][4])) < 1e-6
