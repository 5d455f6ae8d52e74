"""Half spectra in and out and real meshes out that are only 4-byte aligned: the same bits as
aligned ones, nothing written beside them."""
import ctypes

import numpy as np
import pytest
import torch

from gpu_util import context, dev
from synthetic import normal

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [8, 16, 32, 64, 128, 256, 512])
@pytest.mark.parametrize("words", [1, 2, 3])
def test_transforms(n, words):
    pm = context(8, n, 10.0, 1)
    real = dev(normal((n, n, n), 3))
    spec = torch.view_as_real(pm.fft_r2c(real)).reshape(-1)
    back = pm.fft_c2r(torch.view_as_complex(spec.view(n, n, n // 2 + 1, 2)))
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())

    def buffer(size):
        whole = torch.full((size + 8,), 7.0, dtype=torch.float32, device="cuda")
        return whole, whole[words:words + size]

    whole, out = buffer(spec.numel())
    assert pm.lib.pm_fft_r2c(pm.ctx, ptr(real), ptr(out)) == 0
    assert torch.equal(out, spec)
    assert bool((whole[:words] == 7.0).all()) and bool((whole[words + out.numel():] == 7.0).all())
    whole, res = buffer(n ** 3)
    assert pm.lib.pm_fft_c2r(pm.ctx, ptr(out), ptr(res)) == 0
    assert torch.equal(res, back.reshape(-1))
    assert bool((whole[:words] == 7.0).all()) and bool((whole[words + res.numel():] == 7.0).all())
