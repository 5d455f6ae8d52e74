"""pm_loss_pk with a loss that is not finite: PM_ENUMERIC, the loss returned, and the caller's
cotangent array left as it was."""
import ctypes
import math

import numpy as np
import pytest
import torch

from gpu_util import context, dev
from paper_2211_09958_amd import _lib
from synthetic import normal

pytestmark = pytest.mark.gpu


def loss_pk(pm, d, target, weight, g):
    loss = ctypes.c_double(-1.0)
    rc = pm.lib.pm_loss_pk(pm.ctx, ctypes.c_void_p(d.data_ptr()), target.size,
                           target.ctypes.data_as(ctypes.c_void_p), ctypes.c_double(weight),
                           ctypes.byref(loss), ctypes.c_void_p(g.data_ptr()))
    return rc, loss.value


@pytest.mark.parametrize("n", [8, 64, 128, 256])
def test_cotangent_is_left_alone(n):
    pm = context(8, n, 30.0, 1)
    good = dev(normal((n, n, n), 3))
    target = np.linspace(0.5, 1.5, n // 2)
    g = torch.full((n, n, n), 7.0, dtype=torch.float32, device="cuda")
    for value in (math.nan, math.inf):
        bad = good.clone()
        bad[1, 2, 3] = value
        rc, loss = loss_pk(pm, bad, target, 1.0, g)
        assert rc == _lib.PM_ENUMERIC and not math.isfinite(loss)
        assert bool((g == 7.0).all())
    # and written again by the next call
    rc, loss = loss_pk(pm, good, target, 1.0, g)
    assert rc == 0 and math.isfinite(loss)
    want = pm.loss_pk(good, target, target.size)[1]
    # the shell sums add in an order that varies (FP64)
    assert float((g - want).norm() / want.norm()) < 1e-6


def test_weight_that_overflows_is_no_error():
    """The shells' sum is finite, so the call succeeds and returns the infinite loss."""
    pm = context(8, 16, 30.0, 1)
    g = torch.full((16, 16, 16), 7.0, dtype=torch.float32, device="cuda")
    rc, loss = loss_pk(pm, dev(100.0 * normal((16, 16, 16), 3)), np.full(8, 1e-3), 1e308, g)
    assert rc == 0 and loss == math.inf
    assert not bool((g == 7.0).any())
