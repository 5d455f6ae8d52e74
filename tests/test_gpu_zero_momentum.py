"""pm_adjoint without a momentum cotangent (its first reverse step needs no force transpose) against
the same call with explicit zeros."""
import numpy as np
import pytest
import torch

from gpu_util import context, dev
from synthetic import mlp_init, normal

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("np_,ng,steps,ckpt,filt,lpt",
                         [(8, 8, 1, 0, False, 1), (8, 32, 3, 1, False, 2), (16, 32, 2, 0, True, 1),
                          (32, 32, 4, 2, True, 2), (32, 128, 1, 0, False, 1)])
def test_null_equals_zeros(np_, ng, steps, ckpt, filt, lpt):
    pm = context(np_, ng, 4.0 * ng, steps, checkpoint_every=ckpt, filter=filt, lpt_order=lpt)
    if filt:
        pm.set_filter(dev(mlp_init(3, zero_last=False)))
    P = np_ ** 3
    g_dens, g_disp = dev(normal((ng,) * 3, 2)), dev(normal((P, 3), 3))
    pm.forward(dev(normal((np_,) * 3, 1)))
    got = []
    for g_mom in (None, torch.zeros((P, 3), dtype=torch.float32, device="cuda")):
        g_noise, g_cosmo, g_filt = pm.adjoint(g_dens, g_disp, g_mom, want_filter=filt)
        got.append((g_noise, g_cosmo, g_filt, pm.step_gradients(), pm.stats()["ic_max_cells"]))
    a, b = got
    assert torch.equal(a[0], b[0])
    assert a[4] == b[4] == 0.0
    # FP64 sums whose order varies; the filter gradient adds in 32 bits in an order that varies
    scale = np.abs(b[3]).max()
    np.testing.assert_allclose(a[3], b[3], rtol=1e-9, atol=1e-9 * scale)
    np.testing.assert_allclose(a[1], b[1], rtol=1e-7)
    if filt:
        assert float((a[2] - b[2]).norm() / b[2].norm()) < 2e-6


@pytest.mark.parametrize("np_,ng", [(8, 16), (16, 32), (32, 128)])
def test_cotangents_are_taken_where_they_lie(np_, ng):
    """The first sort of the adjoint reads the caller's cotangents: any 4-byte alignment, none for
    zero, left as they were.  The noise gradient repeats bit for bit."""
    pm = context(np_, ng, 2.5 * np_, 3)
    n = np_ ** 3
    noise, gd = dev(normal((np_,) * 3, 5)), dev(normal((ng,) * 3, 6))
    gx, gp = dev(normal((n, 3), 7)), dev(normal((n, 3), 8))

    def shifted(t):
        buf = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
        view = buf[1:].view(t.shape)
        view.copy_(t)
        return view

    def run(**g):
        pm.forward(noise)
        return pm.adjoint(**g)[0].clone()

    ax, ap = shifted(gx), shifted(gp)
    assert torch.equal(run(g_dens=gd, g_disp=gx, g_mom=gp), run(g_dens=gd, g_disp=ax, g_mom=ap))
    assert torch.equal(ax, gx) and torch.equal(ap, gp)
    zero = torch.zeros_like(gx)
    assert torch.equal(run(g_dens=gd, g_mom=gp), run(g_dens=gd, g_disp=zero, g_mom=gp))
    assert torch.equal(run(g_mom=gp), run(g_disp=zero, g_mom=gp))
