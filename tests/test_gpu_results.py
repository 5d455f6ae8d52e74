"""Scalar results that kernels write to pinned host memory: successive calls of different kinds and
sizes on one context, several contexts in turn, and step scales replaced between runs."""
import numpy as np
import pytest
import torch

from gpu_util import CO, dev
from oracle import mesh as M
from oracle import pm as opm
from paper_2211_09958_amd import api
from synthetic import normal

pytestmark = pytest.mark.gpu


def test_results_do_not_mix():
    pms = [api.PMContext(api.make_config(8, ng, 4.0 * ng, 2, a_stop=0.05), CO) for ng in (8, 16, 32)]
    d = [normal((pm.ng,) * 3, 3) for pm in pms]
    t = [normal((pm.ng,) * 3, 4) for pm in pms]
    for _ in range(2):
        for pm, x, y in zip(pms, d, t):
            nb = pm.ng // 2
            k, p, m = pm.power_spectrum(dev(x), nb)
            pk = M.power_spectrum(x, pm.cfg.box, nb)
            np.testing.assert_allclose(p, pk[1], rtol=2e-5)
            np.testing.assert_allclose(k, pk[0], rtol=1e-12)
            loss, _ = pm.loss_mse(dev(x), dev(y))
            assert abs(loss / opm.mse_loss(x, y)[0] - 1) < 1e-6
            lp, _ = pm.loss_pk(dev(x), 1.3 * pk[1], nb)
            assert abs(lp / opm.pk_loss(x, 1.3 * pk[1], pm.cfg.box, nb)[0] - 1) < 1e-4
            s, r = normal((512, 3), 5), normal((512, 3), 6)
            ld, _ = pm.loss_disp(dev(s), dev(r), weight=0.3)
            assert abs(ld / opm.disp_loss(s, r, pm.cfg.box, pm.ng, 0.3)[0] - 1) < 1e-6
            pm.forward(dev(normal((8, 8, 8), 7)))
            a = pm.adjoint(g_dens=dev(y))
            b = pm.adjoint(g_dens=dev(y))
            assert torch.equal(a[0], b[0])
            np.testing.assert_allclose(a[1], b[1], rtol=1e-9)


def test_replaced_step_scales_start_from_the_unscaled_schedule():
    pm = api.PMContext(api.make_config(8, 16, 64.0, 3, a_stop=0.05), CO)
    noise = dev(normal((8, 8, 8), 1))
    plain = pm.forward(noise)[0].clone()
    pm.set_step_scales(np.full((3, 3), 1.7))
    assert not torch.equal(pm.forward(noise)[0], plain)
    pm.set_step_scales(np.ones((3, 3)))
    assert torch.equal(pm.forward(noise)[0], plain)
