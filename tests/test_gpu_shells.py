"""Shell sums taken inside the last transform pass (P(k), with and without a context) and the P(k)
loss's cotangent, at every transform length and at shell counts around the corner of the mesh."""
import numpy as np
import pytest
import torch

from gpu_util import context, dev, host, rel_l2
from oracle import mesh as M
from oracle import pm as opm
from paper_2211_09958_amd import api
from synthetic import normal

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [8, 16, 32, 64, 128])
def test_spectrum(n):
    d = normal((n, n, n), n)
    pm = context(8, n, 30.0, 1)
    for nb in (1, 3, n // 2, round(0.75 ** 0.5 * n), n):
        with np.errstate(invalid="ignore"):
            k, p, m = M.power_spectrum(d, 30.0, nb)
        for got in (pm.power_spectrum(dev(d), nb), api.power_spectrum_noalloc(dev(d), 30.0, nb)):
            assert np.array_equal(got[2], m)
            np.testing.assert_allclose(got[0], k, rtol=1e-12)
            # 32-bit transform: log2(n^3) 2^-24 of the RMS amplitude per mode, twice in |d|^2; a
            # shell of few modes can hold amplitudes well below the RMS
            np.testing.assert_allclose(got[1], p, rtol=2e-5)


@pytest.mark.parametrize("n", [256, 512, 1024])
def test_all_shells_hold_all_modes(n):
    """Counts against integer shells, and Parseval: Sum_b N_b P_b = (L^3 / N^3) Sum delta^2."""
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    d = torch.randn((n, n, n), generator=g, device="cuda")
    d -= d.mean(dtype=torch.float64).float()
    k, p, m = context(8, n, 10.0, 1).power_spectrum(d, n)
    held = m > 0
    assert m.sum() == float(n) ** 3 - 1
    assert np.count_nonzero(held) == round(0.75 ** 0.5 * n) and held[:np.count_nonzero(held)].all()
    total = float(d.double().square().sum()) * 10.0 ** 3 / float(n) ** 3
    assert abs((p[held] * m[held]).sum() / total - 1) < 2e-6
    # mean |k| of a shell is within half a shell of its number
    b = np.arange(1, n + 1)
    assert np.abs(k[held] * 10.0 / (2 * np.pi) - b[held]).max() < 0.5


@pytest.mark.parametrize("n,nb", [(8, 1), (8, 8), (16, 5), (32, 32), (64, 31), (128, 64)])
def test_loss_cotangent(n, nb):
    d = normal((n, n, n), 3)
    pm = context(8, n, 30.0, 1)
    with np.errstate(invalid="ignore"):
        pt = M.power_spectrum(d, 30.0, nb)[1] * np.linspace(0.5, 1.7, nb)
    pt[np.isnan(pt)] = 1.0
    if nb > 4:
        pt[2] = 0.0
        pt[3] = np.inf
    want, g = opm.pk_loss(d, np.where(np.isfinite(pt), pt, 0.0), 30.0, nb, 0.7)
    got, gg = pm.loss_pk(dev(d), pt, nb, weight=0.7)
    assert abs(got / want - 1) < 2e-5
    assert rel_l2(host(gg), g) < 2e-5
    assert abs(pm.loss_pk(dev(d), pt, nb, weight=0.7, want_grad=False)[0] / got - 1) < 1e-9


def test_only_empty_shells_are_refused():
    pm = context(8, 16, 30.0, 1)
    pt = np.zeros(16)
    pt[14:] = 1.0   # round(sqrt(3) 8) = 14 is the last shell with modes
    with pytest.raises(api.PMError):
        pm.loss_pk(dev(normal((16, 16, 16), 3)), pt, 16)
    pt[13] = 1.0
    pm.loss_pk(dev(normal((16, 16, 16), 3)), pt, 16)
