"""Particles so many that the gathers that read the meshes themselves take more than one chunk of
them per work-group (above 2^21: 256^3 on 1024^3), against FP64 transforms on the GPU and against
differences of whole runs."""
import numpy as np
import pytest
import torch

from gpu_util import CO, dev
from paper_2211_09958_amd import api
from synthetic import white_noise

pytestmark = pytest.mark.gpu

NP, NG = 256, 1024
BOX = float(NG)   # cells of 1


class Cic:
    """FP64 cloud-in-cell weights of positions x [P, 3] in cells of 1."""

    def __init__(self, x):
        u = x - 0.5
        fl = torch.floor(u)
        self.t = u - fl
        self.i = torch.remainder(fl.long(), NG)

    def corners(self):
        for c in np.ndindex(2, 2, 2):
            j = [(self.i[:, a] + c[a]) % NG for a in range(3)]
            w = [self.t[:, a] if c[a] else 1.0 - self.t[:, a] for a in range(3)]
            sign = [1.0 if c[a] else -1.0 for a in range(3)]
            yield (j[0] * NG + j[1]) * NG + j[2], w, sign

    def scatter(self, values):
        out = torch.zeros(NG ** 3, dtype=torch.float64, device="cuda")
        for flat, w, _ in self.corners():
            out.index_add_(0, flat, w[0] * w[1] * w[2] * values)
        return out.view(NG, NG, NG)

    def gather(self, field):
        """The field and its gradient at the particles."""
        f, g = 0.0, [0.0, 0.0, 0.0]
        for flat, w, s in self.corners():
            v = field.reshape(-1)[flat]
            f = f + w[0] * w[1] * w[2] * v
            g[0] = g[0] + s[0] * w[1] * w[2] * v
            g[1] = g[1] + w[0] * s[1] * w[2] * v
            g[2] = g[2] + w[0] * w[1] * s[2] * v
        return f, torch.stack(g, 1)


def multiplier(j):
    """i k_j / k^2, zero at k = 0 and on axis j's Nyquist plane."""
    n = torch.fft.fftfreq(NG, 1.0 / NG, device="cuda", dtype=torch.float64)
    half = torch.arange(NG // 2 + 1, device="cuda", dtype=torch.float64)
    axes = [n[:, None, None], n[None, :, None], half[None, None, :]]
    k2 = axes[0] ** 2 + axes[1] ** 2 + axes[2] ** 2
    k2[0, 0, 0] = 1.0
    kj = torch.where(axes[j].abs() == NG // 2, 0.0, axes[j])
    return torch.complex(torch.zeros_like(k2), kj * (BOX / (2 * np.pi)) / k2)


def rel(a, b):
    return float((a.double() - b).norm() / b.norm())


def test_force_and_vjp():
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    P = NP ** 3
    d = 2.0 * torch.randn((P, 3), generator=gen, device="cuda")
    v = torch.randn((P, 3), generator=gen, device="cuda")
    pm = api.PMContext(api.make_config(NP, NG, BOX, 1), CO)
    force, xi = pm.force(d, 0.5).clone(), pm.force_vjp(d, 0.5, v).clone()
    del pm
    torch.cuda.empty_cache()

    line = torch.arange(NP, device="cuda", dtype=torch.float64) * (BOX / NP)
    q = torch.stack(torch.meshgrid(line, line, line, indexing="ij"), -1).reshape(-1, 3)
    units = torch.round(d * np.float32(2.0 ** 32 / BOX)).double()
    cic = Cic(torch.remainder(q + units * (BOX / 2.0 ** 32), BOX))
    mass = (NG / NP) ** 3
    dk = torch.fft.rfftn(cic.scatter(torch.full((P,), mass, dtype=torch.float64, device="cuda")))
    want, want_xi, bar = [], 0.0, 0.0
    for j in range(3):
        m = multiplier(j)
        f, g = cic.gather(torch.fft.irfftn(m * dk, s=(NG,) * 3))
        want.append(f)
        want_xi = want_xi + v[:, j:j + 1].double() * g
        bar = bar + m.conj() * torch.fft.rfftn(cic.scatter(v[:, j].double()))
        del m
    want_xi = want_xi + mass * cic.gather(torch.fft.irfftn(bar, s=(NG,) * 3))[1]
    # 32-bit transforms: some 2^-24 log2(ng^3) of the field's norm; the VJP takes differences of
    # neighbouring nodes and adds three terms of either sign, ten times that
    assert rel(force, torch.stack(want, 1)) < 1e-5
    assert rel(xi, want_xi) < 1e-4


def test_run_and_adjoint():
    """Exact reconstruction, and the gradients of the step scales (sums over all work-groups)
    against central differences.  The functional is at most quadratic in a kick's or drift's scale up
    to the small response of the forces, so differences of 0.02 are off by far less than 2e-3."""
    pm = api.PMContext(api.make_config(NP, NG, BOX, 2, a_stop=3.0 / 64), CO)
    noise = dev(white_noise(NP, 4))
    disp, mom, _ = pm.forward(noise, want_density=False)
    gx, gm = disp.clone(), mom.clone()
    pm.adjoint(g_disp=gx, g_mom=gm)
    assert pm.stats()["ic_max_cells"] == 0.0 and pm.stats()["ic_mom_rel_rms"] == 0.0
    got = pm.step_gradients().copy()

    def loss(scales):
        pm.set_step_scales(scales)
        x, p, _ = pm.forward(noise, want_density=False)
        return float((gx.double() * x).sum() + (gm.double() * p).sum())

    for k in range(3):
        for n in range(2):
            s = np.ones((3, 2))
            s[k, n] = 1.02
            up = loss(s)
            s[k, n] = 0.98
            want = (up - loss(s)) / 0.04
            assert abs(got[k, n] - want) < 2e-3 * abs(want), (k, n, got[k, n], want)
