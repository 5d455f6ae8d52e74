"""The filter's cotangent on a 1024^3 mesh (786433 table entries, shells of 64 KB of LDS)."""
import numpy as np
import pytest
import torch

from gpu_util import CO, dev, host
from paper_2211_09958_amd import api
from synthetic import mlp_init, white_noise

pytestmark = pytest.mark.gpu

NP, NG = 128, 1024


@pytest.fixture(scope="module")
def pm():
    return api.PMContext(api.make_config(NP, NG, 4.0 * NP, 1, a_stop=3.0 / 64, filter=True), CO)


def run(pm, theta):
    pm.set_filter(dev(theta))
    disp, mom, _ = pm.forward(dev(white_noise(NP, 4)), want_density=False)
    return disp, mom


def test_constant_filter(pm):
    """With a last layer of zero weights f = 1 + b3 scales every force, as the scales of all kicks
    do: dL/db3, the sum over the table, is the sum of their gradients.  32-bit fields: one cell from
    a particle (mass 512) the field is some 200 times that of the displacements and its rounding
    2e-6 of itself, 4e-4 of the signal at one particle and far less on the mean of 2 million."""
    theta = mlp_init(4, zero_last=False)
    theta[4352:] = 0.0
    disp, mom = run(pm, theta)
    g = host(pm.adjoint(g_disp=disp.clone(), g_mom=mom.clone(), want_filter=True)[2])
    steps = pm.step_gradients()
    want = steps[0].sum() + steps[2].sum()
    assert abs(g[4416] / want - 1) < 1e-4


def test_difference(pm):
    """Along the gradient itself: central differences of 0.01 in the weights are off by their square
    times the network's curvature, below 2e-3."""
    theta = 0.5 * mlp_init(5, zero_last=False)
    disp, mom = run(pm, theta)
    gx, gm = disp.clone(), mom.clone()
    g = host(pm.adjoint(g_disp=gx, g_mom=gm, want_filter=True)[2])
    u = 0.01 * g / np.linalg.norm(g)

    def loss(th):
        x, p = run(pm, th)
        return float((gx.double() * x).sum() + (gm.double() * p).sum())

    want = (loss(theta + u) - loss(theta - u)) / 0.02
    assert abs(np.linalg.norm(g) / want - 1) < 2e-3
