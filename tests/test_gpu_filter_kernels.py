"""The filter network's table and backward kernels at table lengths around their 64-entry chunks and
over several chunks per work-group (3 (n/2)^2 + 1 = 49, 193, 769, 12289, 196609 entries), against
the FP64 oracle."""
import numpy as np
import pytest

from gpu_util import context, dev, host, rel_l2
from oracle import mlp as omlp
from oracle import pm as opm
from synthetic import Cosmology, mlp_init, normal

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [8, 16, 32, 128, 512])
def test_table(n):
    theta = mlp_init(4, zero_last=False)
    pm = context(8, n, 50.0, 1, filter=True)
    pm.set_filter(dev(theta))
    for a in (0.02, 0.7):
        want, _ = omlp.filter_table(theta, n, 50.0, a)
        # 64-term sums of terms up to ~1 in 32 bits: 64 x 2^-24 relative to the largest value
        assert np.abs(host(pm.filter_table(a)) - want).max() < 4e-6 * np.abs(want).max()


@pytest.mark.parametrize("np_,ng", [(8, 8), (8, 16), (16, 32), (32, 128)])
def test_weight_gradient(np_, ng):
    """One step in the linear regime (no node-plane crossings): the gradient of a seeded linear
    functional of the final displacements.  32-bit transforms and sums over the table: 2e-5.

    Not at 8 cells per spacing (8^3 particles on 64^3): the functional cancels so far there that the
    rounding of the momenta to their fixed-point unit alone, 1.8e-5 of the displacements, moves the
    gradient by 6e-5, whichever kernel computes it."""
    box = 4.0 * ng
    theta = mlp_init(5, zero_last=False)
    noise, gd = normal((np_,) * 3, 6), normal((np_ ** 3, 3), 7)
    st = opm.Setup(np_, ng, box, 1, Cosmology())
    st.a_stop = 3.0 / 64
    ref = opm.adjoint(opm.forward(noise, st, theta), noise, g_disp=gd)
    from paper_2211_09958_amd import api
    pm = api.PMContext(api.make_config(np_, ng, box, 1, a_stop=3.0 / 64, filter=True), Cosmology())
    pm.set_filter(dev(theta))
    pm.forward(dev(noise))
    g_noise, _, g_filter = pm.adjoint(g_disp=dev(gd), want_filter=True)
    assert rel_l2(host(g_noise), ref.noise) < 2e-5
    assert rel_l2(host(g_filter), ref.theta) < 2e-5


def test_run_over_several_table_batches():
    """41 force evaluations: their tables and cotangents come in batches of 32 and 9.  Each step may
    add the 2e-5 of one (above), so 41 x 2e-5 < 1e-3 for the run."""
    np_, ng, steps = 8, 16, 40
    theta = mlp_init(8, zero_last=False)
    noise, gd = normal((np_,) * 3, 9), normal((np_ ** 3, 3), 10)
    st = opm.Setup(np_, ng, 4.0 * ng, steps, Cosmology())
    st.a_stop = 0.5
    run = opm.forward(noise, st, theta)
    ref = opm.adjoint(run, noise, g_disp=gd)
    from paper_2211_09958_amd import api
    pm = api.PMContext(api.make_config(np_, ng, 4.0 * ng, steps, a_stop=0.5, filter=True), Cosmology())
    pm.set_filter(dev(theta))
    disp, _, _ = pm.forward(dev(noise))
    g_noise, _, g_filter = pm.adjoint(g_disp=dev(gd), want_filter=True)
    assert rel_l2(host(disp), run.disp[-1]) < 1e-3
    assert rel_l2(host(g_noise), ref.noise) < 1e-3
    assert rel_l2(host(g_filter), ref.theta) < 1e-3
