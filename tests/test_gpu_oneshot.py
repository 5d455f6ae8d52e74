"""Density, force and force VJP of a caller's displacements: binned once, records in lattice order,
outputs by storage slot."""
import ctypes

import numpy as np
import pytest
import torch

from gpu_util import context, dev, host
from oracle import mesh as M
from oracle import pm as opm
from synthetic import Cosmology, normal

pytestmark = pytest.mark.gpu


def disps(np_, box):
    """All particles of a wave in few bins, in many bins, and a pile in one cell."""
    n = np_ ** 3
    q = opm.lattice(np_, box)
    smooth = 0.3 * box / np_ * normal((n, 3), 1)
    spread = box * normal((n, 3), 2)
    pile = box * 0.37 - q + 1e-3 * box / np_ * normal((n, 3), 3)
    return {"smooth": smooth, "spread": spread, "pile": pile}


@pytest.mark.parametrize("np_,ng", [(8, 8), (8, 16), (16, 32), (16, 64), (32, 32), (16, 128),
                                    (32, 256)])
@pytest.mark.parametrize("kind", ["smooth", "spread", "pile"])
def test_density_into_any_alignment(np_, ng, kind):
    box = 50.0
    pm = context(np_, ng, box, 1)
    d = dev(disps(np_, box)[kind])
    out = torch.full((ng ** 3 + 8,), np.nan, dtype=torch.float32, device="cuda")
    got = []
    for words in (0, 1):
        view = out[words:words + ng ** 3]
        rc = pm.lib.pm_density(pm.ctx, ctypes.c_void_p(d.data_ptr()),
                               ctypes.c_void_p(view.data_ptr()))
        assert rc == 0
        got.append(view.clone())
    assert torch.equal(got[0], got[1])
    # CIC weights of 32-bit positions: 2^-32 box against cells of box / ng, 8 corners of 2^-24
    units = np.rint(host(d).astype(np.float32) * np.float32(2.0 ** 32 / box)).astype(np.float64)
    x = opm.lattice(np_, box) + units * (box / 2.0 ** 32)
    want = M.density(x, ng, box, np_ ** 3)
    assert np.abs(host(got[0]).reshape(want.shape) - want).max() < 1e-6 * max(1.0, want.max())


@pytest.mark.parametrize("np_,ng", [(8, 8), (16, 64), (64, 64), (32, 128)])
def test_one_context_bins_set_after_set(np_, ng):
    """The counts of one sort are cleared for the next, and order and offsets cover every particle:
    from no full work-group to 256 of them, at and beyond the meshes sorted in one launch.  The
    density is a sum of integers, so a used context gives the bits of a new one."""
    box = 50.0
    used = context(np_, ng, box, 1)
    for d in disps(np_, box).values():
        got = used.density(dev(d)).clone()
        assert torch.equal(got, context(np_, ng, box, 1).density(dev(d)))
        assert abs(got.double().sum().item()) < 1e-6 * ng ** 3 * max(1.0, got.max().item())


def test_building_blocks_leave_the_stored_run():
    """Force, VJP and density between pm_forward and pm_adjoint change nothing in the adjoint,
    and a second call gives the same bits as the first."""
    pm = context(16, 32, 40.0, 3)
    noise, g = dev(normal((16, 16, 16), 5)), dev(normal((32, 32, 32), 6))
    pm.forward(noise)
    want = pm.adjoint(g_dens=g)[0].clone()
    d, v = dev(normal((16 ** 3, 3), 7)), dev(normal((16 ** 3, 3), 8))
    first = [t.clone() for t in (pm.force(d, 0.5), pm.force_vjp(d, 0.5, v), pm.density(d))]
    pm.forward(noise)
    again = [pm.force(d, 0.5), pm.force_vjp(d, 0.5, v), pm.density(d)]
    assert all(torch.equal(a, b) for a, b in zip(first, again))
    assert torch.equal(pm.adjoint(g_dens=g)[0], want)


@pytest.mark.parametrize("np_,ng", [(16, 32), (8, 128), (16, 128), (32, 128), (64, 128)])
@pytest.mark.parametrize("kind", ["spread", "edge"])
def test_force_and_vjp_from_tiles_and_from_the_meshes(np_, ng, kind):
    """Particles everywhere, or all in the last cells of every axis, whose far nodes are the first
    ones: on either side of the spacing and mesh size from which the gathers read the meshes
    themselves."""
    box, n = 50.0, np_ ** 3
    q = opm.lattice(np_, box)
    if kind == "spread":
        d = disps(np_, box)["spread"]
    else:   # x in the last 1.5 cells below the box's end
        d = box - 1.5 * box / ng * np.random.default_rng(5).random((n, 3)) - q
    v = normal((n, 3), 11).astype(np.float32)
    d = d.astype(np.float32)
    units = np.rint(d * np.float32(2.0 ** 32 / box)).astype(np.float64)
    x = np.mod(q + units * (box / 2.0 ** 32), box)
    st = opm.Setup(np_, ng, box, 1, Cosmology())
    want, _, force = opm.pm_force_vjp(x, v.astype(np.float64), st)
    pm = context(np_, ng, box, 1)
    rel = lambda got, ref: np.linalg.norm(got - ref) / np.linalg.norm(ref)
    # 32-bit transforms: some 2^-24 log2(ng^3) = 1.3e-6 of the field's norm; the VJP takes
    # differences of neighbouring nodes and adds three terms of either sign, ten times that
    assert rel(host(pm.force(dev(d), 0.5)), force) < 1e-5
    assert rel(host(pm.force_vjp(dev(d), 0.5, dev(v))), want) < 1e-4
