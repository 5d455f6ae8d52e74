"""The bin counts a sort starts from are zero on the device whatever became of earlier calls: calls
that were only captured, captures replayed late, and contexts on memory that held something else."""
import ctypes

import pytest
import torch

from gpu_util import CO, dev
from paper_2211_09958_amd import _lib, api
from synthetic import normal

pytestmark = pytest.mark.gpu


def fresh(np_, ng, steps=1):
    """A context whose workspace most likely reuses memory of all ones."""
    cfg = api.make_config(np_, ng, 50.0, steps)
    old = torch.full((api.workspace_bytes(cfg),), 255, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    del old
    return api.PMContext(cfg, CO)


def density(pm, d, out):
    rc = pm.lib.pm_density(pm.ctx, ctypes.c_void_p(d.data_ptr()), ctypes.c_void_p(out.data_ptr()))
    assert rc == 0


# the counts are cleared by the density scatter (meshes to 64^3) or by the order
@pytest.mark.parametrize("np_,ng", [(8, 8), (16, 64), (32, 128)])
def test_calls_that_were_only_captured(np_, ng):
    d = dev(0.5 * 50.0 / np_ * normal((np_ ** 3, 3), 1))
    other = dev(50.0 * normal((np_ ** 3, 3), 2))
    want = api.PMContext(api.make_config(np_, ng, 50.0, 1), CO).density(d)
    torch.cuda.synchronize()
    with torch.cuda.stream(torch.cuda.Stream()):
        pm = fresh(np_, ng)
        out = [torch.empty_like(want) for _ in range(3)]
        torch.cuda.synchronize()
        dropped, late = torch.cuda.CUDAGraph(), torch.cuda.CUDAGraph()
        for g, o in ((dropped, out[0]), (late, out[1])):
            with torch.cuda.graph(g, stream=pm.stream):
                density(pm, d, o)
        del dropped
        for _ in range(3):
            density(pm, other, out[2])
            density(pm, d, out[2])
            assert torch.equal(out[2], want)
            late.replay()
            torch.cuda.synchronize()
            assert torch.equal(out[1], want)
            out[1].zero_()


@pytest.mark.parametrize("np_,ng", [(16, 64), (32, 128)])
def test_calls_after_a_failed_one(np_, ng):
    """A call that reports a HIP error (left here by a refused hipSetDevice) may have stopped half
    way: the next sorts clear the counts themselves, a captured one too."""
    d = dev(0.5 * 50.0 / np_ * normal((np_ ** 3, 3), 1))
    want = api.PMContext(api.make_config(np_, ng, 50.0, 1), CO).density(d)
    torch.cuda.synchronize()
    with torch.cuda.stream(torch.cuda.Stream()):
        pm = fresh(np_, ng)
        out = torch.empty_like(want)
        torch.cuda.synchronize()
        assert pm.lib.hipSetDevice(1 << 20) != 0
        with pytest.raises(api.PMError) as e:
            pm.density(d)
        assert e.value.code == _lib.PM_EHIP
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=pm.stream):
            density(pm, d, out)
        for _ in range(2):
            assert torch.equal(pm.density(d), want)
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, want)
            out.zero_()


@pytest.mark.parametrize("np_,ng", [(8, 8), (16, 64), (32, 128)])
def test_runs_and_building_blocks_in_turn(np_, ng):
    """Counts left by the gathers of a run and by the building blocks: a used context gives the
    bits of a new one (densities and forces are sums of integers and fixed-order arithmetic)."""
    noise = dev(normal((np_,) * 3, 3))
    used = fresh(np_, ng, 2)
    for seed in (4, 5):
        d = dev(0.5 * 50.0 / np_ * normal((np_ ** 3, 3), seed))
        disp = used.forward(noise)[0]
        used.adjoint(g_disp=d)
        got = used.density(d), used.force(d, 0.5), disp
        new = fresh(np_, ng, 2)
        assert new is not used
        assert torch.equal(got[0], new.density(d))
        assert torch.equal(got[1], new.force(d, 0.5))
        assert torch.equal(got[2], new.forward(noise)[0])
