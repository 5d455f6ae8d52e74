"""pm_destroy beside other streams' work, and the pinned host memory that contexts hand on."""
import pytest
import torch

from gpu_util import CO, dev
from paper_2211_09958_amd import api
from synthetic import normal

pytestmark = pytest.mark.gpu


def make(ng=16, steps=2):
    return api.PMContext(api.make_config(8, ng, 40.0, steps, a_stop=0.1), CO)


def test_does_not_wait_for_other_streams():
    pm = make()
    side, done = torch.cuda.Stream(), torch.cuda.Event()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        torch.cuda._sleep(100_000_000)   # some 40 ms; pm_destroy takes 0.02
        done.record()
    pm.close()
    assert not done.query()
    side.synchronize()


def test_under_capture():
    pm, x = make(), torch.zeros(64, device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        x.add_(1.0)
        pm.close()
        x.add_(1.0)
    for k in (1, 2):
        g.replay()
        torch.cuda.synchronize()
        assert bool((x == 2.0 * k).all())


def test_results_in_memory_handed_on():
    """Contexts of several sizes made and closed in changing order, three open at a time."""
    sizes = [(8, 2), (16, 5), (64, 2), (256, 1), (16, 700)]   # 4 to 16 KB of results
    want, open_ = {}, []
    for turn in range(3):
        for k, (ng, steps) in enumerate(sizes):
            open_.append(((ng, steps), make(ng, steps)))
            if len(open_) > 3:
                open_.pop((turn + k) % 3)[1].close()
            for key, pm in open_:
                d, t = dev(normal((key[0],) * 3, 1)), dev(normal((key[0],) * 3, 2))
                got = (pm.loss_mse(d, t)[0], float(pm.power_spectrum(d)[1][2]))
                ref = want.setdefault(key, got)
                assert abs(got[0] / ref[0] - 1) < 1e-12 and abs(got[1] / ref[1] - 1) < 1e-12
    for _, pm in open_:
        pm.close()
