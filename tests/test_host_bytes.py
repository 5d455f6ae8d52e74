"""Algorithmic bytes booked per kernel family (pm_stats.kernel_bytes) for the first reverse step and
the filter's transposed pass, on the CPU (host_model.py), against counts of what each kernel reads
and writes: positions, momenta and cotangents 12 bytes a particle, ids, keys, ranks and order 4."""
import subprocess

import pytest

from host_model import build
from paper_2211_09958_amd._lib import KERNEL_FAMILIES

P = 8 ** 3


@pytest.fixture(scope="module")
def booked(tmp_path_factory):
    exe = build(tmp_path_factory.mktemp("host_model"))

    def run(mesh, filt, dens, disp, mom):
        args = [str(int(v)) for v in (mesh, filt, dens, disp, mom)]
        out = subprocess.run([exe, *args], check=True, capture_output=True, text=True).stdout
        return dict(zip(KERNEL_FAMILIES, map(float, out.split())))

    return run


@pytest.mark.parametrize("ng", [16, 128])
def test_first_reverse_step(booked, ng):
    r = 4 * ng ** 3
    last = 36 * P + r              # mesh gradient at x_0: x read, xi read and written
    undrift = (24 + 12 + 12 + 12 + 8) * P   # x read, written; p, xi read; pi, key, rank written
    count, order, rebin = 20 * P, 12 * P, 12 * P
    # x, p, ord read, written; id, xi written; xi, pi read where given, pi written then
    compact = (24 + 24 + 8 + 4 + 12) * P
    b = booked(ng, False, False, True, False)
    assert b["wgrad"] == undrift + last
    assert b["bin"] == count + order + compact + 12 * P + rebin
    b = booked(ng, False, True, False, False)
    assert b["wgrad"] == undrift + 2 * last
    assert b["bin"] == count + order + compact + rebin
    # with a momentum cotangent: the whole reverse step, xi written and pi read too
    b = booked(ng, False, False, True, True)
    assert b["wgrad"] == undrift + 24 * P + r + last
    assert b["bin"] == count + order + compact + 36 * P + rebin


@pytest.mark.parametrize("ng", [16, 128])
def test_filtered_transpose(booked, ng):
    c = 8 * ng * ng * (ng // 2 + 1)
    terms = 4 * (ng // 2 + 1) * ng * (ng // 2 + 1)   # |n0|, n1, k2
    assert booked(ng, False, False, True, False)["grad_adj_z"] == 3 * c
    assert booked(ng, True, False, True, False)["grad_adj_z"] == 4 * c + 2 * terms
