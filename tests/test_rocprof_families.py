"""Families and byte rules of the reverse step's and the filter's kernels in the rocprofv3 summary:
the library books them in these families with these bytes (test_host_bytes.py)."""
import pytest

from paper_2211_09958_amd import rocprof_summary as rs


@pytest.mark.parametrize("symbol,family,nbytes", [
    ("k_undrift", "wgrad", 68 * 8),
    ("k_gather_tile<8, 3>", "wgrad", 92 * 8 + 4 * 16 ** 3),
    ("k_grad_adj_z<16, false>", "grad_adj_z", 3 * 8 * 16 * 16 * 9),
    ("k_grad_adj_z<16, true>", "grad_adj_z", 4 * 8 * 16 * 16 * 9 + 4 * 16 * 9 * 9),
    ("k_filter_shells", "grad_adj_z", 4 * 16 * 9 * 9),
    ("k_filter_sum", "grad_adj_z", None),
])
def test_families(symbol, family, nbytes):
    fam, rule = rs.family(symbol, 16)
    assert fam == family
    assert rs.alg_bytes(rule, 1, 8, 16) == nbytes
