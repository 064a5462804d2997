"""The roofline of the bench line is a fraction of what the hardware can do."""
import pytest

import bench


class _Context:
    def __init__(self, stats):
        self.stats = stats

    def profile_read(self):
        return self.stats


@pytest.mark.parametrize("name, runs", [("zgemm3m_128x64", 0.75), ("zgemm3m_queue", 0.75), ("block_solve", 0.75),
                                        ("zgemm_64x64", 1.0), ("dgemm", 1.0)])
def test_products_of_three_real_ones_count_what_they_execute(name, runs):
    """88 TF of 8 M N K are 66 TF on the matrix cores (peak 78.6) where three
    real products make a complex one."""
    flops = 88e12 * 0.25 if runs < 1 else 66e12 * 0.25
    stats = [{"name": name, "launches": 57, "ms": 250.0, "flops": flops, "bytes": 1e9},
             {"name": "lu_panel", "launches": 32, "ms": 88.0, "flops": 0.0, "bytes": 1e10}]
    r = bench.live_roofline(_Context(stats))
    assert r["kernel"] == name
    assert r["achieved"] == pytest.approx(66.0) and r["frac"] == pytest.approx(66.0 / 78.6)
    assert r["flops_per_launch"] == pytest.approx(runs * flops / 57)
    assert r["all_kernels"][name]["TFLOP/s"] == pytest.approx(66.0)
    assert stats[0]["flops"] == flops
