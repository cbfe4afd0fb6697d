"""bench.py's table of launches (no GPU): both halves of the factored step are
priced at what they move, their own input, potential and aux and their output."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

import bench  # noqa: E402


@pytest.mark.parametrize("csz,rsz", [(16, 8), (8, 4)])
def test_second_half_moves_what_the_first_does(csz, rsz):
    n = 128
    moved = n ** 3 * (2 * csz + rsz) + 6 * n * n * 32
    rows = [bench.launch_row("fused2_half_" + h, ms, n, 1, csz, rsz) for h, ms in (("a", 0.019), ("b", 0.0205))]
    for r in rows:
        assert r["impl_bytes"] == moved
        assert r["impl_GB/s"] == pytest.approx(moved / (r["ms"] * 1e-3) / 1e9)
    roof = bench.roofline(rows, n, 1, csz, rsz, 0.0395, None)
    assert roof["kernel"] == "fused2_half_b"
    assert roof["impl_bytes_per_launch"] == moved
    assert roof["impl_frac"] == pytest.approx(moved / 0.0205e-3 / 8e12)
