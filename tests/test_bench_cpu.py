"""What bench.py reports beside its measurements, without a GPU."""
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402

# Gentries/s evaluated by dense plain sweeps: 1 M points per side (d = 3) in 164 ms
DENSE_3D = 2.0 ** 40 / 0.164 / 1e9


@pytest.mark.parametrize("dim", [1, 2, 3])
def test_the_peak_is_a_bound(dim):
    peak = bench.sweep_peak_gentries(dim)
    # no sweep does without its exponential: a quarter-rate instruction takes 8
    # cycles a wavefront, on four SIMDs of 256 CUs at 2.4 GHz
    assert peak < 256 * 4 * 64 * 2.4e9 / 8.0 / 1e9
    assert peak > DENSE_3D  # lower dimensions take fewer steps
    if dim < 3:
        assert peak > bench.sweep_peak_gentries(dim + 1)
