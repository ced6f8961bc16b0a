"""The byte model of the batched kernel by rounds (bench.py, no GPU)."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench  # noqa: E402


def test_rounds_bytes_model():
    sizes = [10, 5000, 300, 20000]
    st = {"work": [[7, 40, 90, 60, 0, 5, 0, 2], [100, 30, 200, 80, 10, 500, 20, 4]]}
    per_state = 112 * 25310  # 32-bit marks
    split = 68 * (5 + 20) + 12 * 4
    assert bench.rounds_bytes(sizes, st, 4) == pytest.approx(
        per_state + 8 * 70 + 20 * 290 + 4 * 500 + split)
    assert bench.rounds_bytes(sizes, st, 8) - bench.rounds_bytes(sizes, st, 4) == 4 * 25310
