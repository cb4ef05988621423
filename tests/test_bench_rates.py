"""bench.py counts the bytes of what it launched (CPU)."""

import pytest

import bench


def test_pairs_of_steps_move_the_bytes_of_one():
    # 100 steps of 1e6 sites at 304 B a site: alone in 50 ms of kernels, in pairs in 26 ms
    alone = bench.launch_rates(304, 10 ** 6, 100, 100, 50.0, 0.051)
    pairs = bench.launch_rates(304, 10 ** 6, 100, 50, 26.0, 0.0265)
    assert alone["kernel"] == pytest.approx(608.0) and alone["step"] == pytest.approx(30.4 / 0.051)
    assert alone["one_step_a_launch"] == alone["step"]
    assert pairs["kernel"] == pytest.approx(15.2 / 0.026)            # 50 launches of 304 MB
    assert pairs["step"] == pytest.approx(15.2 / 0.0265)
    assert pairs["one_step_a_launch"] == pytest.approx(30.4 / 0.0265)
    assert bench.launch_rates(304, 10 ** 6, 100, 0, 0.0, 1.0)["kernel"] == 0.0
