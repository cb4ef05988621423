"""bench.py counts the bytes of what it launched (CPU)."""

import pytest

import bench
from paper_1405_6162_amd import profsummary


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


def test_traffic_is_that_of_the_kernel_that_ran(monkeypatch):
    info = {"kernel": "void lbk::k_single_pair<lbk::Tiling<64, 8>, double>(x)", "traffic_bytes_per_launch": "5227618464",
            "source_digest": profsummary.kernel_source_digest()}
    monkeypatch.setattr(profsummary, "read_traffic", lambda path: info)
    assert bench.traffic_from_profile("single256_f64", "k_single_pair") == 5227618464
    assert bench.traffic_from_profile("single256_f64", "k_collide") is None      # one step a launch (--vvl 2)
    assert bench.traffic_from_profile("single256_f64") == 5227618464
    info["source_digest"] = "older"
    assert bench.traffic_from_profile("single256_f64", "k_single_pair") is None
