"""The bench's headline counts lattice updates that are executed, and its limiter
says one thing (host logic, no GPU)."""
import os
import sys

import pytest

from paper_1601_02708_amd import configs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def bench():
    sys.path.insert(0, ROOT)
    import bench
    return bench


@pytest.mark.parametrize("cfg,precision", [(configs.PORE4096, "fp64"), (configs.PORE2048, "fp32")])
def test_value_counts_executed_updates(bench, cfg, precision):
    spl = bench.default_steps_per_launch(precision)
    r = bench.step_rates(cfg, spl, 10, 4.0)
    whole = cfg.eta * cfg.N ** 2
    assert r["updates_asked_per_step"] == cfg.max_iter * whole
    # the first pass whole, a frame for each later one
    assert whole < r["updates_executed_per_step"] < r["updates_asked_per_step"]
    assert r["value"] == round(r["updates_executed_per_step"] * 10 / 4e-3 / 1e6, 1)
    assert r["mlups_asked"] == round(r["updates_asked_per_step"] * 10 / 4e-3 / 1e6, 1)


def test_single_step_launches_share_nothing(bench):
    r = bench.step_rates(configs.PORE2048, 1, 10, 4.0)
    assert r["value"] == r["mlups_asked"]


def test_one_limiter(bench):
    lim = {"bound": "latency", "limiter": "latency and occupancy"}
    ms = 0.5
    fast, slow = bench.COPY_GBS * 1e9 * ms / 1e3, 0.5 * bench.COPY_GBS * 1e9 * ms / 1e3
    assert bench.hbm_limiter(lim, slow, ms) == lim and bench.hbm_limiter(lim, None, ms) == lim
    got = bench.hbm_limiter(lim, fast, ms)
    assert got["bound"] == "hbm" and "latency" not in got["limiter"]
