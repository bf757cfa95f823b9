"""The benchmark's roofline record: executed operations and counted bytes decide the bound and its
fraction, which no count of work that is not done can push past one."""
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402
from paper_2401_06841_amd import model  # noqa: E402


def _counters(monkeypatch, traffic, flops):
    monkeypatch.setattr(bench, "traffic_from_profiles", lambda *a: traffic)
    monkeypatch.setattr(bench, "executed_flops_from_profiles", lambda *a: flops)


def test_memory_bound(monkeypatch):
    _counters(monkeypatch, 28.0e9, 157.0e9)
    r = bench.roofline("c5", "fp64", "k_rhs", 7.0, 1.0e9)
    assert r["bound"] == "hbm" and r["unit"] == "TB/s" and r["counted"]
    assert r["achieved"] == pytest.approx(4.0) and r["frac"] == pytest.approx(0.5)
    assert r["executed_TFLOP_s"] == pytest.approx(157.0 / 7.0) and r["executed_frac"] < r["frac"]


def test_vector_bound(monkeypatch):
    _counters(monkeypatch, 8.0e9, 350.0e9)
    r = bench.roofline("c5", "fp64", "k_rhs", 7.0, 1.0e9)
    assert r["bound"] == "alu" and r["unit"] == "TFLOP/s"
    assert r["achieved"] == pytest.approx(50.0) and r["frac"] == pytest.approx(50.0 / bench.PEAK_FP64_TFLOPS)
    assert r["hbm_TB_per_s"] == pytest.approx(8.0 / 7.0)


def test_without_counters_the_least_bytes(monkeypatch):
    _counters(monkeypatch, None, None)
    least = model.rhs_bytes_per_cell(2, 8) * 64 ** 3
    assert least == (4 + 3 + 4) * 10 * 8 * 64 ** 3
    assert model.rhs_bytes_per_cell(1, 8, vhat=False) == (4 + 4) * 4 * 8
    r = bench.roofline("c2", "fp64", "k_rhs", 0.125, least)
    assert r["bound"] == "hbm" and not r["counted"] and r["traffic"] is None
    assert r["achieved"] == pytest.approx(least / 0.125e-3 / 1e12) and "executed_frac" not in r
