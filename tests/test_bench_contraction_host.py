"""bench.py's contraction leg on made-up times (no GPU): the fields describe
the contraction that runs, not the panel GEMM beside it."""
import os
import sys
import types

import numpy as np
import pytest

import paper_1607_01249_amd as ttx
import workloads

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench  # noqa: E402


class _Tensor:
    def __getattr__(self, name):
        return lambda *a, **k: self


def test_fields_follow_the_contraction(monkeypatch):
    seconds = iter([0.5e-3, 2e-3, 1e-3] * len(workloads.CONTRACTIONS))   # contraction, panel GEMM, torch
    monkeypatch.setattr(bench, "time_events", lambda *a: (None, next(seconds)))
    monkeypatch.setattr(bench, "fill_uniform", lambda *a: None)
    for name in ("ttx_contraction_execute", "ttx_gemm_panels"):
        monkeypatch.setattr(ttx, name, lambda *a: 0)
    torch = types.SimpleNamespace(float32=None, float64=None, uint8=None, empty=lambda *a, **k: _Tensor(),
                                  tensordot=lambda *a, **k: _Tensor(),
                                  cuda=types.SimpleNamespace(empty_cache=lambda: None))
    rows = bench.bench_contraction(torch, ttx, 5000.0, 0)
    assert [r["case"] for r in rows] == [c["name"] for c in workloads.CONTRACTIONS]
    for r, case in zip(rows, workloads.CONTRACTIONS):
        es = np.dtype(case["dtype"]).itemsize
        flops = 2.0 * r["m"] * r["n"] * r["k"]
        nbytes = es * (r["m"] * r["k"] + r["k"] * r["n"] + r["m"] * r["n"] * (2 if case["beta"] else 1))
        assert r["bytes"] == nbytes and r["ms"] == 0.5
        assert r["GBps"] == pytest.approx(nbytes / 0.5e-3 / 1e9, abs=0.05)
        assert r["pct_of_d2d"] == pytest.approx(100 * r["GBps"] / 5000.0, abs=0.1)
        assert r["TFLOPs"] == pytest.approx(flops / 0.5e-3 / 1e12, abs=0.01)
        assert r["gemm_frac_of_peak"] == pytest.approx(flops / 0.5e-3 / 1e12 / (157.3 if es == 4 else 78.6), abs=1e-3)
        assert r["panel_gemm_ms"] == 2.0 and r["x_torch"] == 2.0
