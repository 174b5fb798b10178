"""bench.py's roofline of a product mesh (no GPU): the kernel is charged with the bytes
that it moves there, and a measured traffic with its own rate."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench  # noqa: E402


@pytest.mark.parametrize("precision,fused", [("fp64", 120.0), ("fp32", 88.0)])
def test_product_mesh_is_not_charged_with_metric_terms(precision, fused, monkeypatch):
    npts, run = 10 ** 9, {"kernel_ms": 4000.0, "launches": 100}
    r = bench.roofline(precision, False, npts, run, "no-such-workload", product=True)
    assert r["fused"]["bytes_per_point"] == fused
    assert r["fused"]["achieved"] == pytest.approx(fused * npts / 0.040 / 1e9, abs=0.05)
    assert r["bound"] != "hbm" and r["moved"] is None
    monkeypatch.setattr(bench, "traffic_for", lambda *a: 1.5e11)
    r = bench.roofline(precision, False, npts, run, "any", product=True)
    assert r["traffic"] == 1.5e11 and r["moved"] == {"achieved": 3750.0, "frac": 0.4688}
    held = bench.roofline(precision, True, npts, run, "any", product=True)
    assert held["fused"]["bytes_per_point"] == fused + bench.HELD_VISC_BYTES[precision]
