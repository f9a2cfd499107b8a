"""Host logic of bench.py's records (CPU): which kernel, tile and peak a record is made with."""
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402


class _Lat:
    """Stands in for a lattice: fixed times."""

    def bench_dirac(self, prec="f64", nrhs=1, region="full", iters=50):
        return {"f64": 2.0, "bf16": 1.0}[prec]


def test_rhs_per_lane_of_the_d_rows(monkeypatch):
    lat = _Lat()
    monkeypatch.setattr(bench, "_TILES", {(id(lat), "bf16"): 4, (id(lat), "f64"): 2})
    r = bench.dirac_rates(lat, 1000, ("f64", "bf16"), nrhs=12)
    assert r["f64"]["rhs_per_lane"] == 1 and r["bf16"]["rhs_per_lane"] == 4
    assert abs(r["f64"]["GB/s"] - bench.dw_bytes("f64", 1) * 12000 / 2e-3 / 1e9) < 1e-9
    assert abs(r["bf16"]["GB/s"] - bench.dw_bytes("bf16", 4) * 12000 / 1e-3 / 1e9) < 1e-9
