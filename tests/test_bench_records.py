"""Host logic of bench.py's records (CPU): which kernel, tile and peak a record is made with."""
import csv
import json
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402


class _Lat:
    """Stands in for a lattice: fixed times."""

    def bench_dirac(self, prec="f64", nrhs=1, region="full", iters=50):
        return {"f64": 2.0, "bf16": 1.0}[prec]

    def bench_sap(self, prec="f32", nrhs=1, nmr=4, iters=20, eo=False):
        return 1.0 if nmr else 0.5


class _Lib:
    """Stands in for the package: the block solver's tile."""

    def __init__(self, tile):
        self.tile = tile

    def sap_eo_tiles(self, lats, nrhs, prec):
        return [self.tile] * len(lats)


def test_rhs_per_lane_of_the_d_rows(monkeypatch):
    lat = _Lat()
    monkeypatch.setattr(bench, "_TILES", {(id(lat), "bf16"): 4, (id(lat), "f64"): 2})
    r = bench.dirac_rates(lat, 1000, ("f64", "bf16"), nrhs=12)
    assert r["f64"]["rhs_per_lane"] == 1 and r["bf16"]["rhs_per_lane"] == 4
    assert abs(r["f64"]["GB/s"] - bench.dw_bytes("f64", 1) * 12000 / 2e-3 / 1e9) < 1e-9
    assert abs(r["bf16"]["GB/s"] - bench.dw_bytes("bf16", 4) * 12000 / 1e-3 / 1e9) < 1e-9


def test_block_solver_of_a_record():
    lat = _Lat()
    assert bench.block_solver(_Lib(4), lat, 12, "bf16") == ("k_sap_eo_mm<3>", 4)
    assert bench.block_solver(_Lib(4), lat, 9, "f16") == ("k_sap_eo_mm<2>", 3)
    assert bench.block_solver(_Lib(1), lat, 12, "bf16") == ("k_sap_eo<3, 1, false>", 1)
    assert bench.block_solver(_Lib(2), lat, 12, "f32") == ("k_sap_eo<1, 2, false>", 2)


def test_roofline_counts_the_operator_per_tile_and_the_peak_of_its_units():
    lat, block, V = _Lat(), (4, 4, 4, 4), 663552
    sites = V // 2 * 12
    vec = bench.roofline_record(lat, V, "bf16", 12, block, "v")
    mat = bench.roofline_record(lat, V, "bf16", 12, block, "m", tile=4, peak=bench.FP32_MATRIX_PEAK_TFLOPS)
    assert vec["alg_bytes_per_launch"] == pytest.approx(612 * sites)
    assert mat["alg_bytes_per_launch"] == pytest.approx((300 / 4 + 312) * sites)
    assert vec["alg_flops_per_launch"] == mat["alg_flops_per_launch"] == pytest.approx(8484 * sites)
    assert bench.FP32_MATRIX_PEAK_TFLOPS == pytest.approx(2 * bench.FP32_PEAK_TFLOPS)
    assert mat["frac_of_fp32_peak"] == mat["frac"] == pytest.approx(vec["frac_of_fp32_peak"] / 2)
    assert mat["ridge"] == pytest.approx(2 * vec["ridge"]) and mat["bound"] == "alu"


def _counters(path, rows):
    with open(path, "w", newline="") as f:
        w = csv.DictWriter(f, fieldnames=["Dispatch_Id", "Kernel_Name", "Counter_Name", "Counter_Value"])
        w.writeheader()
        for i, k, c, v in rows:
            w.writerow({"Dispatch_Id": i, "Kernel_Name": k, "Counter_Name": c, "Counter_Value": v})


def test_issue_record_of_the_kernel_that_ran_last(tmp_path):
    """The autotuner launches the vector kernel too; the timing loops' kernel comes last.  Vector
    instructions hold a SIMD for 4 cycles, matrix instructions (counted with them) for 8."""
    vec, mm = "void wc::k_sap_eo<3, 1, false>(wc::SapLaunch)", "void wc::k_sap_eo_mm<3>(wc::SapLaunch)"
    rows = []
    for i in range(30):
        rows += [(i, vec, "SQ_INSTS_VALU", 50.0), (i, vec, "SQ_INSTS_MFMA", 0.0), (i, vec, "GRBM_GUI_ACTIVE", 8.0)]
    for i in range(30, 74):
        v, m, g = (100.0, 20.0, 1600.0) if i < 52 else (300.0, 120.0, 4800.0)
        rows += [(i, mm, "SQ_INSTS_VALU", v), (i, mm, "SQ_INSTS_MFMA", m), (i, mm, "GRBM_GUI_ACTIVE", g)]
    rows += [(80, "void wc::k_dirac<1, 4, true, 3>(wc::DiracLaunch)", "SQ_INSTS_VALU", 1.0)]
    _counters(tmp_path / "q.csv", rows)
    out = tmp_path / "v.json"
    bench.valu_record(str(tmp_path / "q.csv"), str(out), simds=4, xcds=8)
    (name, k), = json.load(open(out))["kernels"].items()
    assert name == "k_sap_eo_mm<3>"
    assert k["valu_busy_launch"] == pytest.approx((180 * 4 + 120 * 8) / (4 * 600))
    assert k["valu_busy_without_mr_steps"] == pytest.approx((80 * 4 + 20 * 8) / (4 * 200))
    assert k["valu_busy_mr_steps"] == pytest.approx((100 * 4 + 100 * 8) / (4 * 400))
    assert k["valu_instructions_mr_steps"] == 100 and k["mfma_instructions_mr_steps"] == 100
    for kernel in ("k_sap_eo<3, 1, false>", "k_sap_eo<1, 1, false>"):  # no timing loop of it; not launched
        with pytest.raises(ValueError, match="no launch"):
            bench.valu_record(str(tmp_path / "q.csv"), str(out), kernel=kernel)
