"""bench.py names the kernel and the peak of the projector products by the routes that the plan counted."""
import hashlib
import json

import pytest

import bench


def _cls(tflops, routes):
    return {"ms": 10.0, "launches": 10, "bytes": 0.0, "flops": 10 * tflops * 1e9, "routes": routes}


def test_int8_products_below_the_fp64_peak_are_int8():
    r = bench.class_roofline("project", _cls(71.0, {"mfma": 1, "fp16": 0, "fp16_128": 0, "int8": 9}), "f64", 96)
    assert r["kernel"] == "k_rns_gemm" and r["mfma_dtype"] == "i8x48" and r["peak"] == 5000.0
    assert r["executed_frac"] == pytest.approx(71.0 * 12 / 5000.0)


def test_fp64_products_stay_fp64_whatever_their_rate():
    r = bench.class_roofline("backproject", _cls(120.0, {"mfma": 9, "fp16": 0, "fp16_128": 0, "int8": 1}), "f64", 96)
    assert r["mfma_dtype"] == "f64" and r["kernel"] == "k_gemm<double, double, double, double, 1, 2>"


@pytest.mark.parametrize("n,routes,kernel", [
    (128, {"mfma": 1, "fp16": 0, "fp16_128": 18, "int8": 0}, "k_gemm_hp"),
    (128, {"mfma": 1, "fp16": 18, "fp16_128": 0, "int8": 0}, "k_gemm_h<double, double, 0, 1>"),
    (48, {"mfma": 0, "fp16": 1, "fp16_128": 18, "int8": 0}, "k_gemm_hp"),
])
def test_mixed_products_by_their_tile(n, routes, kernel):
    r = bench.class_roofline("project", _cls(200.0, routes), "f32", n)
    assert r["kernel"] == kernel and r["mfma_dtype"] == "f16x3"


def test_traffic_of_a_kernel_that_serves_two_classes(tmp_path, monkeypatch):
    csrc = tmp_path / "paper_1406_4350_amd" / "csrc"
    csrc.mkdir(parents=True)
    (csrc / "k.hip").write_text("kernel")
    h = hashlib.sha256(b"kernel").hexdigest()
    (tmp_path / "profiles").mkdir()
    ent = {"n": 128, "source": "k.hip", "source_sha256": h}
    (tmp_path / "profiles" / "traffic.json").write_text(json.dumps(
        {"k project": dict(ent, bytes_per_launch=1.0), "k backproject": dict(ent, bytes_per_launch=2.0)}))
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    assert bench.load_traffic("k", 128, "project") == 1.0 and bench.load_traffic("k", 128, "backproject") == 2.0
    assert bench.load_traffic("k", 128) is None and bench.load_traffic("k", 128, "small") is None
