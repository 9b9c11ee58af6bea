"""bench.py's roofline record on the CPU: rates and fractions come from the bytes that the kernel's storage format moves."""
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_fractions_are_of_the_stored_bytes():
    sys.path.insert(0, ROOT)
    import bench
    # 102.7 MB as stored, 136.1 MB as CSR, in 16.7 us back to back and 34.9 us from HBM
    r = bench.roofline_entry("k", 102.7e6, 136.1e6, 0.0167, 0.0349, None)
    assert r["bytes_per_launch"] == 102.7e6 and r["csr_bytes_per_launch"] == 136.1e6
    assert abs(r["achieved"] - 102.7e6 / 16.7e-6 / 1e9) < 1e-6 and r["unit"] == "GB/s"
    assert abs(r["frac"] - r["achieved"] / bench.PEAK_HBM_GBS) < 1e-12 and r["frac"] < 0.78
    cold = r["hbm_only"]
    assert abs(cold["achieved"] - 102.7e6 / 34.9e-6 / 1e9) < 1e-6
    assert abs(cold["frac"] - cold["achieved"] / bench.PEAK_HBM_GBS) < 1e-12
    # nothing in the source forms a rate from other bytes than those
    src = open(os.path.join(ROOT, "bench.py")).read()
    assert src.count('"frac":') == 2
