"""Host-side checks of bench.py's command line (no GPU)."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_more_than_one_gpu_exits_with_a_message():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True,
                       text=True, timeout=120)
    assert r.returncode == 2
    assert "one GPU only" in r.stderr and r.stdout == ""


def test_gemm_fractions_are_of_the_unit_that_runs_them():
    sys.path.insert(0, ROOT)
    import bench

    def peak(prec, nfld, kernel):
        unit, products, _ = bench.gemm_unit(prec, nfld, kernel)
        return bench.PEAK[unit] / products

    for k in ("legendre_inverse_gemm", "legendre_direct_gemm"):
        assert peak("fp64", 411, k) == 78.6
        assert peak("fp32", 411, k) == 2500.0 / 6  # six bfloat16 products
        assert peak("bf16x3", 411, k) == peak("fp16x3", 411, k) == 2500.0 / 3
        assert peak("fp32", 16, k) == 157.3  # few fields
    assert peak("fp32", 17, "legendre_inverse_gemm") == 2500.0 / 6 and peak("fp32", 17, "legendre_direct_gemm") == 157.3
