"""Line sums by image columns (csrc/radon_cols.hpp): the strip walk, line
ownership and weights on the host against direct sums over the lines' bilinear
samples, for odd sizes, dense and sparse line grids and sample steps."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "radon_cols_test.cpp")


def test_column_sums_equal_sample_sums(tmp_path):
    exe = tmp_path / "radon_cols_test"
    cmd = ["/opt/rocm/bin/hipcc", "-std=c++17", "-O2", "--offload-arch=gfx950", "-Xclang", "-target-feature",
           "-Xclang", "-packed-fp32-ops", "-x", "hip", SRC, "-o", str(exe)]
    subprocess.run(cmd, check=True, capture_output=True, text=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stdout + res.stderr
    assert "ok worst" in res.stdout
