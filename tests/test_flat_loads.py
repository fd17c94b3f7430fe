"""The addresses of the flat matrix-core kernel's pixel loads, walked through on the host: no load leaves the tensor, and
none depends on whether the hardware counts the uniform part of an offset in its size check."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_pixel_load_stays_inside_the_tensor(tmp_path):
    exe = str(tmp_path / "flat_loads_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Wextra", "-I", os.path.join(ROOT, "paper_1909_05073_amd", "csrc"),
                    os.path.join(ROOT, "tests", "flat_loads_check.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
