"""The kernels' 24-bit division of tile coordinates (csrc/fastdiv.h, SmallDiv) is exact up to the bound it was made for
and is refused where it could not be (compiled for the host, no GPU)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_smalldiv_is_exact_up_to_its_bound(tmp_path):
    exe = str(tmp_path / "smalldiv_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_1603_05279_amd", "csrc"),
                    os.path.join(ROOT, "tests", "smalldiv_check.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and "mismatches 0" in r.stdout, r.stdout
