"""The division by host-known divisors that the kernels' index arithmetic uses, against the division itself."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_fast_div_is_exact(tmp_path):
    exe = str(tmp_path / "fast_div")
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-O2", "-std=c++17", "-I" + os.path.join(ROOT, "include"),
                    "-I" + os.path.join(ROOT, "paper_2505_19634_amd", "csrc"), "-x", "hip", os.path.join(ROOT, "tests", "fast_div_main.cpp"),
                    "-o", exe], check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
