"""Every shape that resident sweeps accept fits a buffer the kernel is built for,
and small work-groups of any shape share a compute unit (host only)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_accepted_shape_fits_and_shares(tmp_path):
    exe = str(tmp_path / "resident_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2102_12416_amd", "csrc"), "-o", exe,
                    os.path.join(ROOT, "tests", "resident_check.cpp")], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout + out.stderr
    words = out.stdout.split()
    assert int(words[1]) > 100000 and words[3] == "0" and words[5] == "0", out.stdout
