"""The four-value division by 6 of the resident sweeps equals s / 6 (host only;
the device's own is in test_gpu_device_helpers.py)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_div6_quad_equals_ieee_division(tmp_path):
    exe = str(tmp_path / "div6_quad_check")
    subprocess.run([HIPCC, "--offload-host-only", "-O2", "-ffp-contract=off", "-fno-fast-math", "-I",
                    os.path.join(ROOT, "paper_2102_12416_amd", "csrc"), "-o", exe,
                    os.path.join(ROOT, "tests", "div6_quad_check.hip")], check=True, capture_output=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stdout + out.stderr[-2000:]
    words = out.stdout.split()
    assert int(words[1]) > 10 ** 7 and words[3] == "0", out.stdout
