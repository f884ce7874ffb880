"""Index arithmetic of the line transforms over the plans the kernels use
(make_plan, Stage and lds_at in csrc/fft.h), checked on the CPU: every length,
stage, butterfly and element, for both element sizes.  Built from the library's
own header with hipcc for the host only."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1907_01194_amd", "csrc")


def test_plan_indices(tmp_path):
    hipcc = shutil.which("hipcc") or ("/opt/rocm/bin/hipcc" if os.path.exists("/opt/rocm/bin/hipcc") else None)
    if hipcc is None:
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "plan_check")
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-std=c++20", "-iquote", CSRC,
                    os.path.join(ROOT, "tests", "native", "plan_check.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout
    assert out.strip().endswith("violations 0"), out
