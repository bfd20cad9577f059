"""The library holds no kernel that nothing launches: FP64 lines of the implicit scheme stop at 4352
unknowns, which chunks of 8 cover, so the x-line kernel with chunks of 16 exists in FP32 only."""
import os
import re
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2005_11931_amd", "csrc")


@pytest.mark.slow
def test_x_line_kernels(tmp_path):
    out = tmp_path / "implicit.s"
    subprocess.run(["/opt/rocm/bin/hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "--offload-device-only", "-S",
                    os.path.join(CSRC, "fdw_implicit.hip"), "-o", str(out)], check=True, capture_output=True)
    names = re.findall(r"\.amdhsa_kernel \S*k_adi_xI([fd])Li(\d+)E", out.read_text())
    assert sorted(names) == [("d", "4"), ("d", "8"), ("f", "16"), ("f", "4"), ("f", "8")]
