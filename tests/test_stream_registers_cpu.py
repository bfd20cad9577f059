"""Registers of streaming variants that sit just below a step of the waves a SIMD holds (512 registers
per lane: three waves up to 168, two up to 256), from the resource descriptors of the gfx950 code
compiled here: a few registers more cost them a wave."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2005_11931_amd", "csrc")

# (variant <type, time block, columns per lane, faces, mode>, most registers); mode bit 0: energies,
# bit 1: traces, bit 2: non-temporal loads
VARIANTS = [
    ("float, 8, 2, 1, 1", 168),  # FP32 with separate h2 and energies: the default of such a solve
    ("float, 8, 2, 1, 5", 168),
    ("float, 6, 4, 1, 1", 256),  # the same with 4 columns per lane at its deepest time block
    ("float, 6, 4, 1, 5", 256),
    ("double, 8, 1, 0, 3", 168),  # FP64 with traces and energies
]


@pytest.fixture(scope="module")
def resources(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("registers")
    src, out = tmp / "variants.hip", tmp / "variants.s"
    src.write_text('#include "fdw_stream.h"\nnamespace fdw {\n'
                   + "".join(f"template __global__ void k_step<{v}>(StepArgs);\n" for v, _ in VARIANTS) + "}\n")
    subprocess.run(["/opt/rocm/bin/hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "--offload-device-only", "-S",
                    "-I", CSRC, str(src), "-o", str(out)], check=True, capture_output=True)
    got = {}
    for name, meta in re.findall(r"\.amdhsa_kernel (\S+)\n(.*?)\.end_amdhsa_kernel", out.read_text(), flags=re.S):
        m = re.match(r"_ZN3fdw6k_stepI([fd])Li(\d)ELi(\d)ELi(\d)ELi(\d)E", name)
        key = ("float" if m.group(1) == "f" else "double",) + m.groups()[1:]
        got[", ".join(key)] = (int(re.search(r"next_free_vgpr (\d+)", meta).group(1)),
                               int(re.search(r"private_segment_fixed_size (\d+)", meta).group(1)))
    return got


@pytest.mark.slow
@pytest.mark.parametrize("variant,most", VARIANTS)
def test_variant_keeps_its_waves(resources, variant, most):
    registers, scratch = resources[variant]
    assert registers <= most and scratch == 0, (registers, scratch)
