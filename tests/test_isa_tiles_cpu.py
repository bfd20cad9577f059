"""Checks on the gfx950 assembly of the kernels that hold small grids in register tiles, compiled here from
source: the reverse tile kernel and the forward one that records traces.

  * nothing spills: a tile's states stay in registers through its levels;
  * the registers allow the workgroups that are launched (a workgroup of 16 waves leaves a lane 128, of
    12 waves 168, of 8 waves 256);
  * plane reads are buffer loads of one element (out-of-range rows read 0 without a branch).
"""
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2005_11931_amd", "csrc")
UNITS = ["fdw_adjoint_tile.hip", "fdw_tile.hip"]


def _asm(unit, tmp):
    out = os.path.join(tmp, unit + ".s")
    subprocess.run(["/opt/rocm/bin/hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "--offload-device-only", "-S",
                    os.path.join(CSRC, unit), "-o", out], check=True, capture_output=True)
    with open(out) as f:
        return f.read()


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    tmp = str(tmp_path_factory.mktemp("isa_tiles"))
    with ThreadPoolExecutor(max_workers=len(UNITS)) as ex:
        return dict(zip(UNITS, ex.map(lambda u: _asm(u, tmp), UNITS)))


def _kernels(text, pattern):
    """(match of `pattern` on the mangled name, body, registers, scratch bytes) of every such kernel."""
    bodies = dict(re.findall(r"^(_Z[^\s:]+):[^\n]*\n(.*?)^\.Lfunc_end", text, flags=re.M | re.S))
    out = []
    for name, meta in re.findall(r"\.amdhsa_kernel (\S+)\n(.*?)\.end_amdhsa_kernel", text, flags=re.S):
        m = re.search(pattern, name)
        if m:
            out.append((m, bodies[name], int(re.search(r"next_free_vgpr (\d+)", meta).group(1)),
                        int(re.search(r"private_segment_fixed_size (\d+)", meta).group(1))))
    return out


@pytest.mark.slow
def test_reverse_tiles(asm):
    # <type, rows per wave, faces, separate gradients>: 12 waves of 4 rows, 8 waves of 8 rows
    kernels = _kernels(asm["fdw_adjoint_tile.hip"], r"k_adjoint_tileI([fd])Li(\d)ELi(\d)ELi(\d)E")
    assert len(kernels) == 16
    for m, body, registers, scratch in kernels:
        assert scratch == 0, m.groups()
        assert registers <= (168 if m.group(2) == "4" else 256), (m.groups(), registers)
        loads = set(re.findall(r"\b(buffer_load_\w+)", body))  # (accumulators and sources are FP64)
        assert loads == ({"buffer_load_dwordx2"} if m.group(1) == "d" else {"buffer_load_dword", "buffer_load_dwordx2"})


@pytest.mark.slow
def test_recording_tiles(asm):
    kernels = _kernels(asm["fdw_tile.hip"], r"k_record_tileI([fd])Li(\d)ELi(\d)E")
    assert len(kernels) == 8
    for m, body, registers, scratch in kernels:
        assert scratch == 0 and registers <= 128, (m.groups(), registers, scratch)
        loads = set(re.findall(r"\b(buffer_load_\w+)", body))
        assert loads == ({"buffer_load_dwordx2"} if m.group(1) == "d" else {"buffer_load_dword"}), (m.groups(), loads)


@pytest.mark.slow
def test_no_forbidden_instructions(asm):
    import test_isa_cpu

    test_isa_cpu.test_no_scalar_cache_writes_or_packed_fp32({"fdw_adjoint_tile.hip": asm["fdw_adjoint_tile.hip"]})
