"""What the compiler gives the decode's kernels: registers decide how many workgroups share a CU (no GPU needed)."""
import os
import re
import subprocess

import pytest

from paper_2410_17980_amd import build

# waves per SIMD: three, two and one workgroup of eight waves a CU for the nearest keys, as many as LDS leaves room for; six, four and two of four waves for the far ones
WAVES = {32: 6, 64: 4, 128: 2}


@pytest.fixture(scope="module")
def remarks():
    src = os.path.join(build.CSRC, "sb_decode.hip")
    cmd = [build.HIPCC, *build.FLAGS, "--offload-device-only", "-Rpass-analysis=kernel-resource-usage", "-S", src, "-o", os.devnull]
    out = subprocess.run(cmd, capture_output=True, text=True, check=True).stderr
    kernels, name = {}, None
    for line in out.splitlines():
        if m := re.search(r"remark: .*?Function Name: (\S+)", line):
            name = m.group(1)
        elif m := re.search(r"remark:\s+(.+?): (\d+) \[-Rpass", line):
            kernels.setdefault(name, {})[m.group(1).strip()] = int(m.group(2))
    return kernels


@pytest.mark.parametrize("far", [0, 1])
@pytest.mark.parametrize("d", list(WAVES))
def test_decode_kernels_keep_their_workgroups_a_cu(remarks, d, far):
    got = [v for k, v in remarks.items() if f"decode_kernelILi{d}ELb{far}E" in k]
    assert got
    for g in got:
        assert g["Occupancy [waves/SIMD]"] >= WAVES[d] and g["VGPRs Spill"] == 0 and g["SGPRs Spill"] == 0, g
