"""Registers of the batched kernels as the compiler reports them (no GPU).

The kernels of a batch without teams hold four workgroups per CU in 64 registers; the code for
teams must not be paid for there in spilled ones.
"""
import os
import re
import subprocess

import pytest

from paper_0811_2518_amd import build


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="hipcc not installed")
def test_batched_kernels_without_teams_do_not_pay_for_them():
    r = subprocess.run([build.HIPCC, *build.CFLAGS, "--offload-device-only", "-c", os.path.join(build.CSRC, "batched.hip"),
                        "-o", os.devnull, "-Rpass-analysis=kernel-resource-usage"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    name, spills, waves = None, {}, {}
    for line in r.stderr.splitlines():
        if m := re.search(r"Function Name: (\S+)", line):
            name = m.group(1)
        elif m := re.search(r"VGPRs Spill: (\d+)", line):
            spills[name] = int(m.group(1))
        elif m := re.search(r"Occupancy \[waves/SIMD\]: (\d+)", line):
            waves[name] = int(m.group(1))
    for kernel, most in (("k_bprec", 0), ("k_brhs", 6)):
        plain = [k for k in spills if kernel in k and k.endswith("Lb0EEEvNS0_9BatchArgsE")]
        assert len(plain) == 2, sorted(spills)  # both schedules
        for k in plain:
            assert spills[k] <= most and waves[k] == 8, (k, spills[k], waves[k])
