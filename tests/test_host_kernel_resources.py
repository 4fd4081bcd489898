"""Registers of the sampler's kernels, as the compiler reports them for gfx950: two workgroups of 1024 threads to a CU leave 64
to a thread, and sweeps that need more go through memory in every round (51 registers over: a nucleus call took a third longer)."""
import os
import re
import subprocess

import pytest

from paper_2506_06122_amd import build


def test_sampler_sweeps_fit_their_registers(tmp_path):
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    src = "kernels_sampler.hip"
    res = subprocess.run([build.HIPCC, *build.FLAGS, *build.PER_FILE[src], "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage",
                          "-c", os.path.join(build.CSRC, src), "-o", str(tmp_path / "o")], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr
    scratch = dict(re.findall(r"Function Name: (\S+)(?:.|\n)*?ScratchSize \[bytes/lane\]: (\d+)", res.stderr))
    assert len([k for k in scratch if "sample_" in k]) == 4, scratch
    # what is left is stored and loaded once a launch, outside the sweeps
    for kernel, n in scratch.items():
        assert int(n) <= (32 if "sample_rest_kernelILb1" in kernel else 0), f"{kernel}: {n} bytes a lane"
