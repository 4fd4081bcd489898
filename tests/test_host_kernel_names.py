"""The names under which kernels are timed are the names a profiler shows, so that rollout_kernel_stats and a
rocprofv3 summary can be joined (bench.py does).  Compared with the launch stubs of the built library."""
import re
import shutil
import subprocess

import pytest

from paper_2506_06122_amd import binding


def test_every_projection_and_attention_kernel_is_timed_under_its_own_name():
    nm = shutil.which("nm")
    if not nm:
        pytest.skip("no nm")
    path = binding.load_library()._name
    stubs = subprocess.run([nm, "-C", path], capture_output=True, text=True, check=True).stdout
    kernels = {m.group(1).replace(" ", "")
               for m in re.finditer(r"__device_stub__((?:gemm_|attn_decode_)\w+<[^>]*>)\(", stubs)}
    assert len(kernels) > 30
    with open(path, "rb") as fh:
        literals = {m.decode() for m in re.findall(rb"(?:gemm_|attn_decode_)\w+<[0-9a-z,]+>", fh.read())}
    assert not kernels - literals, sorted(kernels - literals)
