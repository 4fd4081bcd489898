"""The built library's launches, without a GPU.  The names under which kernels are timed are the names a profiler shows, so that
rollout_kernel_stats and a rocprofv3 summary can be joined (bench.py does): compared with the launch stubs.  And what a
launcher refuses."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2506_06122_amd import binding, build


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


def test_every_sampler_kernel_is_timed_under_its_own_name():
    nm = shutil.which("nm")
    if not nm:
        pytest.skip("no nm")
    path = binding.load_library()._name
    stubs = subprocess.run([nm, "-C", path], capture_output=True, text=True, check=True).stdout
    kernels = {m.group(1).replace(" ", "") for m in re.finditer(r"__device_stub__(sample_\w+(?:<[^>]*>)?)\(", stubs)}
    assert len(kernels) == 4, kernels
    with open(path, "rb") as fh:
        strings = set(fh.read().split(b"\0"))
    assert all(k.encode() in strings for k in kernels), kernels


def test_decode_attention_refuses_what_its_kernel_leaves_out(tmp_path):
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    lib = binding.load_library()._name
    out = str(tmp_path / "driver")
    src = os.path.join(os.path.dirname(os.path.abspath(__file__)), "host", "attn_launch_driver.cpp")
    res = subprocess.run([build.HIPCC, *build.FLAGS, "-x", "hip", src, "-x", "none", lib, "-Wl,-rpath," + os.path.dirname(lib), "-o", out],
                         capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr
    res = subprocess.run([out], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, res.stdout + res.stderr
