"""The tile launch's mapping of workgroups to blocks (csrc/tile_grid.h), the choice of tile shapes (csrc/tile_plan.h) and of the
streamed projections' shapes (csrc/stream_plan.h), plain integers and floats, on the CPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def run_driver(name, tmp_path):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no host C++ compiler")
    out = str(tmp_path / name)
    res = subprocess.run([cxx, "-std=c++17", "-O2", "-Wall", "-Wextra", "-Werror",
                          os.path.join(ROOT, "tests", "host", name + ".cpp"), "-o", out], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    res = subprocess.run([out], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr
    return res.stdout


def test_every_block_is_visited_once(tmp_path):
    assert int(run_driver("tile_grid_driver", tmp_path).split()[0]) > 1000


def test_a_plan_is_evaluated_once(tmp_path):
    assert run_driver("tile_plan_driver", tmp_path).count("plans") == 4


def test_streamed_plans_are_near_the_best_measured(tmp_path):
    assert int(run_driver("stream_plan_driver", tmp_path).split()[0]) > 100000
