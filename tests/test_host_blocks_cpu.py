"""-m "not gpu": the store of pinned host memory blocks (what a ctx takes from it and gives back), compiled for the
host on counted memory."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_blocks_are_kept_within_bounds_and_not_allocated_again_and_again(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    exe = str(tmp_path / "host_blocks_driver")
    build = subprocess.run([gxx, "-O1", "-g", "-std=c++17", "-Wall", os.path.join(HERE, "host_blocks_driver.cpp"), "-o", exe, "-pthread"],
                           capture_output=True, text=True, timeout=300)
    assert build.returncode == 0, build.stderr
    run = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0 and run.stdout.startswith("host_blocks_driver ok"), run.stdout + run.stderr
